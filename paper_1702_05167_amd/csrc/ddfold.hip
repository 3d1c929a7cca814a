// Algorithms 1 and 2 in double-double: frontal assembly, blocked Gauss-Jordan
// inversion of the pivot blocks, the multiplier / Schur-update products, and the
// row kernels of the extraction (gathers, lesser-channel seeds, diagonals).  Same
// structure as the FP64 kernels (inverse.hip, gemm.hip, kernels.hip); every value
// is a complex double-double (dd.h) and the products run on the FP64 vector units
// (on this chip their peak equals the FP64 matrix cores', and double-double needs
// the error-free fused multiply-add).
#include <hip/hip_runtime.h>

#include "dd.h"
#include "kern.h"

namespace hsc {

namespace {

constexpr int RB = 256;

// ---------------------------------------------------------------------------------------------
// assembly: F[a][b] = sum_children U_k[invrel_k[a]][invrel_k[b]] + (-H)[a][b] + delta_ab (z - Sigma_a - U_a)
__global__ __launch_bounds__(RB) void k_dd_assemble(const RowJob* __restrict__ jobs,
                                                    const int32_t* __restrict__ row_job,
                                                    const EnergyScalars* __restrict__ es) {
  const int g = blockIdx.x;
  const RowJob& jb = jobs[row_job[g]];
  const int a = g - jb.row_off;
  const int cols = jb.cols;
  const ChildRef* kids = reinterpret_cast<const ChildRef*>(jb.p0);
  const FrontSparse* fs = reinterpret_cast<const FrontSparse*>(jb.p1);
  const int nk = jb.aux0, n = jb.aux1, nL = jb.aux2, nR = jb.aux3;
  __shared__ int s_col[64];
  __shared__ double2 s_val[64];
  const int q0 = fs->ptr[a], q1 = fs->ptr[a + 1];
  const int nq = min(q1 - q0, 64);
  if (threadIdx.x < nq) {
    s_col[threadIdx.x] = fs->col[q0 + threadIdx.x];
    s_val[threadIdx.x] = fs->val[q0 + threadIdx.x];
  }
  __syncthreads();
  zdd diag_add = zdd_zero();
  if (a < n) {   // z - Sigma_a, as the exact sum of the two FP64 inputs
    const EnergyScalars& s = es[jb.e];
    if (a < nL + nR) {
      const double2 sg = a < nL ? s.sig[0] : s.sig[1];
      diag_add = zdd{two_sum(s.z.x, -sg.x), two_sum(s.z.y, -sg.y)};
    } else {
      diag_add = zdd_from(s.z);
    }
    if (fs->pot) diag_add.re = dd_add(diag_add.re, dd{-fs->pot[a], 0.0});
  }
  zdd* out = reinterpret_cast<zdd*>(jb.dst) + (int64_t)a * jb.ldd;
  // whole-face contact cluster: minus its dense self-energy block (rows and columns < nface)
  const int nface = jb.aux4;
  const double2* dsig = a < nface ? reinterpret_cast<const double2*>(jb.p2) : nullptr;
  for (int b = threadIdx.x; b < cols; b += RB) {
    zdd v = zdd_zero();
    for (int k = 0; k < nk; ++k) {
      const int ia = kids[k].invrel[a];
      if (ia < 0) continue;
      const int ib = kids[k].invrel[b];
      if (ib < 0) continue;
      v = zdd_add(v, reinterpret_cast<const zdd*>(kids[k].U)[(int64_t)ia * kids[k].ldU + ib]);
    }
    for (int q = 0; q < nq; ++q)
      if (s_col[q] == b) v = zdd_add(v, zdd_from(s_val[q]));
    for (int q = q0 + 64; q < q1; ++q)
      if (fs->col[q] == b) v = zdd_add(v, zdd_from(fs->val[q]));
    if (b == a) v = zdd_add(v, diag_add);
    if (dsig && b < nface) {
      const double2 sv = dsig[(int64_t)a * nface + b];
      v = zdd_sub(v, zdd_from(sv));
    }
    out[b] = v;
  }
}

// ---------------------------------------------------------------------------------------------
// Gauss-Jordan in double-double with partial pivoting inside the block and no row interchanges: the pivot
// row p_k of column k stays where it is (piv[k] = p_k, mark[p_k] = 1), later columns choose among the
// unmarked rows, and the inverse comes out permuted: X[p_j][k] = (A^-1)[j][p_k].
constexpr int PT = 512;

// largest of a wave's 64 lanes, or of the last LANES <= 8 of every 16 (which all hold the same keys), in scalar registers
template <int LANES>
__device__ __forceinline__ uint32_t wave_max_u32(uint32_t v) {
#define HSC_DPP_MAX(ctrl) v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, ctrl, 0xf, 0xf, false))
  if (LANES > 1) HSC_DPP_MAX(0x111);   // row_shr 1, 2, 4, 8: lane 15 of every 16 has the row's largest
  if (LANES > 2) HSC_DPP_MAX(0x112);
  if (LANES > 4) HSC_DPP_MAX(0x114);
  if (LANES > 8) HSC_DPP_MAX(0x118);
  if (LANES > 16) {
    HSC_DPP_MAX(0x142);   // row_bcast 15, 31: lane 63 has the wave's
    HSC_DPP_MAX(0x143);
  }
#undef HSC_DPP_MAX
  return (uint32_t)__builtin_amdgcn_readlane((int)v, LANES > 16 ? 63 : 15);
}

// a row that may become the pivot: the bits of its |Re| + |Im| (the upper word plus one, 0 = no row) and its index
struct alignas(16) PivotKey {
  uint32_t hi, lo;
  int row;
};
// larger, or as large and the earlier row
__device__ __forceinline__ bool pivot_before(PivotKey a, PivotKey b) {
  return a.hi > b.hi || (a.hi == b.hi && (a.lo > b.lo || (a.lo == b.lo && a.row < b.row)));
}
// the lane with the first in that order of a wave's keys (of LANES <= 8 keys that the lanes hold in turn): the upper
// words decide unless two are equal
template <int LANES>
__device__ __forceinline__ int pivot_lane(PivotKey k) {
  constexpr uint64_t lanes = LANES == 64 ? ~0ull : (1ull << (LANES & 63)) - 1;
  const uint32_t hi = wave_max_u32<LANES>(k.hi);
  uint64_t at = __ballot(k.hi == hi) & lanes;
  if (hi != 0 && (at & (at - 1)) != 0) {
    const uint32_t lo = wave_max_u32<LANES>(k.hi == hi ? k.lo : 0u);
    const bool equal = k.hi == hi && k.lo == lo;
    const uint32_t last = wave_max_u32<LANES>(equal ? 4095u - (uint32_t)k.row : 0u);
    at = __ballot(equal && (uint32_t)k.row == 4095u - last) & lanes;
  }
  return __builtin_ctzll(at);
}

// One panel of NB columns from k0, one workgroup per matrix, each thread RPT rows.  A serial chain of NB
// column steps: pivot search, reciprocal, update of the panel.  The pivot is the row with the largest
// |Re| + |Im| in FP64, the first of equals: one maximum over the upper words (20 mantissa bits) finds it unless
// two of a wave's rows are equal there (inverses of order 128 to 256 take 3 to 5 % longer than with keys of 8
// mantissa bits and the row in one word; waves offering their rows before the search ends, which saves a barrier,
// take 4 % more again).  Every thread forms the reciprocal itself (no round trip through LDS), and the columns
// rotate through the registers so that the step's code is a loop body (the current column is P[.][0]).
// Columns are read and written a column at a time, rows side by side, in the T workspace: the finished panel
// as its first NB rows (zero beyond nb), the next panel's columns in the NB rows after (from its rank update; the
// first panel of a super-panel comes from X).  Row by row in X every lane touched a line of its own: 39 and 62 us
// a panel for n = 500 and 1024 (4 matrices) instead of 30 and 48 (with the keys of 8 bits).  Also written: R (NB x n) =
// the pivot rows' old values in the other columns of the super-panel (zero in the panel's own and beyond its nb columns).
template <int TH, int RPT, int NB>
__global__ __launch_bounds__(TH) __attribute__((amdgpu_waves_per_eu(1, 2))) void k_dd_inv_panel(
    const InvJobDD* __restrict__ jobs, int k0, int s0, int sw, int32_t* __restrict__ status) {
  const InvJobDD jb = jobs[blockIdx.x];
  const int n = jb.n;
  if (k0 >= n) return;
  const int nb = min(NB, n - k0);
  const int t = threadIdx.x, lane = t & 63, w = t >> 6;
  __shared__ PivotKey red[2][TH / 64];
  __shared__ zdd rowp[2][NB];
  __shared__ int prows[NB];
  bool bad = false;

  zdd P[RPT][NB];
  bool open[RPT];   // not a pivot row yet
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = t + q * TH;
    open[q] = r < n && (k0 == 0 || jb.mark[r] == 0);
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      P[q][j] = zdd_zero();
      if (r < n && j < nb)
        P[q][j] = load_zdd(k0 > s0 ? jb.T + (int64_t)(NB + j) * n + r : jb.X + (int64_t)r * jb.ld + k0 + j);
    }
  }
#pragma unroll 1
  for (int j = 0; j < nb; ++j) {
    const int par = j & 1;
    // this thread's largest open row, its wave's, the workgroup's
    PivotKey key{0u, 0u, 0};
#pragma unroll
    for (int q = 0; q < RPT; ++q)
      if (open[q]) {
        const double v = zdd_cabs1(P[q][0]);
        // (a NaN too is a row)
        const PivotKey c{((uint32_t)__double2hiint(v) & 0x7fffffffu) + 1u, (uint32_t)__double2loint(v), t + q * TH};
        if (RPT == 1 || pivot_before(c, key)) key = c;
      }
    int first = pivot_lane<64>(key);
    if (TH > 64) {
      if (lane == first) red[par][w] = key;
      __syncthreads();
      key = red[par][lane % (TH / 64)];
      first = pivot_lane<(TH > 64 ? TH / 64 : 64)>(key);
    }
    const int prow = __builtin_amdgcn_readlane(key.row, first);
#pragma unroll
    for (int q = 0; q < RPT; ++q)
      if (t + q * TH == prow) {
#pragma unroll
        for (int jj = 0; jj < NB; ++jj) rowp[par][jj] = P[q][jj];
      }
    __syncthreads();
    const zdd pivv = rowp[par][0];
    const zdd inv = zdd_rcp(pivv);
    bad = bad || !(zdd_cabs1(pivv) > 0.0) || !isfinite(pivv.re.hi) || !isfinite(pivv.im.hi);
    if (t == 0) prows[j] = prow;
    zdd g[RPT];
#pragma unroll
    for (int q = 0; q < RPT; ++q) {
      g[q] = zdd_neg(zdd_mul(P[q][0], inv));
      if (t + q * TH == prow) {   // the pivot row becomes inv times itself
        g[q] = inv;
        open[q] = false;
#pragma unroll
        for (int jj = 1; jj < NB; ++jj) P[q][jj] = zdd_zero();
      }
    }
#pragma unroll
    for (int jj = 1; jj < NB; ++jj) {
      const zdd b = rowp[par][jj];
#pragma unroll
      for (int q = 0; q < RPT; ++q) {
        zddacc a = zddacc_from(P[q][jj]);
        zddacc_fma(a, g[q], b);
        P[q][jj - 1] = zddacc_value(a);
      }
    }
#pragma unroll
    for (int q = 0; q < RPT; ++q) P[q][NB - 1] = g[q];
  }
  // after nb rotations P[q][i] holds column (i + nb) mod NB of the panel
  const int ws = min(s0 + sw, n) - s0;
  const bool alone = ws <= NB;   // no other columns: no rank update, which would bring these to X
  __syncthreads();
#pragma unroll
  for (int q = 0; q < RPT; ++q) {
    const int r = t + q * TH;
    if (r < n) {
      jb.mark[r] = open[q] ? 0 : 1;
#pragma unroll
      for (int i = 0; i < NB; ++i) {
        const int j = i + nb < NB ? i + nb : i + nb - NB;
        const zdd v = j < nb ? P[q][i] : zdd_zero();
        if (!alone) store_zdd(jb.T + (int64_t)j * n + r, v);
        else if (j < nb) store_zdd(jb.X + (int64_t)r * jb.ld + k0 + j, v);
      }
    }
  }
  if (t < nb) jb.piv[k0 + t] = prows[t];
  for (int i = t; i < NB * ws; i += TH) {
    const int j = i / ws, c = s0 + i % ws;
    jb.R[(int64_t)j * n + c] =
        (j >= nb || (c >= k0 && c < k0 + nb)) ? zdd_zero() : jb.X[(int64_t)prows[j] * jb.ld + c];
  }
  if (t == 0 && bad && status) atomicMin(&status[jb.e], (int32_t)HSC_E_SINGULAR);
}

// X[r][c] += sum_k T[k][r] R[k][c] over the super-panel's columns [s0, s0 + ns), T = the finished panel less the
// identity at its pivots.  The panel's own columns (where R is zero) come from the T workspace to X, the next
// panel's go from X to the T workspace (k_dd_inv_panel).  A lane holds one column
// and its NB values of R, a wave walks rows, whose T values wait in LDS.  Super-panels of at most 32 or 16
// columns (the last of a matrix) put 2 or 4 rows side by side in a wave.  Bound by the vector units: 50 FP64
// instructions per complex multiply-add, 1.74 ps at their measured 2.3 ns a wave; 55e6 of them (16^3, 32
// energies, 108e3 rows) take 150 us, 2.7 ps (2.4 without the two panels' detour through the T workspace, which
// saves the panel kernel 12 us and on smaller launches costs nothing).  The grouped product that
// this replaces took 158 us, and 13 us against 7 us for one small matrix.
constexpr int kRankRows = 32;   // rows of a workgroup at most

template <int NB, int CW>
__device__ __forceinline__ void inv_rank_rows(const InvJobDD& jb, const zdd* T, int k0, int s0, int ns, int r0, int rows,
                                              int lane) {
  constexpr int RS = 64 / CW;   // rows side by side
  const int n = jb.n, c = lane % CW, q = lane / CW;
  if (c >= ns) return;
  const zdd* R = jb.R + s0 + c;
  const int j = s0 + c - k0;   // column of this panel (j < NB), of the next one (j < 2 NB)
  zdd* const X = jb.X + (int64_t)r0 * jb.ld + s0 + c;
  zdd* const buf = jb.T + (int64_t)j * n + r0;
  const bool own = j >= 0 && j < NB, next = j >= NB && j < 2 * NB;
  const zdd* const src = own ? buf : X;
  zdd* const dst = next ? buf : X;
  const int64_t ls = own ? 1 : jb.ld, ld = next ? 1 : jb.ld;
  const int last = rows - 1;
  int i = q;
  // (rows beyond the end are read at the last one and not written)
  zdd x0 = load_zdd(src + min(i, last) * ls), x1 = load_zdd(src + min(i + RS, last) * ls);
  zdd b[NB];
#pragma unroll
  for (int k = 0; k < NB; ++k) b[k] = load_zdd(R + (int64_t)k * n);
#pragma unroll 1
  for (;;) {
    const zdd y0 = load_zdd(src + min(i + 2 * RS, last) * ls), y1 = load_zdd(src + min(i + 3 * RS, last) * ls);
    zddacc a0 = zddacc_from(x0), a1 = zddacc_from(x1);
#pragma unroll
    for (int k = 0; k < NB; ++k) {
      zddacc_fma(a0, T[min(i, last) * NB + k], b[k]);
      zddacc_fma(a1, T[min(i + RS, last) * NB + k], b[k]);
    }
    if (i < rows) store_zdd(dst + i * ld, zddacc_value(a0));
    if (i + RS < rows) store_zdd(dst + (i + RS) * ld, zddacc_value(a1));
    i += 2 * RS;
    if (i >= rows) return;
    x0 = y0;
    x1 = y1;
  }
}

template <int NB>
__global__ __launch_bounds__(256) void k_dd_inv_rank(const InvJobDD* __restrict__ jobs, int k0, int s0, int sw,
                                                     int rows_w, int chunks) {
  __shared__ zdd T[kRankRows * NB];
  const InvJobDD jb = jobs[blockIdx.x / chunks];
  const int n = jb.n, ns = min(s0 + sw, n) - s0;
  const int b0 = (int)(blockIdx.x % chunks) * 4 * rows_w;
  if (k0 >= n || ns <= NB || b0 >= n) return;   // (at most NB columns: no others)
  const int rows_b = min(4 * rows_w, n - b0);
  for (int i = threadIdx.x; i < 4 * rows_w * NB; i += 256) {
    const int k = i / (4 * rows_w), r = i % (4 * rows_w);
    if (r < rows_b) {
      zdd v = load_zdd(jb.T + (int64_t)k * n + b0 + r);
      if (k0 + k < n && jb.piv[k0 + k] == b0 + r) v.re = dd_add(v.re, dd_from(-1.0));
      T[r * NB + k] = v;
    }
  }
  __syncthreads();
  const int w = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int rows = min(rows_w, rows_b - w * rows_w);
  if (rows <= 0) return;
  const zdd* Tw = T + w * rows_w * NB;
  if (ns > 32) inv_rank_rows<NB, 64>(jb, Tw, k0, s0, ns, b0 + w * rows_w, rows, lane);
  else if (ns > 16) inv_rank_rows<NB, 32>(jb, Tw, k0, s0, ns, b0 + w * rows_w, rows, lane);
  else inv_rank_rows<NB, 16>(jb, Tw, k0, s0, ns, b0 + w * rows_w, rows, lane);
}

// After the panels of the columns [s0, s0 + ws), ws <= W, of a matrix with other columns to update:
//   U[r][c] = X[r][s0 + c] - (r == p_(s0 + c))   (n x ws, row stride W; the T workspace)
//   R[c][j] = X[p_(s0 + c)][j]                     (ws x n; the R workspace)
__global__ __launch_bounds__(64) void k_dd_inv_super_u(const InvJobDD* __restrict__ jobs, int s0, int W, int chunks) {
  const InvJobDD jb = jobs[blockIdx.x / chunks];
  const int n = jb.n;
  if (s0 >= n || n <= (W == kDDSuper ? W : kDDBlockMin)) return;
  const int ws = min(W, n - s0);
  const int r0 = (blockIdx.x % chunks) * 16;
  for (int c = threadIdx.x; c < ws; c += 64) {
    const int p = jb.piv[s0 + c];
    for (int r = r0; r < min(n, r0 + 16); ++r) {
      zdd v = jb.X[(int64_t)r * jb.ld + s0 + c];
      if (r == p) v.re = dd_add(v.re, dd_from(-1.0));
      jb.T[(int64_t)r * W + c] = v;
    }
  }
}

__global__ __launch_bounds__(256) void k_dd_inv_super_r(const InvJobDD* __restrict__ jobs, int s0, int W, int chunks) {
  const InvJobDD jb = jobs[blockIdx.x / (W * chunks)];
  const int n = jb.n;
  if (s0 >= n || n <= (W == kDDSuper ? W : kDDBlockMin)) return;
  const int ws = min(W, n - s0);
  const int rem = blockIdx.x % (W * chunks);
  const int c = rem / chunks;
  const int j = (rem % chunks) * 256 + threadIdx.x;
  if (c >= ws || j >= n) return;
  jb.R[(int64_t)c * n + j] = jb.X[(int64_t)jb.piv[s0 + c] * jb.ld + j];
}

// Y[j][p_k] = X[p_j][k], with its rounded copy
__global__ __launch_bounds__(256) void k_dd_inv_unscramble(const InvJobDD* __restrict__ jobs, int rows_per_block,
                                                           int chunks) {
  extern __shared__ int idx[];
  const InvJobDD jb = jobs[blockIdx.x / chunks];
  const int n = jb.n;
  const int r0 = (blockIdx.x % chunks) * rows_per_block;
  if (r0 >= n) return;
  for (int k = threadIdx.x; k < n; k += blockDim.x) idx[jb.piv[k]] = k;
  __syncthreads();
  const int r1 = min(n, r0 + rows_per_block);
  for (int r = r0; r < r1; ++r) {
    const int64_t src = (int64_t)jb.piv[r] * jb.ld;
    for (int j = threadIdx.x; j < n; j += blockDim.x) {
      const zdd v = jb.X[src + idx[j]];
      jb.Y[(int64_t)r * jb.ldy + j] = v;
      jb.Y64[(int64_t)r * jb.ldy64 + j] = zdd_round(v);
    }
  }
}

// ---------------------------------------------------------------------------------------------
// grouped complex double-double GEMM: 256 threads as 16 x 16, each with an RM x RN block of outputs
// (tile BM x BN = 16 RM x 16 RN: 32x32, 64x32, 64x64 or 16x16), three real products per complex
// multiply-add (Gauss; the sums re + im of both operands are formed once, when a tile is staged),
// lazily accumulated (dd.h: ddacc) and renormalised after every 8-deep k step.
//   OPA 0: A'(m,k) = A[m*lda + k];  OPA 1: A'(m,k) = A[k*lda + m]
//   OPB 0: B'(k,n) = B[k*ldb + n];  OPB 1: B'(k,n) = B[n*ldb + k]
constexpr int DK = 8;
constexpr int kDDConfigs = 4;
constexpr int kDDRM[kDDConfigs] = {2, 4, 4, 1}, kDDRN[kDDConfigs] = {2, 2, 4, 1};

template <int OPA, int OPB, int RM, int RN>
__global__ __launch_bounds__(256) void k_dd_gemm(const GemmProbDD* __restrict__ probs,
                                                 const int32_t* __restrict__ tile_prob, int total_tiles, int negate,
                                                 int beta) {
  constexpr int BM = 16 * RM, BN = 16 * RN;
  __shared__ zdd As[DK][BM + 1];
  __shared__ zdd Bs[DK][BN + 1];
  __shared__ dd Ass[DK][BM + 1];   // re + im of each staged element (the third product of the Gauss form)
  __shared__ dd Bss[DK][BN + 1];
  const int per = (total_tiles + 7) >> 3;
  const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
  if (tile >= total_tiles) return;
  const GemmProbDD& pr = probs[tile_prob[tile]];
  const int local = tile - pr.tile_off;
  const int m0 = (local / pr.tiles_n) * BM, n0 = (local % pr.tiles_n) * BN;
  const int M = pr.M, N = pr.N, K = pr.K;
  const int t = threadIdx.x;
  const int tm = (t / 16) * RM, tn = (t % 16) * RN;   // this thread's RM x RN block
  // three real products per complex multiply-add (Gauss): t1 = sum ar br, t2 = sum ai bi,
  // t3 = sum (ar + ai)(br + bi); re = t1 - t2, im = t3 - t1 - t2
  ddacc t1[RM][RN], t2[RM][RN], t3[RM][RN];
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j) t1[i][j] = t2[i][j] = t3[i][j] = ddacc{0.0, 0.0};
  for (int k0 = 0; k0 < K; k0 += DK) {
    // stage A' (BM x DK) and B' (DK x BN); the 16 x 16 tile takes half the threads for each
#pragma unroll
    for (int u = 0; u < (RM + 1) / 2; ++u) {
      const int idx = t + u * 256;
      if (RM == 1 && idx >= BM * DK) break;
      const int mm = OPA == 0 ? idx / DK : idx % BM;
      const int kk = OPA == 0 ? idx % DK : idx / BM;
      const int gm = m0 + mm, gk = k0 + kk;
      zdd v = zdd_zero();
      if (gm < M && gk < K) v = OPA == 0 ? pr.A[(int64_t)gm * pr.lda + gk] : pr.A[(int64_t)gk * pr.lda + gm];
      As[kk][mm] = v;
      Ass[kk][mm] = dd_add(v.re, v.im);
    }
#pragma unroll
    for (int u = 0; u < (RN + 1) / 2; ++u) {
      const int idx = RN == 1 ? t - BM * DK : t + u * 256;
      if (RN == 1 && idx < 0) break;
      const int bk = OPB == 0 ? idx / BN : idx % DK;
      const int bn = OPB == 0 ? idx % BN : idx / DK;
      const int gbk = k0 + bk, gbn = n0 + bn;
      zdd v = zdd_zero();
      if (gbk < K && gbn < N) v = OPB == 0 ? pr.B[(int64_t)gbk * pr.ldb + gbn] : pr.B[(int64_t)gbn * pr.ldb + gbk];
      Bs[bk][bn] = v;
      Bss[bk][bn] = dd_add(v.re, v.im);
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < DK; ++kk) {
      zdd a[RM], b[RN];
      dd sa[RM], sb[RN];
#pragma unroll
      for (int i = 0; i < RM; ++i) { a[i] = As[kk][tm + i]; sa[i] = Ass[kk][tm + i]; }
#pragma unroll
      for (int j = 0; j < RN; ++j) { b[j] = Bs[kk][tn + j]; sb[j] = Bss[kk][tn + j]; }
#pragma unroll
      for (int i = 0; i < RM; ++i)
#pragma unroll
        for (int j = 0; j < RN; ++j) {
          ddacc_add_prod(t1[i][j], a[i].re, b[j].re);
          ddacc_add_prod(t2[i][j], a[i].im, b[j].im);
          ddacc_add_prod(t3[i][j], sa[i], sb[j]);
        }
    }
#pragma unroll
    for (int i = 0; i < RM; ++i)
#pragma unroll
      for (int j = 0; j < RN; ++j) {
        ddacc_renorm(t1[i][j]);
        ddacc_renorm(t2[i][j]);
        ddacc_renorm(t3[i][j]);
      }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < RM; ++i)
#pragma unroll
    for (int j = 0; j < RN; ++j) {
      const int row = m0 + tm + i, col = n0 + tn + j;
      if (row < M && col < N) {
        const dd v1 = two_sum(t1[i][j].hi, t1[i][j].lo), v2 = two_sum(t2[i][j].hi, t2[i][j].lo);
        const dd v3 = two_sum(t3[i][j].hi, t3[i][j].lo);
        const zdd v{dd_sub(v1, v2), dd_sub(dd_sub(v3, v1), v2)};
        zdd o = negate ? zdd_neg(v) : v;
        if (beta) o = zdd_add(o, pr.C[(int64_t)row * pr.ldc + col]);
        pr.D[(int64_t)row * pr.ldd + col] = o;
        if (pr.D64) pr.D64[(int64_t)row * pr.ldd64 + col] = zdd_round(o);
      }
    }
}

template <int RM, int RN>
void dd_gemm_dispatch(hipStream_t st, int opA, int opB, const GemmProbDD* probs, const int32_t* tile_prob,
                      int total_tiles, int negate, int beta) {
  const dim3 g(((total_tiles + 7) / 8) * 8), b(256);
  if (opA == 0 && opB == 0)
    hipLaunchKernelGGL((k_dd_gemm<0, 0, RM, RN>), g, b, 0, st, probs, tile_prob, total_tiles, negate, beta);
  else if (opA == 1 && opB == 0)
    hipLaunchKernelGGL((k_dd_gemm<1, 0, RM, RN>), g, b, 0, st, probs, tile_prob, total_tiles, negate, beta);
  else if (opA == 0)
    hipLaunchKernelGGL((k_dd_gemm<0, 1, RM, RN>), g, b, 0, st, probs, tile_prob, total_tiles, negate, beta);
  else
    hipLaunchKernelGGL((k_dd_gemm<1, 1, RM, RN>), g, b, 0, st, probs, tile_prob, total_tiles, negate, beta);
}

// ---------------------------------------------------------------------------------------------
// extraction row kernels (Algorithm 2 and the lesser channels), as in kernels.hip

// dst[r][c] = op(trans ? src[cmap[c]][rmap[r]] : src[rmap[r]][cmap[c]]);  op 1 = -conj
template <int TRANS, int OP>
__global__ __launch_bounds__(RB) void k_dd_gather(const RowJob* __restrict__ jobs,
                                                  const int32_t* __restrict__ row_job) {
  const int g = blockIdx.x;
  const RowJob& jb = jobs[row_job[g]];
  const int r = g - jb.row_off;
  const int rr = jb.rmap ? jb.rmap[r] : r;
  const int32_t* __restrict__ cmap = jb.cmap;
  const zdd* __restrict__ src = reinterpret_cast<const zdd*>(jb.src);
  zdd* __restrict__ out = reinterpret_cast<zdd*>(jb.dst) + (int64_t)r * jb.ldd;
  for (int c = threadIdx.x; c < jb.cols; c += RB) {
    const int cc = cmap ? cmap[c] : c;
    zdd v = TRANS ? src[(int64_t)cc * jb.lds + rr] : src[(int64_t)rr * jb.lds + cc];
    if (OP == 1) v.re = dd_neg(v.re);
    out[c] = v;
  }
}

// NF[rr][b] = sum_children U_k[invrel_k[a(rr)]][b] + seed(rr, b), the seed i * w * conj(G[a][b])
// on the contact rows (argument layout of k_assemble_n)
__global__ __launch_bounds__(RB) void k_dd_assemble_n(const RowJob* __restrict__ jobs,
                                                      const int32_t* __restrict__ row_job,
                                                      const EnergyScalars* __restrict__ es, int channel) {
  const int g = blockIdx.x;
  const RowJob& jb = jobs[row_job[g]];
  const int rr = g - jb.row_off;
  const ChildRef* kids = reinterpret_cast<const ChildRef*>(jb.p0);
  const int nk = jb.aux0, r = jb.aux1, row0 = jb.aux2, n = jb.aux3, nL = jb.aux4, nR = jb.aux5;
  const int a = rr < r ? row0 + rr : n + (rr - r);
  // whole-face contact: p1 holds Gamma G (same leading dimension) and w is the occupation alone
  const zdd* gam_g = reinterpret_cast<const zdd*>(jb.p1);
  double w = 0.0;
  if (rr < r && a < nL + nR)
    w = gam_g ? channel_occ(es[jb.e], channel, a < nL ? 0 : 1) : channel_weight(es[jb.e], channel, a < nL ? 0 : 1);
  const zdd* grow = (gam_g ? gam_g : reinterpret_cast<const zdd*>(jb.src)) + (int64_t)a * jb.lds;
  zdd* out = reinterpret_cast<zdd*>(jb.dst) + (int64_t)rr * jb.ldd;
  for (int b = threadIdx.x; b < jb.cols; b += RB) {
    zdd v = zdd_zero();
    for (int k = 0; k < nk; ++k) {
      const int ia = kids[k].invrel[a];
      if (ia >= 0) v = zdd_add(v, reinterpret_cast<const zdd*>(kids[k].U)[(int64_t)ia * kids[k].ldU + b]);
    }
    if (w != 0.0) {
      const zdd gv = grow[b];
      v.re = dd_add(v.re, dd_mul(dd_from(w), gv.im));
      v.im = dd_add(v.im, dd_mul(dd_from(w), gv.re));
    }
    out[b] = v;
  }
}

__device__ __forceinline__ double shfl_xor_d(double v, int off) { return __shfl_xor(v, off, 64); }

// diagonal outputs, one wave per row, rounded to complex128 at the store (modes of k_diag)
template <int MODE>
__global__ __launch_bounds__(RB) void k_dd_diag(const RowJob* __restrict__ jobs, const int32_t* __restrict__ row_job,
                                                int total_rows, int out_kind, void* out, int64_t out_stride,
                                                int e_base, int nvalid) {
  const int g = blockIdx.x * (RB / 64) + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (g >= total_rows) return;
  const RowJob& jb = jobs[row_job[g]];
  const int k = g - jb.row_off;
  if (jb.e >= nvalid) return;
  const zdd* src = reinterpret_cast<const zdd*>(jb.src);
  zdd v = zdd_zero();
  if (MODE == DIAG_SEP) {
    v = src[(int64_t)k * jb.lds + k];
  } else {
    const int f = jb.aux0;
    const zdd* psi = reinterpret_cast<const zdd*>(jb.p0) + (int64_t)k * f;
    const zdd* x = src + (int64_t)k * jb.lds;
    zdd acc = zdd_zero();
    for (int j = lane; j < f; j += 64) {
      zdd y = x[j];
      if (MODE == DIAG_LEAF_P) y.im = dd_neg(y.im);
      acc = zdd_fma(acc, psi[j], y);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
      zdd o;
      o.re.hi = shfl_xor_d(acc.re.hi, off);
      o.re.lo = shfl_xor_d(acc.re.lo, off);
      o.im.hi = shfl_xor_d(acc.im.hi, off);
      o.im.lo = shfl_xor_d(acc.im.lo, off);
      acc = zdd_add(acc, o);
    }
    const zdd* base = reinterpret_cast<const zdd*>(jb.p1);
    const zdd d = base ? base[(int64_t)k * jb.aux1 + k] : zdd_zero();
    v = MODE == DIAG_LEAF_P ? zdd_sub(d, acc) : zdd_add(d, acc);
  }
  if (lane != 0) return;
  const double2 r = zdd_round(v);
  const int64_t site = reinterpret_cast<const int64_t*>(jb.p2)[k];
  const int64_t idx = (int64_t)(e_base + jb.e) * out_stride + site;
  if (out_kind == OUT_COMPLEX) reinterpret_cast<double2*>(out)[idx] = r;
  else reinterpret_cast<double*>(out)[idx] = r.y;
}

}  // namespace

int dd_gemm_configs() { return kDDConfigs; }
int dd_gemm_tile_m(int config) { return 16 * kDDRM[config]; }
int dd_gemm_tile_n(int config) { return 16 * kDDRN[config]; }
int dd_inv_nb(int max_n) { return max_n <= 1024 ? 8 : max_n <= 2048 ? 4 : 2; }

void launch_dd_gemm(hipStream_t st, int opA, int opB, int config, const GemmProbDD* probs,
                    const int32_t* tile_prob, int total_tiles, int negate, int beta) {
  if (total_tiles <= 0) return;
  if (config == 1) dd_gemm_dispatch<4, 2>(st, opA, opB, probs, tile_prob, total_tiles, negate, beta);
  else if (config == 2) dd_gemm_dispatch<4, 4>(st, opA, opB, probs, tile_prob, total_tiles, negate, beta);
  else if (config == 3) dd_gemm_dispatch<1, 1>(st, opA, opB, probs, tile_prob, total_tiles, negate, beta);
  else dd_gemm_dispatch<2, 2>(st, opA, opB, probs, tile_prob, total_tiles, negate, beta);
}

void launch_dd_gather(hipStream_t st, const RowJob* jobs, const int32_t* row_job, int total_rows, int trans, int op) {
  if (total_rows <= 0) return;
  const dim3 g(total_rows), b(RB);
  if (trans == 0 && op == 0) hipLaunchKernelGGL((k_dd_gather<0, 0>), g, b, 0, st, jobs, row_job);
  else if (trans == 1 && op == 0) hipLaunchKernelGGL((k_dd_gather<1, 0>), g, b, 0, st, jobs, row_job);
  else if (trans == 0) hipLaunchKernelGGL((k_dd_gather<0, 1>), g, b, 0, st, jobs, row_job);
  else hipLaunchKernelGGL((k_dd_gather<1, 1>), g, b, 0, st, jobs, row_job);
}

void launch_dd_assemble_n(hipStream_t st, const RowJob* jobs, const int32_t* row_job, int total_rows,
                          const EnergyScalars* es, int channel) {
  if (total_rows <= 0) return;
  hipLaunchKernelGGL(k_dd_assemble_n, dim3(total_rows), dim3(RB), 0, st, jobs, row_job, es, channel);
}

void launch_dd_diag(hipStream_t st, const RowJob* jobs, const int32_t* row_job, int total_rows, int mode,
                    int out_kind, void* out, int64_t out_stride, int e_base, int nvalid) {
  if (total_rows <= 0) return;
  const dim3 grid((total_rows + RB / 64 - 1) / (RB / 64)), block(RB);
  if (mode == DIAG_SEP)
    hipLaunchKernelGGL(k_dd_diag<DIAG_SEP>, grid, block, 0, st, jobs, row_job, total_rows, out_kind, out,
                       out_stride, e_base, nvalid);
  else if (mode == DIAG_LEAF_G)
    hipLaunchKernelGGL(k_dd_diag<DIAG_LEAF_G>, grid, block, 0, st, jobs, row_job, total_rows, out_kind, out,
                       out_stride, e_base, nvalid);
  else
    hipLaunchKernelGGL(k_dd_diag<DIAG_LEAF_P>, grid, block, 0, st, jobs, row_job, total_rows, out_kind, out,
                       out_stride, e_base, nvalid);
}

void launch_dd_assemble(hipStream_t st, const RowJob* jobs, const int32_t* row_job, int total_rows,
                        const EnergyScalars* es) {
  if (total_rows <= 0) return;
  hipLaunchKernelGGL(k_dd_assemble, dim3(total_rows), dim3(RB), 0, st, jobs, row_job, es);
}

void launch_dd_inv_panel(hipStream_t st, const InvJobDD* jobs, int njobs, int k0, int s0, int sw, int max_n,
                         int32_t* status) {
  if (njobs <= 0 || max_n > 8 * PT) return;
  const dim3 g(njobs);
  // as few waves as hold the rows: they share the CU's vector units
  if (max_n <= 64) hipLaunchKernelGGL((k_dd_inv_panel<64, 1, 8>), g, dim3(64), 0, st, jobs, k0, s0, sw, status);
  else if (max_n <= 128) hipLaunchKernelGGL((k_dd_inv_panel<128, 1, 8>), g, dim3(128), 0, st, jobs, k0, s0, sw, status);
  else if (max_n <= 256) hipLaunchKernelGGL((k_dd_inv_panel<256, 1, 8>), g, dim3(256), 0, st, jobs, k0, s0, sw, status);
  else if (max_n <= 512) hipLaunchKernelGGL((k_dd_inv_panel<512, 1, 8>), g, dim3(512), 0, st, jobs, k0, s0, sw, status);
  else if (max_n <= 1024) hipLaunchKernelGGL((k_dd_inv_panel<512, 2, 8>), g, dim3(512), 0, st, jobs, k0, s0, sw, status);
  else if (max_n <= 2048) hipLaunchKernelGGL((k_dd_inv_panel<512, 4, 4>), g, dim3(512), 0, st, jobs, k0, s0, sw, status);
  else hipLaunchKernelGGL((k_dd_inv_panel<512, 8, 2>), g, dim3(512), 0, st, jobs, k0, s0, sw, status);
}

void launch_dd_inv_rank(hipStream_t st, const InvJobDD* jobs, int njobs, int k0, int s0, int sw, int max_n) {
  if (njobs <= 0 || k0 >= max_n) return;
  // 8 rows of a wave share its R values (122 us for 512 matrices of order 216, 133 us with 4 and 158 us with
  // 2, X alone); fewer where that leaves under 3 waves per SIMD (18 of order 960: 26 us with 8, 23 us with 4)
  int rows_w = kRankRows / 4;
  while (rows_w > 2 && (int64_t)njobs * ((max_n + rows_w - 1) / rows_w) < 3072) rows_w /= 2;
  const int chunks = (max_n + 4 * rows_w - 1) / (4 * rows_w);
  const dim3 g((unsigned)(njobs * chunks)), b(256);
  const int nb = dd_inv_nb(max_n);
  if (nb == 8) hipLaunchKernelGGL((k_dd_inv_rank<8>), g, b, 0, st, jobs, k0, s0, sw, rows_w, chunks);
  else if (nb == 4) hipLaunchKernelGGL((k_dd_inv_rank<4>), g, b, 0, st, jobs, k0, s0, sw, rows_w, chunks);
  else hipLaunchKernelGGL((k_dd_inv_rank<2>), g, b, 0, st, jobs, k0, s0, sw, rows_w, chunks);
}

void launch_dd_inv_super(hipStream_t st, const InvJobDD* jobs, int njobs, int s0, int W, int max_n) {
  if (njobs <= 0 || W <= 0) return;
  const int cu = (max_n + 15) / 16, cr = (max_n + 255) / 256;
  hipLaunchKernelGGL(k_dd_inv_super_u, dim3(njobs * cu), dim3(64), 0, st, jobs, s0, W, cu);
  hipLaunchKernelGGL(k_dd_inv_super_r, dim3(njobs * W * cr), dim3(256), 0, st, jobs, s0, W, cr);
}

void launch_dd_inv_unscramble(hipStream_t st, const InvJobDD* jobs, int njobs, int max_n) {
  if (njobs <= 0) return;
  const int rpb = 16;
  const int chunks = (max_n + rpb - 1) / rpb;
  hipLaunchKernelGGL(k_dd_inv_unscramble, dim3(njobs * chunks), dim3(256), max_n * sizeof(int), st, jobs, rpb,
                     chunks);
}

}  // namespace hsc
