// Complex double-double block products on the integer matrix cores.
//
// The double-double solve forms every block product of Algorithms 1 and 2
// (multipliers, Schur updates, extraction and lesser-channel products) as
// D = (-1)^negate op(A) op(B) + beta C with ~106-bit operands.  Instead of
// emulating double-double arithmetic on the FP64 vector units, each operand is
// rounded to integers of 7 S bits (S = 16, or 15 on request) times a power of
// two per row (of op(A)) or per column (of op(B)):
//
//   x = 2^(e_r - (7 S - 1)) X + rem,   |rem| <= 2^(e_r - 7 S),
//   e_r = exponent with max_k (|Re x_rk| + |Im x_rk|) < 2^e_r,
//
// and the product of the integer matrices is formed exactly from its residues
// modulo 32 small coprime numbers (residue.h): residues are int8, sums over k of
// their products are exact in int32 (v_mfma_i32_16x16x64_i8), and the Chinese
// remainder theorem gives the integers back (Ozaki, Uchino and Imamura, "Ozaki
// Scheme II", 2025).  A complex product takes two real products for each of the
// 18 moduli in which -1 is a square and four for the other 14: 92 int8 products
// of 64 residue planes, where slices of 7 bits (16 per operand, the 136 leading
// pairs, three real products each) take 408 products of 48 planes.
//
// Error: only the operands' rounding and the final double-double operations
// (2^-104 relative, with beta C).  Per k, re and im are each off by at most
// 2^-7S (|a| + |b|) in units of the scales, so a product is within
// 2 K 2^-7S (1 + 2^-7S) 2^(e_i + f_j), i.e. K 2^-109 (S = 16) or K 2^-102 (S = 15)
// times max_k (|Re| + |Im|) of row i of op(A) times the same of column j of
// op(B) (2^e <= twice that maximum).  The bound is relative to the largest
// entries of the row and column, not to sum_k |a_ik| |b_kj|: entries far below
// their row's largest keep fewer bits, which is why S = 16 is the default.
//
// Layout: the residues of one operand are 64 planes of int8 (two per modulus;
// rows padded to 32, K padded to 64 with zeros), each stored as 1 KB
// fragments of 16 rows x 64 k in the order in which the matrix cores take an
// operand: per row block of 16, the planes in sixteen slots of four (modulus 2 s and 2 s + 1), per slot
// the fragments of one k step after the other, four planes each.  A product takes slot after slot,
// so it reads every row block's data as one stream.  Row scales int32 [Rp].
#include <hip/hip_runtime.h>

#include "dd.h"
#include "kern.h"
#include "residue.h"

namespace hsc {

namespace {

typedef int v4i __attribute__((ext_vector_type(4)));

constexpr int OZ_KC = 64;     // k depth of one matrix-core step (v_mfma_i32_16x16x64_i8)
constexpr int OZ_GROUP = 8;   // tile rows per group of the tile order

__constant__ const ResTables kTab = res_tables();

// c mod p_m as a signed byte in the low 8 bits: c - p rint(c / p), the quotient taken from the
// low bits of the rounded float (1.5 2^23 + q; 24-bit product, its 2^22 p does not reach the byte).
// |c| < 2^25 keeps the residue within +-127 of p <= 243 (the quotient's float error stays below
// 2^25 2^-22.4 / p); 256 needs no quotient.
__device__ __forceinline__ int res_byte(int c, int p, float inv) {
  const int q = __float_as_int(fmaf((float)c, inv, 12582912.0f));
  return c + __mul24(q, -p);
}

// The same for sums that start from the bits of the float M = res_bias(p): no conversion.  (M + c) / p misses
// by at most 0.8 / p, so the residue stays within (p + 2) / 2.
__device__ __forceinline__ int res_byte_biased(int s, int p, float inv) {
  if (p == 256) return s;
  const int q = __float_as_int(fmaf(__int_as_float(s), inv, (float)(kResBias - res_bias(p) / p)));
  return s + __mul24(q, -p);
}

// low bytes of four residues in one word
__device__ __forceinline__ uint32_t res_pack(int a, int b, int c, int d) {
  const uint32_t ab = __builtin_amdgcn_perm((uint32_t)b, (uint32_t)a, 0x0c0c0400);
  const uint32_t cd = __builtin_amdgcn_perm((uint32_t)d, (uint32_t)c, 0x0c0c0400);
  return __builtin_amdgcn_perm(cd, ab, 0x05040100);
}

// ---------------------------------------------------------------------------------------------
// splitting

// element (r, k) of the operand as stored: X[r * ldr + k * ldk]; zero outside R x K
// (piv_mode: see OzSplitJob)
__device__ __forceinline__ zdd oz_elem(const OzSplitJob& jb, int r, int k) {
  if (r >= jb.R || k >= jb.K) return zdd_zero();
  if (jb.piv_mode == kOzPlain) return load_zdd(jb.X + (int64_t)r * jb.ldr + (int64_t)k * jb.ldk);
  const int p = ((global_ptr<const int32_t>)jb.piv)[k];
  if (jb.piv_mode == kOzPivotRows) return load_zdd(jb.X + (int64_t)r * jb.ldr + (int64_t)p * jb.ldk);
  zdd v = load_zdd(jb.X + (int64_t)r * jb.ldr + (int64_t)k * jb.ldk);
  if (r == p) v.re = dd_add(v.re, dd_from(-1.0));
  return v;
}

__device__ __forceinline__ double oz_mag(const zdd& v) {
  return (fabs(v.re.hi) + fabs(v.re.lo)) + (fabs(v.im.hi) + fabs(v.im.lo));
}

// the four 28-bit chunks (lowest first) of rint(y), |y| <= 2^111: every step is exact, the last
// one drops the remainder; each chunk as four signed bytes (balanced base-256 digits)
__device__ __forceinline__ v4i oz_chunks(dd y) {
#pragma clang fp contract(off)
  v4i out;
#pragma unroll
  for (int b = 3; b >= 0; --b) {
    const double up = ldexp(1.0, -28 * b), down = ldexp(1.0, 28 * b);
    const double q = rint(y.hi * up);
    const double t = fma(-q, down, y.hi);   // exact: a multiple of ulp(y.hi), at least 2 |y.lo| or zero
    const double hi = t + y.lo;
    y = dd{hi, y.lo - (hi - t)};
    out[b] = ((int)q + 0x00808080) ^ 0x00808080;
  }
  return out;
}

// Scales and residues of sixteen rows of one job, jb.kper steps of 64 k per workgroup (every
// workgroup of a row block takes the maximum over all k; the first one stores the scales).  Wave w takes the
// 16 k from 64 kc + 16 w; lane l holds row l & 15 and the four k = 16 w + (l >> 4) + 4 u, u < 4 (the order
// of k inside a fragment is free as long as both operands use it: byte 4 (l >> 4) + u of the row's
// 16).  The sums over a chunk's bytes run on the matrix cores: the weights of four moduli, block
// diagonal over the four k groups of the operand, times the lane's own 16 bytes give each lane its own
// four sums, at a quarter of the matrix rate but four times that of dot products on the vector units.
//
// Bound by memory: 32 B read, read again from beyond L2, and 64 B written per complex element, 26-30 ps over the
// operands of a 16^3 or 32^3 solve (4.9 TB/s), with the four waves per SIMD that the registers allow (28-31 ps
// with three, accumulators in the other half of the register file and sums converted to float).  Elements
// held in registers instead of read again take those registers: no faster up to K = 128, slower beyond.
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(4, 4))) void k_oz_split(const OzSplitJob* __restrict__ jobs,
                                                  const int32_t* __restrict__ tile_job, int bits) {
  // weights [plane, part][modulus], then as many zeros for the lanes off the block diagonal
  __shared__ v4i wt[2 * 4 * kResMods];
  __shared__ double red[16][16];
  const OzSplitJob jb = jobs[__builtin_amdgcn_readfirstlane(tile_job[blockIdx.x])];
  const int local = blockIdx.x - jb.tile_off;
  const int kcs = jb.Kp / 64, chunks = max(1, (kcs + jb.kper - 1) / jb.kper);
  const int rb = local / chunks, c0 = (local % chunks) * jb.kper;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int g = lane >> 4, ri = lane & 15;
  const v4i zero = {0, 0, 0, 0};
  if (t < 4 * kResMods) wt[t] = reinterpret_cast<const v4i*>(kTab.split)[t];
  else wt[t] = zero;
  // row maxima: red[row][phase]
  if (jb.ldk == 1) {
    // k contiguous: lanes along k, four rows per wave
    double m[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = lane; k < jb.K; k += 64)
#pragma unroll
      for (int i = 0; i < 4; ++i) m[i] = fmax(m[i], oz_mag(oz_elem(jb, 16 * rb + 4 * w + i, k)));
#pragma unroll
    for (int i = 0; i < 4; ++i) {
#pragma unroll
      for (int off = 32; off >= 16; off >>= 1) m[i] = fmax(m[i], __shfl_xor(m[i], off, 64));
      if (g == 0) red[4 * w + i][ri] = m[i];
    }
  } else {
    // rows contiguous (or general strides): lanes along rows, sixteen k phases
    double m[4] = {0.0, 0.0, 0.0, 0.0};
    for (int k = 4 * w + g; k < jb.K; k += 64)
#pragma unroll
      for (int i = 0; i < 4; ++i) m[i] = fmax(m[i], oz_mag(oz_elem(jb, 16 * rb + ri, k + 16 * i)));
    red[ri][4 * w + g] = fmax(fmax(m[0], m[1]), fmax(m[2], m[3]));
  }
  __syncthreads();
  // e with max_k (|Re| + |Im|) of the row < 2^e (0 for a zero row)
  double mx = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) mx = fmax(mx, red[ri][i]);
  int e = 0;
  if (mx > 0.0 && isfinite(mx)) (void)frexp(mx, &e);
  if (c0 == 0 && t < 16) jb.ex[16 * rb + t] = e;
  const int sh = bits - e;
  const v4i* wl = wt + ((ri >> 2) == g ? 0 : 4 * kResMods) + (lane & 3);
  for (int kc = c0; kc < min(kcs, c0 + jb.kper); ++kc) {
    v4i cr[4], ci[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const zdd v = oz_elem(jb, 16 * rb + ri, 64 * kc + 16 * w + g + 4 * u);
      const dd nr = two_sum(v.re.hi, v.re.lo), ni = two_sum(v.im.hi, v.im.lo);
      cr[u] = oz_chunks(dd{ldexp(nr.hi, sh), ldexp(nr.lo, sh)});
      ci[u] = oz_chunks(dd{ldexp(ni.hi, sh), ldexp(ni.lo, sh)});
    }
    int8_t* out = jb.out + (int64_t)rb * kcs * (kResPlanes * 1024) + kc * 4096 + 256 * w + 16 * ri + 4 * g;
    const int slot = kcs * 4096;
#pragma unroll
    for (int q = 0; q < kResMods / 4; ++q)
#pragma unroll
      for (int pl = 0; pl < 2; ++pl) {
        const v4i wr = wl[(2 * pl) * kResMods + 4 * q], wi = wl[(2 * pl + 1) * kResMods + 4 * q];
        const v4i bias = {res_bias_bits(kResModuli[4 * q]), res_bias_bits(kResModuli[4 * q + 1]),
                          res_bias_bits(kResModuli[4 * q + 2]), res_bias_bits(kResModuli[4 * q + 3])};
        v4i s[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          // moduli that do not split: plane 0 is Re alone, plane 1 Im alone
          s[u] = bias;
          if (4 * q < kResSplit || pl == 0) s[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wr, cr[u], s[u], 0, 0, 0);
          if (4 * q < kResSplit || pl == 1) s[u] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wi, ci[u], s[u], 0, 0, 0);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int m = 4 * q + j, p = kResModuli[m];
          const float inv = 1.0f / (float)p;
          *(global_ptr<uint32_t>)(out + (m >> 1) * slot + (2 * (m & 1) + pl) * 1024) =
              res_pack(res_byte_biased(s[0][j], p, inv), res_byte_biased(s[1][j], p, inv),
                       res_byte_biased(s[2][j], p, inv), res_byte_biased(s[3][j], p, inv));
        }
        // (groups of moduli one after the other: interleaved they need 170 registers and two waves per SIMD)
        if (pl == 1) __builtin_amdgcn_sched_barrier(0);
      }
  }
}

// ---------------------------------------------------------------------------------------------
// products of the residues

// 16 bytes per lane from global memory (base + the lane's off) into 1 KB of LDS at byte address `to`
// (base and to wave-uniform).  Written
// as assembly because the compiler, which cannot tell the ring's buffers apart, waits for every such
// load before each LDS read when it knows of them; the kernel's own waits count them.  No register is
// written.
__device__ __forceinline__ void load_lds(const void* base, uint32_t off, uint32_t to) {
  asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %0" ::"s"(base), "v"(off), "s"(to)
               : "memory", "m0");
}
__device__ __forceinline__ const int8_t* uniform(const int8_t* p) {   // a wave-uniform address, in scalar registers
  const uint64_t v = (uint64_t)p;
  return (const int8_t*)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
                         (uint32_t)__builtin_amdgcn_readfirstlane((int)v));
}
__device__ __forceinline__ uint32_t lds_address(const void* p) {
  return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const void*)p;
}

// the four signed bytes of each word negated (-128 stays)
__device__ __forceinline__ v4i neg_bytes(v4i x) {
  v4i r;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    r[i] = (int)((0x80808080u - ((uint32_t)x[i] & 0x7f7f7f7fu)) ^ (~(uint32_t)x[i] & 0x80808080u));
  return r;
}

// Sum of 20 limbs of weights 2^(-8 (l + 1)) taken mod 1 (into [-1/2, 1/2)), as a double-double to
// 2^-133: groups of four limbs are exact in FP64 (|limb| <= 2^19), the leading group wraps in 32 bits.
__device__ __forceinline__ dd res_fraction(const v4i (&L)[5]) {
#pragma clang fp contract(off)
  double x[5];
  x[0] = (double)(int)(((uint32_t)L[0][0] << 24) + ((uint32_t)L[0][1] << 16) + ((uint32_t)L[0][2] << 8) +
                       (uint32_t)L[0][3]) * 0x1p-32;
#pragma unroll
  for (int q = 1; q < 5; ++q)
    x[q] = fma((double)((L[q][0] << 8) + L[q][1]), 65536.0, (double)((L[q][2] << 8) + L[q][3])) *
           ldexp(1.0, -32 * (q + 1));
  const dd s = two_sum(x[0], x[1]);
  dd a = two_sum(s.hi, s.lo + x[2]);          // s.lo + x[2] is exact: multiples of 2^-96 below 2^-51
  const dd b = two_sum(a.lo, x[3] + x[4]);
  a = two_sum(a.hi, b.hi);
  a.lo += b.lo;
  return quick_two_sum(a.hi, a.lo);
}

// One 64 x 32 output tile per workgroup of four waves, two workgroups per CU: one multiplies while the
// other takes residues, reconstructs or starts.  Wave (c, h) forms the rows 32 h .. 32 h + 31 for the
// sixteen moduli 2 slot + c: 16 outputs per lane, whose residues stay in registers (two parts of
// sixteen bytes), so the accumulators of one modulus at a time are all that is live.  The four planes of
// a slot and one 64-deep k step (24 fragments of 1 KB) are staged by direct global-to-LDS loads into a
// ring of kRing buffers.  At the end the two waves of a half swap the residues of half its outputs
// through LDS, and the Chinese remainder sums run on the matrix cores (limbs of the result as int8
// products with the weights' digits, block diagonal as in k_oz_split).
constexpr int kRing = 3, kStage = 24 * 1024;
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void k_oz_gemm(
    const GemmProbOZ* __restrict__ probs, const int32_t* __restrict__ tile_prob, int total_tiles, int scale_bits,
    int negate, int beta) {
  constexpr int kCrt = 2 * 2 * kResLimbs;
  __shared__ v4i lds[kRing * kStage / 16];
  __shared__ v4i crt[2 * kCrt];   // weights, then as many zeros for the lanes off the block diagonal
  const int per = (total_tiles + 7) >> 3;
  const int tile = (blockIdx.x & 7) * per + (blockIdx.x >> 3);   // XCD-aware order
  if (tile >= total_tiles) return;
  const GemmProbOZ pr = probs[__builtin_amdgcn_readfirstlane(tile_prob[tile])];   // held in scalar registers
  const int local = tile - pr.tile_off;
  // tiles of a problem in groups of OZ_GROUP tile rows, column by column inside a group: the tiles
  // an XCD runs at once share a few row and column blocks of the planes in its L2
  const int tm = (pr.Mp + 63) / 64, tn = pr.tiles_n;
  const int grp = local / (OZ_GROUP * tn), idx = local % (OZ_GROUP * tn);
  const int rows = min(OZ_GROUP, tm - grp * OZ_GROUP);
  const int m0 = (grp * OZ_GROUP + idx % rows) * 64, n0 = (idx / rows) * 32;
  const int t = threadIdx.x, lane = t & 63, w = __builtin_amdgcn_readfirstlane(t >> 6);
  const int c = w >> 1, h = w & 1;
  const int kcs = pr.Kp / OZ_KC;
  const v4i zero = {0, 0, 0, 0};
  if (t < 2 * kCrt) crt[t] = t < kCrt ? reinterpret_cast<const v4i*>(kTab.crt)[t] : zero;

  // wave w stages plane w of the slot's four: four row blocks of A (the last one again past the end of
  // an operand that is not a multiple of 64) and two of B
  const uint32_t row = kcs * (kResPlanes * 1024);   // bytes of a row block
  const int8_t* const baseA = uniform(pr.A8 + (int64_t)(m0 / 16) * row + w * 1024);
  const int8_t* const baseB = uniform(pr.B8 + (int64_t)(n0 / 16) * row + w * 1024);
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_address(lds)) + w * 6144;
  uint32_t off[4];
#pragma unroll
  for (int f = 0; f < 4; ++f) off[f] = min(f, pr.Mp / 16 - m0 / 16 - 1) * row + 16 * lane;
  // loads of the next step; past the last one, the last again (its buffer is not read any more)
  uint32_t pos = 0, to = 0;             // of the loads within the row blocks, and in LDS
  auto advance = [&]() {
    to = to == (kRing - 1) * kStage ? 0 : to + kStage;
    pos = __builtin_amdgcn_readfirstlane(min(pos + 4096, row - 4096));
  };

  uint32_t rre[4][4][4], rim[4][4][4];   // residues: [block of 16 x 16][register][word of four slots]
#pragma unroll
  for (int f = 0; f < 4; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r)
#pragma unroll
      for (int q = 0; q < 4; ++q) rre[f][r][q] = rim[f][r][q] = 0;

  if (kcs > 0) {
#pragma unroll
    for (int q = 0; q < kRing; ++q) {
#pragma unroll
      for (int f = 0; f < 4; ++f) load_lds(baseA + pos, off[f], lds0 + to + f * 1024);
#pragma unroll
      for (int f = 0; f < 2; ++f) load_lds(baseB + pos + f * row, 16 * lane, lds0 + to + (4 + f) * 1024);
      advance();
    }
    v4i a0[2], a1[2], b0[2], b1[2];   // operands of one step
    const v4i* const la = &lds[(12 * c + 2 * h) * 64 + lane];
    const v4i* const lb = &lds[(12 * c + 4) * 64 + lane];
    uint32_t buf = 0;                 // of the step's buffer, in LDS
    __builtin_amdgcn_s_waitcnt(0x007c);   // vmcnt(12), lgkmcnt(0): the first step's loads
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      a0[i] = la[i * 64];
      b0[i] = lb[i * 64];
      a1[i] = la[(6 + i) * 64];
      b1[i] = lb[(6 + i) * 64];
    }
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
#pragma nounroll
    for (int slot = 4 * q4; slot < 4 * q4 + 4; ++slot) {
      const bool split = 2 * slot < kResSplit;
      const int p = kTab.p[2 * slot + c];
      const float inv = kTab.inv[2 * slot + c];
      v4i acc0[4], acc1[4];   // block 2 i + j: rows 32 h + 16 i, columns 16 j
#pragma unroll
      for (int f = 0; f < 4; ++f) acc0[f] = acc1[f] = zero;
      // scalar loads are waited for here: pending in the loop, they would turn its partial LDS waits into full ones
      asm volatile("" ::"s"(p), "s"(inv));
      for (int kc = 0; kc < kcs; ++kc) {
        // Loads are issued kRing steps ahead and the operands read from LDS one step ahead, each set as
        // soon as its last product is issued.  Here: this wave's six loads of the next step have landed
        // (the six of the step after may be under way) and this step's operands have been read ...
        __builtin_amdgcn_s_waitcnt(0x0076);   // vmcnt(6), lgkmcnt(0)
        __builtin_amdgcn_s_barrier();         // ... by every wave: this step's buffer takes the new loads
        asm volatile("" ::: "memory");
        const uint32_t dst = lds0 + buf;
        buf = buf == (kRing - 1) * kStage ? 0 : buf + kStage;
        const v4i* const na = la + buf / 16;
        const v4i* const nb = lb + buf / 16;
#define HSC_OZ_MMA(acc, a, b)                                                                                   \
  for (int f = 0; f < 4; ++f) acc[f] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[f >> 1], b[f & 1], acc[f], 0, 0, 0)
        if (split) {
          HSC_OZ_MMA(acc0, a0, b0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            a0[i] = na[i * 64];
            b0[i] = nb[i * 64];
          }
          load_lds(baseA + pos, off[0], dst);
          load_lds(baseA + pos, off[1], dst + 1024);
          load_lds(baseA + pos, off[2], dst + 2048);
          __builtin_amdgcn_sched_barrier(0);
          HSC_OZ_MMA(acc1, a1, b1);
        } else {
          const v4i mb[2] = {neg_bytes(b1[0]), neg_bytes(b1[1])};
          HSC_OZ_MMA(acc0, a0, b0);
          HSC_OZ_MMA(acc1, a0, b1);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 2; ++i) a0[i] = na[i * 64];
          load_lds(baseA + pos, off[0], dst);
          load_lds(baseA + pos, off[1], dst + 1024);
          load_lds(baseA + pos, off[2], dst + 2048);
          __builtin_amdgcn_sched_barrier(0);
          HSC_OZ_MMA(acc0, a1, mb);
          HSC_OZ_MMA(acc1, a1, b0);
          __builtin_amdgcn_sched_barrier(0);
#pragma unroll
          for (int i = 0; i < 2; ++i) b0[i] = nb[i * 64];
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          a1[i] = na[(6 + i) * 64];
          b1[i] = nb[(6 + i) * 64];
        }
        load_lds(baseA + pos, off[3], dst + 3072);
        load_lds(baseB + pos, 16 * lane, dst + 4096);
        load_lds(baseB + pos + row, 16 * lane, dst + 5120);
        advance();
        asm volatile("" ::: "memory");
        if ((kc & 7) == 7 && kc + 1 < kcs) {
          // every 512 of depth the sums go back into [-p/2, p/2]: below 2^25 whatever the depth
#pragma unroll
          for (int f = 0; f < 4; ++f)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              acc0[f][r] -= p * (int)rintf((float)acc0[f][r] * inv);
              acc1[f][r] -= p * (int)rintf((float)acc1[f][r] * inv);
            }
        }
      }
#pragma unroll
      for (int f = 0; f < 4; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int u = acc0[f][r], v = acc1[f][r];
          const int x = split ? u + v : u, y = split ? u - v : v;
          // the word's bytes move down, the residue comes in on top
          rre[f][r][q4] = __builtin_amdgcn_perm((uint32_t)res_byte(x, p, inv), rre[f][r][q4], 0x04030201);
          rim[f][r][q4] = __builtin_amdgcn_perm((uint32_t)res_byte(y, p, inv), rim[f][r][q4], 0x04030201);
        }
    }
  }

  // reconstruction: wave c of a half takes its blocks 2 c and 2 c + 1 and gives the other two away
  const int g = lane >> 4;
  const v4i* wl = crt + (((lane & 15) >> 2) == g ? 0 : kCrt) + (lane & 3);
  // this wave's outputs: rows row0 + r of block c, columns col0 and col0 + 16; their scales (and C)
  // are fetched before the sums need them
  const int row0 = m0 + 32 * h + 16 * c + 4 * g, col0 = n0 + (lane & 15);
  const global_ptr<const int32_t> ea = (global_ptr<const int32_t>)pr.ea, eb = (global_ptr<const int32_t>)pr.eb;
  int sc[2][4];
#pragma unroll
  for (int f = 0; f < 2; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) sc[f][r] = ea[min(row0 + r, pr.Mp - 1)] + eb[col0 + 16 * f] + kResBits - scale_bits;
  __builtin_amdgcn_s_waitcnt(0x0070);   // the last loads are in LDS: it changes hands
  __syncthreads();
  v4i own[2][4][2];   // [block][register][part]
  {
    v4i* x = &lds[w * 16 * 64 + lane];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int part = 0; part < 2; ++part) {
          const uint32_t* lo = part == 0 ? rre[f][r] : rim[f][r];
          const uint32_t* up = part == 0 ? rre[2 + f][r] : rim[2 + f][r];
          v4i give;
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            own[f][r][part][q] = (int)(c ? up[q] : lo[q]);
            give[q] = (int)(c ? lo[q] : up[q]);
          }
          x[(f * 8 + 2 * r + part) * 64] = give;
        }
  }
  __syncthreads();
  const v4i* x = &lds[(w ^ 2) * 16 * 64 + lane];
#pragma unroll
  for (int f = 0; f < 2; ++f) {
    const int col = col0 + 16 * f;
    zdd old[4];
    if (beta) {
#pragma unroll
      for (int r = 0; r < 4; ++r)
        if (row0 + r < pr.M && col < pr.N) old[r] = load_zdd(pr.C + (int64_t)(row0 + r) * pr.ldc + col);
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      dd res[2];
#pragma unroll
      for (int part = 0; part < 2; ++part) {
        const v4i other = x[(f * 8 + 2 * r + part) * 64];
        const v4i* wp = wl + 2 * part * kResLimbs;
        v4i L[5];
#pragma unroll
        for (int q = 0; q < 5; ++q) {
          L[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wp[c * kResLimbs + 4 * q], own[f][r][part], zero, 0, 0, 0);
          L[q] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wp[(c ^ 1) * kResLimbs + 4 * q], other, L[q], 0, 0, 0);
        }
        res[part] = dd_mul(res_fraction(L), dd{kTab.P_hi, kTab.P_lo});
      }
      if (row0 + r < pr.M && col < pr.N) {
        const int e = sc[f][r];
        zdd o{dd{ldexp(res[0].hi, e), ldexp(res[0].lo, e)}, dd{ldexp(res[1].hi, e), ldexp(res[1].lo, e)}};
        if (negate) o = zdd_neg(o);
        if (beta) o = zdd_add(o, old[r]);
        store_zdd(pr.D + (int64_t)(row0 + r) * pr.ldd + col, o);
        if (pr.D64) {
          const double2 v = zdd_round(o);
          *(global_ptr<v2d>)(pr.D64 + (int64_t)(row0 + r) * pr.ldd64 + col) = v2d{v.x, v.y};
        }
      }
    }
  }
}

// ---------------------------------------------------------------------------------------------
// the allocation-free product: descriptors and maps of one problem written on the device

// jobs A, B at ws (an array of two), the product at ws + 256, maps at ws + 1024: split workgroups
// (ta of job 0, tb of job 1), product tiles (all 0)
__global__ __launch_bounds__(256) void k_oz_setup(char* ws, OzSplitJob ja, OzSplitJob jb, GemmProbOZ p, int ta, int tb,
                                                  int tiles) {
  if (threadIdx.x == 0) {
    *reinterpret_cast<OzSplitJob*>(ws) = ja;
    reinterpret_cast<OzSplitJob*>(ws)[1] = jb;
    *reinterpret_cast<GemmProbOZ*>(ws + 256) = p;
  }
  int32_t* m = reinterpret_cast<int32_t*>(ws + 1024);
  for (int i = threadIdx.x; i < ta + tb + tiles; i += 256) m[i] = i >= ta && i < ta + tb ? 1 : 0;
}

// Scratch of the allocation-free product: one array per device, allocated with the code object;
// host code uses the address obtained from hipGetSymbolAddress, never the array's name.
__device__ __align__(256) char scratch[kOzNoAllocScratch];

size_t pad256(size_t v) { return (v + 255) / 256 * 256; }

}  // namespace

// Device address of `scratch` on the current device (looked up once per device by the caller and
// kept); nullptr if the runtime cannot resolve it.
void* oz_noalloc_scratch_address() {
  void* ptr = nullptr;
  if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) {
    (void)hipGetLastError();
    return nullptr;
  }
  return ptr;
}

size_t oz_noalloc_bytes(int M, int N, int K) {
  const size_t Mp = (M + 31) / 32 * 32, Np = (N + 31) / 32 * 32, Kp = (K + 63) / 64 * 64;
  const size_t ba = (Mp + 63) / 64, bb = (Np + 63) / 64, ta = ba * (Kp / 32), tb = bb * (Kp / 32);
  const size_t tiles = (Mp / 32) * (Np / 32);
  return pad256(1024 + 4 * (ba + bb + ta + tb + tiles)) + pad256(48 * Mp * Kp) + pad256(48 * Np * Kp) +
         pad256(4 * Mp) + pad256(4 * Np);
}

int launch_oz_gemm_noalloc(hipStream_t st, char* ws, int opA, int opB, int M, int N, int K, int negate,
                           const void* A, int lda, const void* B, int ldb, int beta, const void* C, int ldc, void* D,
                           int ldd) {
  const int Mp = oz_rows(M), Np = oz_rows(N), Kp = (K + 63) / 64 * 64;
  const int kper = oz_split_steps((Mp + Np) / 16, Kp);
  const int ta = oz_split_blocks(Mp, Kp, kper), tb = oz_split_blocks(Np, Kp, kper);
  const int tiles = (Mp + 63) / 64 * (Np / 32);
  const size_t o_a8 = pad256(1024 + 4 * ((size_t)ta + tb + tiles));
  const size_t o_b8 = o_a8 + pad256((size_t)kOzPlanes * Mp * Kp);
  const size_t o_ea = o_b8 + pad256((size_t)kOzPlanes * Np * Kp);
  const size_t o_eb = o_ea + pad256(4 * (size_t)Mp);
  if (o_eb + 4 * (size_t)Np > kOzNoAllocScratch) return -1;   // beyond every product the caller accepts
  OzSplitJob ja{}, jb{};
  ja.X = (const zdd*)A; ja.R = M; ja.K = K; ja.Rp = Mp; ja.Kp = Kp;
  if (opA == 0) { ja.ldr = lda; ja.ldk = 1; } else { ja.ldr = 1; ja.ldk = lda; }
  ja.out = (int8_t*)(ws + o_a8); ja.ex = (int32_t*)(ws + o_ea);
  ja.tile_off = 0; ja.kper = kper;
  jb.X = (const zdd*)B; jb.R = N; jb.K = K; jb.Rp = Np; jb.Kp = Kp;
  if (opB == 0) { jb.ldr = 1; jb.ldk = ldb; } else { jb.ldr = ldb; jb.ldk = 1; }
  jb.out = (int8_t*)(ws + o_b8); jb.ex = (int32_t*)(ws + o_eb);
  jb.tile_off = ta; jb.kper = kper;
  GemmProbOZ p{};
  p.A8 = ja.out; p.B8 = jb.out; p.ea = ja.ex; p.eb = jb.ex;
  p.C = (const zdd*)C; p.D = (zdd*)D; p.D64 = nullptr;
  p.M = M; p.N = N; p.Mp = Mp; p.Np = Np; p.Kp = Kp; p.ldc = ldc; p.ldd = ldd; p.ldd64 = 0;
  p.tiles_n = Np / 32; p.tile_off = 0;
  hipLaunchKernelGGL(k_oz_setup, dim3(1), dim3(256), 0, st, ws, ja, jb, p, ta, tb, tiles);
  const int32_t* m = reinterpret_cast<const int32_t*>(ws + 1024);
  launch_oz_split(st, kOzSlices, reinterpret_cast<const OzSplitJob*>(ws), m, ta + tb);
  launch_oz_gemm(st, kOzSlices, reinterpret_cast<const GemmProbOZ*>(ws + 256), m + ta + tb, tiles, negate, beta);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

void launch_oz_split(hipStream_t st, int slices, const OzSplitJob* jobs, const int32_t* tile_job, int total_tiles) {
  if (total_tiles <= 0) return;
  hipLaunchKernelGGL(k_oz_split, dim3(total_tiles), dim3(256), 0, st, jobs, tile_job, 7 * slices - 1);
}

void launch_oz_gemm(hipStream_t st, int slices, const GemmProbOZ* probs, const int32_t* tile_prob, int total_tiles,
                    int negate, int beta) {
  if (total_tiles <= 0) return;
  hipLaunchKernelGGL(k_oz_gemm, dim3(((total_tiles + 7) / 8) * 8), dim3(256), 0, st, probs, tile_prob, total_tiles,
                     2 * (7 * slices - 1), negate, beta);
}

}  // namespace hsc
