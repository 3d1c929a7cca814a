// Moduli and tables of the residue products (ozaki.hip): exact integer matrix products of wide
// integers by the Chinese remainder theorem, one int8 product per residue plane (Ozaki, Uchino and
// Imamura, "Ozaki Scheme II", 2025).  Plain constexpr host code: the device tables are initialised
// from it at compile time and the CPU tests check it.
//
// 32 pairwise coprime moduli up to 256.  The first kResSplit have -1 as a square (every prime
// factor is 1 mod 4): with j^2 = -1 mod p the map a + ib -> (a + jb, a - jb) turns the complex
// product into two independent real ones, two planes and two products per modulus.  The others
// carry the residues of Re and Im and take four products on the same two planes.  The product P of
// all is 2^237.07: |Re|, |Im| of a product of depth K of operands with |Re| + |Im| <= 2^111 + 1 stay
// below K 2^222 (1 + 2^-109) < P / 2 for K <= 17152.
#pragma once

#include <cstdint>

namespace hsc {

constexpr int kResMods = 32;       // moduli
constexpr int kResSplit = 18;      // of which split the complex product
constexpr int kResPlanes = 64;     // residue planes of an operand, two per modulus
constexpr int kResLimbs = 20;      // base-256 digits of the reconstruction weights
constexpr int kResBits = 237;      // floor(log2 P)

constexpr int kResModuli[kResMods] = {
    // products of primes that are 1 mod 4
    241, 233, 229, 221, 205, 197, 193, 181, 173, 157, 149, 137, 113, 109, 101, 97, 89, 73,
    256, 243, 239, 227, 223, 217, 209, 199, 191, 179, 167, 163, 151, 139};

// M, the multiple of 256 p (of 256 for p = 256) nearest to 1.5 2^23, and the bits of the float M: an integer sum
// c started from them is, read as a float, M + c, without a conversion and with c's low byte, as long as
// |c| < 2^22 - 2^15 keeps it inside the float's binade (p = 256 takes the byte alone)
constexpr int kResBias = 12582912;
constexpr int res_bias(int p) { return p == 256 ? kResBias : (kResBias + 128 * p) / (256 * p) * (256 * p); }
constexpr int res_bias_bits(int p) { return 0x4b000000 + res_bias(p) - 8388608; }

struct alignas(16) ResTables {
  int32_t p[kResMods];
  float inv[kResMods];
  // residues from the four 28-bit chunks of an integer (chunk b of weight 2^(28 b) as four signed
  // bytes of weights 2^(8 k)): weight of byte 4 b + k, per plane and part; index 2 plane + part
  int8_t split[4][kResMods][16];
  // digit l (weight 2^(-8 (l + 1))) of a_m / p_m mod 1 with the residues of one part (Re, Im) as
  // coefficients; the 32 moduli as two groups of 16 bytes: byte b of group g belongs to modulus
  // 2 b + g
  int8_t crt[2][2][kResLimbs][16];
  double P_hi, P_lo;               // P / 2^kResBits as a double-double
};

constexpr int res_mod(long long a, int p) { return (int)(((a % p) + p) % p); }
constexpr int res_inverse(int a, int p) {
  for (int x = 1; x < p; ++x)
    if ((long long)a * x % p == 1) return x;
  return 0;
}
constexpr int res_root(int p) {   // j with j^2 = -1 mod p, or 0
  for (int x = 1; x < p; ++x)
    if ((x * x + 1) % p == 0) return x;
  return 0;
}
constexpr int res_centred(int r, int p) { return 2 * r >= p ? r - p : r; }

constexpr ResTables res_tables() {
  ResTables t{};
  for (int m = 0; m < kResMods; ++m) {
    const int p = kResModuli[m];
    t.p[m] = p;
    t.inv[m] = 1.0f / (float)p;
    const int j = m < kResSplit ? res_root(p) : 0;
    const int coef[4] = {1, m < kResSplit ? j : 0, m < kResSplit ? 1 : 0, m < kResSplit ? -j : 1};
    for (int b = 0; b < 4; ++b)
      for (int k = 0; k < 4; ++k) {
        int w = 1 % p;
        for (int e = 0; e < 28 * b + 8 * k; ++e) w = 2 * w % p;
        for (int q = 0; q < 4; ++q)
          t.split[q][m][4 * b + k] = (int8_t)res_centred(res_mod((long long)coef[q] * w, p), p);
      }
    int others = 1 % p;   // P / p_m mod p_m
    for (int i = 0; i < kResMods; ++i)
      if (i != m) others = others * (kResModuli[i] % p) % p;
    const int inv = res_inverse(others, p);
    for (int part = 0; part < 2; ++part) {
      // split: Re = (U + V) / 2 and Im = (U - V) / (2 j), from the residues of U + V and U - V
      int a = inv;
      if (m < kResSplit) a = (int)((long long)inv * res_inverse(part == 0 ? 2 : 2 * j % p, p) % p);
      int d[kResLimbs] = {};
      for (int l = 0, rem = a; l < kResLimbs; ++l) {
        d[l] = rem * 256 / p;
        rem = rem * 256 % p;
      }
      for (int l = kResLimbs - 1; l >= 0; --l)   // balanced digits; the carry out of the top is an integer
        if (d[l] > 127) {
          d[l] -= 256;
          if (l > 0) d[l - 1] += 1;
        }
      for (int l = 0; l < kResLimbs; ++l) t.crt[part][m & 1][l][m >> 1] = (int8_t)d[l];
    }
  }
  // P as 32-bit words, then its leading 106 bits
  uint32_t w[9] = {1};
  for (int m = 0; m < kResMods; ++m) {
    uint64_t carry = 0;
    for (int i = 0; i < 9; ++i) {
      carry += (uint64_t)w[i] * (uint32_t)kResModuli[m];
      w[i] = (uint32_t)carry;
      carry >>= 32;
    }
  }
  double hi = 0.0, lo = 0.0, scale = 1.0;   // bit kResBits has weight 1
  for (int b = kResBits; b >= 0; --b, scale *= 0.5) {
    const int bit = (w[b / 32] >> (b % 32)) & 1;
    if (kResBits - b < 53) hi += bit * scale;
    else if (kResBits - b < 106) lo += bit * scale;
  }
  const double s = hi + lo;
  t.P_hi = s;
  t.P_lo = lo - (s - hi);
  return t;
}

}  // namespace hsc
