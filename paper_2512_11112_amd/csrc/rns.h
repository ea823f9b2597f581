// Residue number system of the int8 matrix engine over p = 2^61 - 1.
//
// A residue x mod p is taken balanced (|x| < 2^60) and written as its residues
// modulo T pairwise coprime numbers of at most 8 bits, each a signed byte.  A
// matrix product then is T independent int8 products, exact in int32, whose
// entries mod m_t determine the integer sum S of K' products as long as
// 2 |S| < M = prod m_t; |S| < K' 2^120.  The Chinese remainder theorem gives S
// mod p without forming S: with u_t = S (M / m_t)^-1 mod m_t,
//   S = sum_t u_t (M / m_t) - q M,   q = round(sum_t u_t / m_t),
// so S mod p is a short sum of bytes times constants mod p.  The factors
// (M / m_t)^-1 are multiplied into the left operand's residues.
//
// Products of two 61-bit residues summed over K' carry 120 + log2 K' + 1 bits,
// which needs 17 or 18 such moduli; eight base-256 digits a side would take 64
// byte products.  The moduli are the coprime set of this size whose product is
// largest among 256 and the primes and products of two primes below it.
#pragma once
#include "field.h"

namespace spdz {
namespace rns {

constexpr int TMAX = 18;
constexpr int MODS[TMAX] = {256, 253, 251, 249, 247, 241, 239, 235, 233, 229, 227, 223, 217, 211, 199, 197, 193, 191};
// M of the first 17 is 2^133.22: sums of up to 4287 products stay below 0.45 M (the rounding of q
// tolerates an error of 0.05, its own is below 3e-4); all 18 give 2^140.79
constexpr int64_t T17_TERMS = 4287;
constexpr int64_t MAX_TERMS = 16382;
static_assert(MAX_TERMS * 128 * 128 < (int64_t)1 << 28, "sums of bytes for round_mod28 (within 0.02 % of it)");
// whether sums of `terms` products, each at most 2^120, stay below 0.45 M of the first T moduli
constexpr bool covered(int T, int64_t terms) {
  double m = 1;
  for (int t = 0; t < T; t++) m *= MODS[t];
  return (double)terms * 0x1p120 < 0.45 * m;
}
static_assert(covered(17, T17_TERMS) && !covered(17, T17_TERMS + 1) && covered(18, MAX_TERMS), "moduli");
constexpr int FRAC = 23;  // u_t / m_t is summed in units of 2^-23

constexpr u64 P = (1ull << 61) - 1;
constexpr u64 mulp(u64 a, u64 b) { return (u64)((u128)a * b % P); }

// Residue of a balanced value mod m_t: the dot product of its signed base-256 digits with the powers of 256
// mod m_t, balanced (c0 low digits, c1 high), and what round_mod takes.  One record, one scalar load.
struct alignas(32) Digits {
  int c0, c1;
  int bias;  // bits of the float 2^23 + b with b = 2^18 to 2^18 + 255 and m_t | 2^23 + b: an integer
             // |s| < 2^18 added to them is the float 2^23 + b + s
  int neg;   // -m_t
  float inv;
};

// constants of one choice of T (17 or 18)
struct Tables {
  Digits digits[2][TMAX + 1];  // [left][t] (left: the powers times (M / m_t)^-1); one more is read ahead
  float inv[TMAX];     // 1 / m_t
  int neg[TMAX];       // -m_t
  int c14[TMAX];       // 2^14 mod m_t, balanced
  // bits of the float 2^23 + b, b a multiple of 2^14 from 130 2^14 on, m_t | 2^23 + b: as Digits::bias for |s| < 2^21
  u32 bias14[TMAX];
  // (M / m_t) mod p: byte j of the weights of moduli 4 g .. 4 g + 3, packed
  u32 w[5][8];
  u32 f[5][2];         // bytes of round(2^FRAC / m_t), packed alike
  u64 wsum;            // -128 sum_t weight_t - 16 M mod p
  u64 mp;              // M mod p
  u32 fsum;            // 128 sum_t round(2^FRAC / m_t)
};

constexpr Tables make_tables(int T) {
  Tables r{};
  u64 mp = 1, ws = 0;
  u32 fs = 0;
  for (int t = 0; t < T; t++) mp = mulp(mp, (u64)MODS[t]);
  for (int t = 0; t < T; t++) {
    const int m = MODS[t];
    u64 w = 1;
    int rest = 1;  // M / m_t mod m_t
    for (int s = 0; s < T; s++)
      if (s != t) {
        w = mulp(w, (u64)MODS[s]);
        rest = rest * (MODS[s] % m) % m;
      }
    int inverse = 1;
    while (rest * inverse % m != 1) inverse++;
    for (int left = 0; left < 2; left++) {
      const int k = left ? inverse : 1;
      int pw = 1;  // 256^j mod m
      u32 c[2] = {0, 0};
      for (int j = 0; j < 8; j++) {
        const int v = pw * k % m;
        const u32 byte = (u32)(v > 127 ? v - m : v) & 255;  // m even only for 256: 128 stays -128
        if (j < 4) c[0] |= byte << (8 * j);
        else c[1] |= byte << (8 * (j - 4));
        pw = pw * 256 % m;
      }
      r.digits[left][t].c0 = (int)c[0];
      r.digits[left][t].c1 = (int)c[1];
    }
    r.inv[t] = 1.0f / (float)m;
    r.neg[t] = -m;
    const int c14 = 16384 % m;
    r.c14[t] = c14 > m / 2 ? c14 - m : c14;
    u32 b = 1u << 18, b14 = 130u << 14;
    while (((1u << 23) + b) % (u32)m != 0) b++;
    while (((1u << 23) + b14) % (u32)m != 0) b14 += 1u << 14;
    for (int left = 0; left < 2; left++) {
      Digits &d = r.digits[left][t];
      d.bias = (int)(0x4B000000u + b);
      d.neg = r.neg[t];
      d.inv = r.inv[t];
    }
    r.bias14[t] = 0x4B000000u + b14;
    const u32 f = (u32)(((2u << FRAC) / (u32)m + 1) / 2);
    for (int j = 0; j < 8; j++) r.w[t / 4][j] |= (u32)((w >> (8 * j)) & 255) << (8 * (t % 4));
    for (int j = 0; j < 2; j++) r.f[t / 4][j] |= ((f >> (8 * j)) & 255) << (8 * (t % 4));
    ws = (ws + w) % P;
    fs += f;
  }
  r.mp = mp;
  r.wsum = (P - (mulp(128, ws) + mulp(16, mp)) % P) % P;
  r.fsum = 128 * fs;
  return r;
}

constexpr Tables TAB17 = make_tables(17), TAB18 = make_tables(18);

// round_mod28's argument, |s >> 14| <= 2^14 times c14 and 14 more bits over the bias, stays the bits of a float
// 2^23 + v with 0 < v < 2^23
constexpr bool bias14_holds() {
  for (int t = 0; t < TMAX; t++) {
    const int64_t b = (int64_t)TAB18.bias14[t] - 0x4B000000, c = TAB18.c14[t] < 0 ? -TAB18.c14[t] : TAB18.c14[t];
    if (b % 16384 != 0 || b <= c * 16384 || b + c * 16384 + 16383 >= 1 << 23) return false;
  }
  return true;
}
static_assert(bias14_holds(), "round_mod28");
template <int T>
constexpr const Tables &tab() {
  if constexpr (T == 17) return TAB17;
  else return TAB18;
}

// signed base-256 digits (|value| < 2^60) of the balanced value of a canonical word, packed
__device__ __forceinline__ u64 digits(u64 w) {
  const u64 y = w - ((w >> 60) ? P : 0);
  return (y + 0x0080808080808080ull) ^ 0x0080808080808080ull;
}

// Low byte of r = s - m round(s / m) for the integer s in fb = bias + s, the bits of the float
// n m + s: its product with 1 / m plus 1.5 2^23 leaves n + round(s / m) in the low mantissa bits, the
// 24-bit product takes them as they are, and the 2^22 m that the constant contributes is 0 mod 256.
// The rounded inverse moves the quotient by less than 0.006: |r| <= 127 for the odd moduli; modulo 256 the
// inverse is exact and a tie may be 128 or -128, which are one byte, -128.
__device__ __forceinline__ int round_mod(u32 fb, float inv, int neg) {
  float x;
  __builtin_memcpy(&x, &fb, 4);
  const float q = __builtin_fmaf(x, inv, 12582912.0f);
  int qb;
  __builtin_memcpy(&qb, &q, 4);
  return __mul24(qb, neg) + (int)fb;
}
// the same for a sum |s| < 2^28
__device__ __forceinline__ int round_mod28(int s, float inv, int neg, int c14, u32 bias14) {
  return round_mod((u32)__mul24(s >> 14, c14) + (((u32)s & 16383u) | bias14), inv, neg);
}

}  // namespace rns
}  // namespace spdz
