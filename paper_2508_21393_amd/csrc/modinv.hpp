// Modular inverses (host and device) by division steps: Bernstein and Yang,
// "Fast constant-time gcd computation and modular inversion" (CHES 2019).
//
// For an odd modulus M and x prime to it, the divstep
//     (delta, f, g) -> (1 - delta, g, (g - f) / 2)           delta > 0, g odd
//                      (1 + delta, f, (g + (g mod 2) f) / 2)   otherwise
// starting from (1, M, x) reaches g = 0, f = +-1 after at most
// (49 b + 57) / 17 steps for b-bit inputs.  A batch of 30 steps depends only
// on delta and the low words of f and g, so it runs on 32-bit integers (one
// lane, about 22 instructions a step) and yields a 2 x 2 matrix t that is
// applied to the long f and g (exactly divided by 2^30) and to d, e with
// f = d x, g = e x mod M (divided by 2^30 mod M).  About 18 batches for Fr and
// 27 for Fq, against 383 field products of a Fermat power or about 800 long
// shifts and subtractions of a binary Euclid.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__) || defined(__HIP__)
#include <hip/hip_runtime.h>
#ifndef VL_HD
#define VL_HD __host__ __device__ __forceinline__
#endif
#else
#ifndef VL_HD
#define VL_HD inline
#endif
#endif

namespace vl {

// One batch of 30 divsteps on the low words: t = {u, v, q, r} with
// 2^30 (f', g') = (u f + v g, q f + r g).  c is all ones in a swapping step,
// odd in a step with odd g.
VL_HD void divsteps30(int32_t& delta, uint32_t f, uint32_t g, int32_t (&t)[4]) {
  uint32_t u = 1, v = 0, q = 0, r = 1;
  int32_t nd = -delta;
#pragma unroll 1
  for (int i = 0; i < 30; i += 5) {
#pragma unroll
    for (int k = 0; k < 5; ++k) {
      const uint32_t odd = 0u - (g & 1u);
      const uint32_t c = (uint32_t)(nd >> 31) & odd;     // delta > 0 and g odd
      const uint32_t c1 = c & 1u;
      const uint32_t sf = ((f ^ c) + c1) & odd;           // g odd: f, or -f in a swapping step
      const uint32_t su = ((u ^ c) + c1) & odd;
      const uint32_t sv = ((v ^ c) + c1) & odd;
      f = (g & c) | (f & ~c);
      u = (q & c) | (u & ~c);
      v = (r & c) | (v & ~c);
      g = (g + sf) >> 1;
      q += su;
      r += sv;
      u <<= 1;
      v <<= 1;
      nd = (int32_t)(((uint32_t)nd ^ c) + c1) - 1;
    }
  }
  delta = -nd;
  t[0] = (int32_t)u;
  t[1] = (int32_t)v;
  t[2] = (int32_t)q;
  t[3] = (int32_t)r;
}

// The multiple k of M that makes 2^30 divide u d + v e + k M and keeps the
// quotient short: first M towards zero for d and for e (by their signs neg_d,
// neg_e), which takes values in [-3 M / 2, 3 M / 2] into [-M, M], then a
// centred multiple in [-2^29, 2^29).  As |u| + |v| <= 2^30, the quotient is in
// [-3 M / 2, 3 M / 2] again; the multiple is below 3 2^29.  low: limb 0 of
// u d + v e.
template <typename Mod>
VL_HD int32_t modinv_multiple(int32_t u, int32_t v, bool neg_d, bool neg_e, uint32_t low) {
  const int32_t back = (neg_d ? u : -u) + (neg_e ? v : -v);   // at most 2^30
  low += (uint32_t)back * Mod::limb(0);
  return back + ((int32_t)((0u - low * Mod::inv30) << 2) >> 2);
}

// A batch's matrix applied to f, g (divided by 2^30, exactly for the batch's own
// matrix) and to d, e (divided by 2^30 mod M)
template <typename Mod>
VL_HD void modinv_apply(const int32_t (&t)[4], int32_t (&f)[Mod::L], int32_t (&g)[Mod::L], int32_t (&d)[Mod::L],
                        int32_t (&e)[Mod::L]) {
  constexpr int L = Mod::L;
  constexpr int32_t kM = 0x3fffffff;
  const int64_t u = t[0], v = t[1], q = t[2], r = t[3];
  int64_t cf = u * f[0] + v * g[0], cg = q * f[0] + r * g[0];
  int64_t cd = u * d[0] + v * e[0], ce = q * d[0] + r * e[0];
  const bool nd = d[L - 1] < 0, ne = e[L - 1] < 0;
  const int64_t kd = modinv_multiple<Mod>(t[0], t[1], nd, ne, (uint32_t)cd);
  const int64_t ke = modinv_multiple<Mod>(t[2], t[3], nd, ne, (uint32_t)ce);
  cd += kd * (int32_t)Mod::limb(0);
  ce += ke * (int32_t)Mod::limb(0);
  cf >>= 30;
  cg >>= 30;
  cd >>= 30;
  ce >>= 30;
#pragma unroll
  for (int i = 1; i < L; ++i) {   // below 5 2^59 + a carry: at most 2^60 of each pair of products, 3 2^59 of k m
    const int64_t m = (int32_t)Mod::limb(i);
    cf += u * f[i] + v * g[i];
    cg += q * f[i] + r * g[i];
    cd += u * d[i] + v * e[i] + kd * m;
    ce += q * d[i] + r * e[i] + ke * m;
    f[i - 1] = (int32_t)cf & kM;
    g[i - 1] = (int32_t)cg & kM;
    d[i - 1] = (int32_t)cd & kM;
    e[i - 1] = (int32_t)ce & kM;
    cf >>= 30;
    cg >>= 30;
    cd >>= 30;
    ce >>= 30;
  }
  f[L - 1] = (int32_t)cf;
  g[L - 1] = (int32_t)cg;
  d[L - 1] = (int32_t)cd;
  e[L - 1] = (int32_t)ce;
}

// Mod: L 30-bit limbs, limb(i), inv30 = M^-1 mod 2^30, kBatches (the bound
// above).  x: limbs of a value in (0, 2 M) prime to M.  Returns d = x^-1 mod M
// in [-3 M / 2, 3 M / 2] as 30-bit limbs with a signed top limb.  x = 0 gives 0.
template <typename Mod>
VL_HD void modinv30(const int32_t (&x)[Mod::L], int32_t (&out)[Mod::L]) {
  constexpr int L = Mod::L;
  constexpr int32_t kM = 0x3fffffff;
  int32_t f[L], g[L], d[L], e[L];
#pragma unroll
  for (int i = 0; i < L; ++i) {
    f[i] = (int32_t)Mod::limb(i);
    g[i] = x[i];
    d[i] = 0;
    e[i] = i == 0 ? 1 : 0;
  }
  int32_t delta = 1;
#pragma unroll 1
  for (int batch = 0; batch < Mod::kBatches; ++batch) {
    int32_t nz = 0;
#pragma unroll
    for (int i = 0; i < L; ++i) nz |= g[i];
    if (nz == 0) break;
    int32_t t[4];
    // 32-bit low words: limb 0 and the low bits of limb 1
    divsteps30(delta, (uint32_t)f[0] | ((uint32_t)f[1] << 30), (uint32_t)g[0] | ((uint32_t)g[1] << 30), t);
    modinv_apply<Mod>(t, f, g, d, e);
  }
  // f = +-1: the inverse is d or -d
  const bool neg = f[L - 1] < 0;
  int32_t carry = 0;
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int32_t s = (neg ? -d[i] : d[i]) + carry;
    out[i] = i < L - 1 ? s & kM : s;
    carry = s >> 30;
  }
}

// W 32-bit words to 30-bit limbs, and a non-negative value back
template <int W, int L>
VL_HD void words_to_30(const uint32_t (&w)[W], int32_t (&l)[L]) {
#pragma unroll
  for (int i = 0; i < L; ++i) {
    const int bit = 30 * i, k = bit >> 5, sh = bit & 31;
    uint64_t v = k < W ? w[k] : 0u;
    if (k + 1 < W) v |= (uint64_t)w[k + 1] << 32;
    l[i] = (int32_t)((uint32_t)(v >> sh) & 0x3fffffffu);
  }
}
template <int W, int L>
VL_HD void limbs30_to_words(const int32_t (&l)[L], uint32_t (&w)[W]) {
#pragma unroll
  for (int k = 0; k < W; ++k) {
    const int bit = 32 * k, i = bit / 30, sh = bit - 30 * i;
    uint64_t v = (uint64_t)(uint32_t)l[i] >> sh;
    if (i + 1 < L) v |= (uint64_t)(uint32_t)l[i + 1] << (30 - sh);
    if (i + 2 < L) v |= (uint64_t)(uint32_t)l[i + 2] << (60 - sh);
    w[k] = (uint32_t)v;
  }
}

// x + 2 M with carries passed on: brings an inverse into [M / 2, 7 M / 2]
template <typename Mod>
VL_HD void add_2m30(int32_t (&x)[Mod::L]) {
  uint32_t carry = 0;
#pragma unroll
  for (int i = 0; i < Mod::L; ++i) {
    const uint32_t s = (uint32_t)x[i] + 2u * Mod::limb(i) + carry;   // below 2^32 below the top limb
    x[i] = (int32_t)(i < Mod::L - 1 ? s & 0x3fffffffu : s);
    carry = s >> 30;
  }
}

}  // namespace vl
