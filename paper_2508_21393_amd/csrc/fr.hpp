// Arithmetic in Fr, the BLS12-381 scalar field (host and device).
//
// The paper only asks for a field of about 2^254 elements "such as" the
// BLS12-381 one (Sec. V); this library fixes that field.
//   p = 0x73eda753299d7d483339d80809a1d80553bda402fffe5bfeffffffff00000001
// Elements are 8 little-endian 32-bit limbs.  Inside the library they are kept
// in Montgomery form x*R mod p with R = 2^256; on the wire (proof bytes, host
// API) they are canonical.  Multiplication is Montgomery multiplication (Koc,
// Acar, Kaliski, IEEE Micro 1996): on the device on 29-bit limbs in 64-bit
// columns, on the host CIOS on 64-bit limbs.
#pragma once
#include <stdint.h>

#if defined(__HIPCC__) || defined(__HIP__)
#include <hip/hip_runtime.h>
#define VL_HD __host__ __device__ __forceinline__
#else
#define VL_HD inline
#endif

namespace vl {

struct Fr {
  uint32_t w[8];
};

// p, R mod p and R^2 mod p as limbs.
#define VL_P_LIMBS 0x00000001u, 0xffffffffu, 0xfffe5bfeu, 0x53bda402u, \
                   0x09a1d805u, 0x3339d808u, 0x299d7d48u, 0x73eda753u
#define VL_R_LIMBS 0xfffffffeu, 0x00000001u, 0x00034802u, 0x5884b7fau, \
                   0xecbc4ff5u, 0x998c4fefu, 0xacc5056fu, 0x1824b159u
#define VL_R2_LIMBS 0xf3f29c6du, 0xc999e990u, 0x87925c23u, 0x2b6cedcbu, \
                    0x7254398fu, 0x05d31496u, 0x9f59ff11u, 0x0748d9d9u
VL_HD uint32_t p_limb(int i) {
  // switch keeps the constant in the instruction stream on the device
  switch (i) {
    case 0: return 0x00000001u; case 1: return 0xffffffffu;
    case 2: return 0xfffe5bfeu; case 3: return 0x53bda402u;
    case 4: return 0x09a1d805u; case 5: return 0x3339d808u;
    case 6: return 0x299d7d48u; default: return 0x73eda753u;
  }
}

VL_HD Fr fr_zero() { Fr r; for (int i = 0; i < 8; ++i) r.w[i] = 0; return r; }
VL_HD Fr fr_from_limbs(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t a4,
                       uint32_t a5, uint32_t a6, uint32_t a7) {
  Fr r; r.w[0] = a0; r.w[1] = a1; r.w[2] = a2; r.w[3] = a3;
  r.w[4] = a4; r.w[5] = a5; r.w[6] = a6; r.w[7] = a7; return r;
}
VL_HD Fr fr_R() { return fr_from_limbs(VL_R_LIMBS); }     // Montgomery form of 1
VL_HD Fr fr_R2() { return fr_from_limbs(VL_R2_LIMBS); }
VL_HD Fr fr_one_raw() { return fr_from_limbs(1, 0, 0, 0, 0, 0, 0, 0); }

VL_HD bool fr_eq(const Fr& a, const Fr& b) {
  uint32_t d = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) d |= a.w[i] ^ b.w[i];
  return d == 0;
}

VL_HD bool fr_is_zero(const Fr& a) {
  uint32_t d = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) d |= a.w[i];
  return d == 0;
}

// 32-bit add/subtract with carry in and out (one v_add_co/v_addc_co or
// v_sub_co/v_subb_co on the device with clang's builtins)
VL_HD uint32_t adc32(uint32_t a, uint32_t b, uint32_t cin, uint32_t& cout) {
#if defined(__clang__)
  unsigned c;
  const uint32_t r = __builtin_addc(a, b, cin, &c);
  cout = c;
  return r;
#else
  const uint64_t t = (uint64_t)a + b + cin;
  cout = (uint32_t)(t >> 32);
  return (uint32_t)t;
#endif
}
VL_HD uint32_t sbb32(uint32_t a, uint32_t b, uint32_t bin, uint32_t& bout) {
#if defined(__clang__)
  unsigned c;
  const uint32_t r = __builtin_subc(a, b, bin, &c);
  bout = c;
  return r;
#else
  const uint64_t t = (uint64_t)a - b - bin;
  bout = (uint32_t)(t >> 63);
  return (uint32_t)t;
#endif
}

// a < p ?
VL_HD bool fr_lt_p(const Fr& a) {
  uint32_t borrow = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) (void)sbb32(a.w[i], p_limb(i), borrow, borrow);
  return borrow != 0;
}

// r = a - p if a >= p else a   (a < 2p)
VL_HD Fr fr_reduce_once(const Fr& a) {
  Fr t;
  uint32_t borrow = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) t.w[i] = sbb32(a.w[i], p_limb(i), borrow, borrow);
  Fr r;
#pragma unroll
  for (int i = 0; i < 8; ++i) r.w[i] = borrow ? a.w[i] : t.w[i];
  return r;
}

VL_HD Fr fr_add(const Fr& a, const Fr& b) {
  Fr s;
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) s.w[i] = adc32(a.w[i], b.w[i], c, c);
  return fr_reduce_once(s);   // a + b < 2p < 2^256: no carry out
}

VL_HD Fr fr_sub(const Fr& a, const Fr& b) {
  Fr d;
  uint32_t borrow = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) d.w[i] = sbb32(a.w[i], b.w[i], borrow, borrow);
  // if it went negative add p back
  const uint32_t mask = 0u - borrow;
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < 8; ++i) d.w[i] = adc32(d.w[i], p_limb(i) & mask, c, c);
  return d;
}

VL_HD Fr fr_neg(const Fr& a) { return fr_sub(fr_zero(), a); }
VL_HD Fr fr_double(const Fr& a) { return fr_add(a, a); }

// a / 2: a (even) or a + p (odd) shifted right by one; a + p < 2^256
VL_HD Fr fr_half(const Fr& a) {
  const uint32_t mask = 0u - (a.w[0] & 1u);
  Fr t;
  uint32_t c = 0;
#pragma unroll
  for (int j = 0; j < 8; ++j) t.w[j] = adc32(a.w[j], p_limb(j) & mask, c, c);
  Fr r;
#pragma unroll
  for (int j = 0; j < 7; ++j) r.w[j] = (t.w[j] >> 1) | (t.w[j + 1] << 31);
  r.w[7] = t.w[7] >> 1;
  return r;
}

#if defined(__HIP_DEVICE_COMPILE__)
// Device Montgomery product on 9 limbs of 29 bits.  A product of two limbs is
// below 2^58, so a column of the schoolbook product and of the reduction (at
// most 17 such terms) stays below 2^63: every multiply-add is one
// v_mad_u64_u32 into a 64-bit column with no carry to pass on, the 17 columns
// are independent, and the kernel is plain C++ that the compiler schedules
// (an inline-asm multiply-add with its carry took two instructions, and the
// compiler puts an s_nop between an asm and a dependent one).
// The limbs of a are taken from 32 a (260 bits), so that the reduction by
// 2^261 = 2^(9 * 29) yields a b / 2^256.  As p = 1 mod 2^29 the quotient digit
// of a column is m = -c mod 2^29, and c + m carries ceil(c / 2^29) on.
// 1 wave: 2224 -> 1260 cycles per product (interleaved pairs 1580 -> 1220);
// whole GPU: 117 -> 133 G products/s (pairs 126 -> 140).
constexpr uint32_t kM29 = 0x1fffffffu;
__device__ __forceinline__ constexpr uint32_t p_limb29(int j) {
  constexpr uint32_t P[8] = {VL_P_LIMBS};
  const int bit = 29 * j, w = bit >> 5, sh = bit & 31;
  uint64_t v = P[w];
  if (w + 1 < 8) v |= (uint64_t)P[w + 1] << 32;
  return (uint32_t)(v >> sh) & kM29;
}

// the 29-bit limbs of a << UP (UP = 0 or 5: at most 261 bits)
template <int UP>
__device__ __forceinline__ void fr_split29(const Fr& a, uint32_t (&l)[9]) {
#pragma unroll
  for (int j = 0; j < 9; ++j) {
    const int bit = 29 * j - UP;
    uint32_t v;
    if (bit < 0) {
      v = a.w[0] << -bit;
    } else {
      const int w = bit >> 5, sh = bit & 31;
      v = w == 7 ? a.w[7] >> sh : (sh ? __builtin_amdgcn_alignbit(a.w[w + 1], a.w[w], sh) : a.w[w]);
    }
    l[j] = j < 8 ? v & kM29 : v;
  }
}

// columns c (c[17] = 0) to c / 2^261 mod p: below 2p if c < 2^261 p
__device__ __forceinline__ Fr fr_redc29(uint64_t (&c)[18]) {
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const uint32_t m = (0u - (uint32_t)c[k]) & kM29;
    c[k + 1] += (c[k] + kM29) >> 29;
#pragma unroll
    for (int j = 1; j < 9; ++j) c[k + j] += (uint64_t)m * p_limb29(j);
  }
  uint32_t z[9];
  uint64_t t = c[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    z[k] = (uint32_t)t & kM29;
    t = (t >> 29) + (k < 8 ? c[10 + k] : 0);
  }
  Fr r;
#pragma unroll
  for (int w = 0; w < 8; ++w) {
    const int bit = 32 * w, j = bit / 29, sh = bit - 29 * j;
    uint32_t v = (z[j] >> sh) | (z[j + 1] << (29 - sh));
    if (58 - sh < 32 && j + 2 < 9) v |= z[j + 2] << (58 - sh);
    r.w[w] = v;
  }
  return fr_reduce_once(r);
}
#endif

#if !defined(__HIP_DEVICE_COMPILE__)
// Host Montgomery product with 64-bit limbs (CIOS, 128-bit partial
// products): 32 multiplications instead of the 128 of 32-bit limbs.  R is
// 2^256 either way, so the result is the same field element.
inline Fr fr_mul_host64(const Fr& a, const Fr& b) {
  typedef unsigned __int128 u128;
  constexpr uint64_t P[4] = {0xffffffff00000001ull, 0x53bda402fffe5bfeull, 0x3339d80809a1d805ull,
                             0x73eda753299d7d48ull};
  constexpr uint64_t kPInv64 = 0xfffffffeffffffffull;   // -p^-1 mod 2^64
  uint64_t A[4], Bv[4], t[6] = {0, 0, 0, 0, 0, 0};
  for (int j = 0; j < 4; ++j) {
    A[j] = (uint64_t)a.w[2 * j] | ((uint64_t)a.w[2 * j + 1] << 32);
    Bv[j] = (uint64_t)b.w[2 * j] | ((uint64_t)b.w[2 * j + 1] << 32);
  }
  for (int i = 0; i < 4; ++i) {
    u128 C = 0;
    for (int j = 0; j < 4; ++j) {
      C = (u128)A[j] * Bv[i] + t[j] + (uint64_t)(C >> 64);
      t[j] = (uint64_t)C;
    }
    u128 s = (u128)t[4] + (uint64_t)(C >> 64);
    t[4] = (uint64_t)s;
    t[5] = (uint64_t)(s >> 64);
    const uint64_t m = t[0] * kPInv64;
    C = (u128)m * P[0] + t[0];
    for (int j = 1; j < 4; ++j) {
      C = (u128)m * P[j] + t[j] + (uint64_t)(C >> 64);
      t[j - 1] = (uint64_t)C;
    }
    s = (u128)t[4] + (uint64_t)(C >> 64);
    t[3] = (uint64_t)s;
    t[4] = t[5] + (uint64_t)(s >> 64);
  }
  Fr r;
  for (int j = 0; j < 4; ++j) {
    r.w[2 * j] = (uint32_t)t[j];
    r.w[2 * j + 1] = (uint32_t)(t[j] >> 32);
  }
  return fr_reduce_once(r);
}
#endif

// Montgomery product a*b*R^-1 mod p (inputs < p, output < p).  The device
// build uses the 29-bit form above; the host build the 64-bit CIOS form.
VL_HD Fr fr_mul(const Fr& a, const Fr& b) {
#if defined(__HIP_DEVICE_COMPILE__)
  uint32_t x[9], y[9];
  fr_split29<5>(a, x);
  fr_split29<0>(b, y);
  uint64_t c[18];
#pragma unroll
  for (int k = 0; k < 18; ++k) c[k] = 0;
#pragma unroll
  for (int i = 0; i < 9; ++i)
#pragma unroll
    for (int j = 0; j < 9; ++j) c[i + j] += (uint64_t)x[i] * y[j];
  return fr_redc29(c);
#else
  return fr_mul_host64(a, b);
#endif
}

VL_HD Fr fr_to_mont(const Fr& a) { return fr_mul(a, fr_R2()); }
VL_HD Fr fr_from_mont(const Fr& a) { return fr_mul(a, fr_one_raw()); }

// limb sums t_i (i < 10, weight 2^(26 i), signed, total in [0, 2^272)) mod p
VL_HD Fr fr_of_limb_sums(const uint64_t (&t)[10]) {
  uint32_t l[11];
  int64_t c = 0;
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    c += (int64_t)t[i];
    l[i] = (uint32_t)c & 0x3ffffffu;
    c >>= 26;
  }
  l[10] = (uint32_t)c;
  uint32_t w[9];
#pragma unroll
  for (int k = 0; k < 9; ++k) {
    const int bit = 32 * k, i = bit / 26, sh = bit - 26 * i;
    uint32_t v = l[i] >> sh;
    if (i + 1 < 11) v |= l[i + 1] << (26 - sh);
    if (i + 2 < 11 && 52 - sh < 32) v |= l[i + 2] << (52 - sh);
    w[k] = v;
  }
  // T = floor(total / 2^240) below 2^32 times floor(2^286 / p), over 2^46:
  // total / p less T 2^240 / p is below 2^240 / p < 2^-14, and the rounded
  // constant takes at most T / 2^46 < 2^-14 more, so the quotient is exact or
  // one too small
  const uint32_t q = (uint32_t)(((uint64_t)((w[8] << 16) | (w[7] >> 16)) * 2371102011u) >> 46);
  Fr r;
  uint64_t m = 0;
  uint32_t borrow = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    m += (uint64_t)q * p_limb(k);
    r.w[k] = sbb32(w[k], (uint32_t)m, borrow, borrow);
    m >>= 32;
  }
  return fr_reduce_once(r);
}

// canonical little-endian 32-byte encoding
VL_HD void fr_to_bytes(const Fr& a, uint8_t* out) {
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    out[4 * i + 0] = (uint8_t)(a.w[i]);
    out[4 * i + 1] = (uint8_t)(a.w[i] >> 8);
    out[4 * i + 2] = (uint8_t)(a.w[i] >> 16);
    out[4 * i + 3] = (uint8_t)(a.w[i] >> 24);
  }
}

VL_HD Fr fr_from_bytes(const uint8_t* in) {
  Fr a;
#pragma unroll
  for (int i = 0; i < 8; ++i)
    a.w[i] = (uint32_t)in[4 * i] | ((uint32_t)in[4 * i + 1] << 8) |
             ((uint32_t)in[4 * i + 2] << 16) | ((uint32_t)in[4 * i + 3] << 24);
  return a;
}

}  // namespace vl
