// Device helpers of the sumcheck kernels (kernels.hip, bmm.hip, lookup.hip): wave
// and workgroup sums of field elements, proof-byte stores, LDS element access,
// the transcript's hashing.
#pragma once
#include "device.hpp"
#include "sha256.hpp"

namespace vl {

// sum of K field elements over the lanes of a wave (xor butterfly over
// lane distances < width, a power of two <= 64: every lane of each aligned
// group of `width` lanes ends with that group's sum)
template <int K>
__device__ __forceinline__ void wave_sum(Fr (&v)[K], uint32_t width) {
  for (uint32_t off = width >> 1; off >= 1; off >>= 1) {
#pragma unroll
    for (int k = 0; k < K; ++k) {
      Fr o;
#pragma unroll
      for (int j = 0; j < 8; ++j) o.w[j] = __shfl_xor(v[k].w[j], (int)off, kWave);
      v[k] = fr_add(v[k], o);
    }
  }
}

// Sums of K elements per thread over a workgroup of NW waves, for K values
// that end up in lanes 0 .. K - 1 of wave 0 (lane k: the sum of value k,
// reduced; other lanes hold nothing of use).  Every element is cut into ten
// 26-bit limbs, whose sums over 64 lanes stay below 2^32, so a wave adds them
// with one DPP add per limb and level and no carries (wave_sum takes 8 lane
// shuffles and a field addition per element and level: 4100 cycles for three
// values on one wave, this about 900); lane k of wave 0 then adds the waves'
// limbs, carries once and reduces once.  lds: K * 10 * NW words.
//
// ten sums side by side (a DPP operand needs two instructions between its
// write and its read: the other limbs')
#define VL_DPP_LEVEL(ctrl, rows, bc)                                                                        \
  _Pragma("unroll") for (int i = 0; i < 10; ++i)                                                            \
      x[i] += (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x[i], ctrl, rows, 0xf, bc);
__device__ __forceinline__ void row_add10(uint32_t (&x)[10]) {   // a row's sums, in its lane 15
  VL_DPP_LEVEL(0x111, 0xf, true)    // row_shr:1, 2, 4, 8
  VL_DPP_LEVEL(0x112, 0xf, true)
  VL_DPP_LEVEL(0x114, 0xf, true)
  VL_DPP_LEVEL(0x118, 0xf, true)
}
__device__ __forceinline__ void wave_add10(uint32_t (&x)[10]) {   // the wave's sums, in lane 63
  row_add10(x);
  VL_DPP_LEVEL(0x142, 0xa, false)   // row_bcast:15, row_bcast:31
  VL_DPP_LEVEL(0x143, 0xc, false)
}
#undef VL_DPP_LEVEL
// Value sums of a workgroup whose rows of 16 lanes each hold one value: acc
// holds ten 64-bit limb sums per value (zeroed and read between barriers).
// acc_add adds the row's 16 elements to value k (the same in the row's lanes)
// if the row takes part.
__device__ __forceinline__ void acc_add(unsigned long long* acc, uint32_t k, const Fr& v, bool take = true) {
  uint32_t x[10];
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    const int bit = 26 * i, j = bit >> 5, sh = bit & 31;
    x[i] = (sh == 0 ? v.w[j] : (j < 7 ? __builtin_amdgcn_alignbit(v.w[j + 1], v.w[j], sh) : v.w[7] >> sh)) & 0x3ffffffu;
  }
  row_add10(x);
  if (take && (threadIdx.x & 15u) == 15u)
#pragma unroll
    for (int i = 0; i < 10; ++i) atomicAdd(acc + 10 * k + i, (unsigned long long)x[i]);
}
// The value at X = k (0 .. 3, per lane) of the quadratic with sums[base],
// [base + 1] its values at 0 and 1 and [base + 2] its leading coefficient:
// q(2) = 2 q1 - q0 + 2 q2, q(3) = 3 q1 - 2 q0 + 6 q2, formed on the limb sums
// (up to 2^13 elements each; 2^14 p keeps the total positive).
__device__ __forceinline__ Fr acc_point(const unsigned long long* acc, uint32_t base, uint32_t k) {
  const int64_t c0 = k == 0 ? 1 : (k == 1 ? 0 : (k == 2 ? -1 : -2));
  const int64_t c1 = k == 0 ? 0 : (k == 1 ? 1 : (k == 2 ? 2 : 3));
  const int64_t c2 = k < 2 ? 0 : (k == 2 ? 2 : 6);
  uint64_t t[10];
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    constexpr uint32_t P[9] = {VL_P_LIMBS, 0u};
    const int bit = 26 * i, j = bit >> 5, sh = bit & 31;
    const uint64_t pl = ((((uint64_t)P[j + 1 < 9 ? j + 1 : 8] << 32) | P[j]) >> sh) & 0x3ffffffu;
    t[i] = (uint64_t)(c0 * (int64_t)acc[10 * base + i] + c1 * (int64_t)acc[10 * base + 10 + i] +
                      c2 * (int64_t)acc[10 * base + 20 + i]) + (pl << 14);
  }
  return fr_of_limb_sums(t);
}
// the same for a line with sums[base], [base + 1] its values at 0 and 1, at X =
// k <= 2
__device__ __forceinline__ Fr acc_line(const unsigned long long* acc, uint32_t base, uint32_t k) {
  const int64_t c0 = 1 - (int64_t)k, c1 = (int64_t)k;
  uint64_t t[10];
#pragma unroll
  for (int i = 0; i < 10; ++i) {
    constexpr uint32_t P[9] = {VL_P_LIMBS, 0u};
    const int bit = 26 * i, j = bit >> 5, sh = bit & 31;
    const uint64_t pl = ((((uint64_t)P[j + 1 < 9 ? j + 1 : 8] << 32) | P[j]) >> sh) & 0x3ffffffu;
    t[i] = (uint64_t)(c0 * (int64_t)acc[10 * base + i] + c1 * (int64_t)acc[10 * base + 10 + i]) + (pl << 14);
  }
  return fr_of_limb_sums(t);
}
// value k itself
__device__ __forceinline__ Fr acc_value(const unsigned long long* acc, uint32_t k) {
  uint64_t t[10];
#pragma unroll
  for (int i = 0; i < 10; ++i) t[i] = acc[10 * k + i];
  return fr_of_limb_sums(t);
}
// 8 words, 16-byte aligned
__device__ __forceinline__ Fr ld_rec(const uint32_t* p) {
  const u32x4 a = reinterpret_cast<const u32x4*>(p)[0], b = reinterpret_cast<const u32x4*>(p)[1];
  return fr_from_limbs(a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w);
}
__device__ __forceinline__ void st_rec(uint32_t* p, const Fr& v) {
  reinterpret_cast<u32x4*>(p)[0] = u32x4{v.w[0], v.w[1], v.w[2], v.w[3]};
  reinterpret_cast<u32x4*>(p)[1] = u32x4{v.w[4], v.w[5], v.w[6], v.w[7]};
}
// e folded by r with e': e + r (e' - e)
__device__ __forceinline__ Fr fr_fold(const Fr& r, const Fr& x0, const Fr& x1) {
  return fr_add(x0, fr_mul(r, fr_sub(x1, x0)));
}
__device__ __forceinline__ Fr fr_pick(bool c, const Fr& a, const Fr& b) {
  Fr r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.w[j] = c ? a.w[j] : b.w[j];
  return r;
}
// the quadratic with values v0, v1 at 0 and 1 and leading coefficient v2, at r
__device__ __forceinline__ Fr fr_eval2(const Fr& v0, const Fr& v1, const Fr& v2, const Fr& r) {
  return fr_add(v0, fr_mul(r, fr_add(fr_sub(fr_sub(v1, v0), v2), fr_mul(r, v2))));
}
// eq1(u, X) = (1 - u) + X (2 u - 1) as om + X slope, and its value at X = k (per lane, k <= 3)
__device__ __forceinline__ Fr fr_eq1(const Fr& u, uint32_t k, Fr& om, Fr& slope) {
  om = fr_sub(fr_R(), u);
  slope = fr_sub(u, om);
  Fr e = om;
#pragma unroll
  for (uint32_t q = 0; q < 3; ++q) {
    const Fr n = fr_add(e, slope);
#pragma unroll
    for (int j = 0; j < 8; ++j) e.w[j] = k > q ? n.w[j] : e.w[j];
  }
  return e;
}
// x in vector registers: the compiler computes products of wave-uniform
// values on the scalar unit, four instructions per partial product
__device__ __forceinline__ Fr fr_vgpr(Fr x) {
#pragma unroll
  for (int j = 0; j < 8; ++j) asm("" : "+v"(x.w[j]));
  return x;
}
// x of lane + N within rows of 16 lanes (zero past the row)
template <int N>
__device__ __forceinline__ Fr fr_row_shl(const Fr& x) {
  Fr r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.w[j] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x.w[j], 0x100 + N, 0xf, 0xf, true);
  return r;
}

template <int K, int NW>
__device__ __forceinline__ Fr block_sum_lanes(const Fr (&v)[K], uint32_t* lds) {
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    uint32_t x[10];
#pragma unroll
    for (int i = 0; i < 10; ++i) {
      const int bit = 26 * i, j = bit >> 5, sh = bit & 31;
      x[i] = (sh == 0 ? v[k].w[j] : (j < 7 ? __builtin_amdgcn_alignbit(v[k].w[j + 1], v[k].w[j], sh) : v[k].w[7] >> sh)) &
             0x3ffffffu;
    }
    wave_add10(x);
    if (lane == 63)
#pragma unroll
      for (int i = 0; i < 10; ++i) lds[(k * 10 + i) * NW + wave] = x[i];
  }
  __syncthreads();
  Fr r = fr_zero();
  if (wave == 0) {
    const uint32_t k = lane < K ? lane : K - 1;
    uint64_t t[10];
#pragma unroll
    for (int i = 0; i < 10; ++i) {
      t[i] = 0;
#pragma unroll
      for (int q = 0; q < NW; ++q) t[i] += lds[(k * 10 + i) * NW + q];
    }
    r = fr_of_limb_sums(t);
  }
  return r;
}

// rounds workgroup: 8 waves, two per SIMD (16 waves take a round of 256 pairs
// in 5 instead of 6 us, later ones no faster, but need a CU to themselves beside running
// contractions)
constexpr int kRoundsBlock = 512;

// canonical element c to 32 proof bytes (little-endian words); word stores
// when the destination is 4-byte aligned
__device__ __forceinline__ void put_canon(uint8_t* dst, const Fr& c) {
  if ((reinterpret_cast<uintptr_t>(dst) & 3u) == 0) {
    uint32_t* d = reinterpret_cast<uint32_t*>(dst);
#pragma unroll
    for (int j = 0; j < 8; ++j) d[j] = c.w[j];
  } else {
    uint8_t b[32];
    fr_to_bytes(c, b);
    for (int i = 0; i < 32; ++i) dst[i] = b[i];
  }
}

__device__ __forceinline__ void lds_put(uint32_t* dst, const Fr& v) {
#pragma unroll
  for (int j = 0; j < 8; ++j) dst[j] = v.w[j];
}
__device__ __forceinline__ Fr lds_get(const uint32_t* src) {
  Fr v;
#pragma unroll
  for (int j = 0; j < 8; ++j) v.w[j] = src[j];
  return v;
}

__device__ __forceinline__ Fr lds_or_global_fr(const uint32_t* src) {
  Fr v;
#pragma unroll
  for (int j = 0; j < 8; ++j) v.w[j] = src[j];
  return v;
}

__device__ __forceinline__ Fr readlane_fr(const Fr& x, int l) {
  Fr r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.w[j] = __builtin_amdgcn_readlane(x.w[j], l);
  return r;
}

// LDS words of one workgroup's transcript: the state, a message's values (up
// to five), the message words and the challenge.
struct RoundLds {
  uint32_t st[8];
  uint32_t v[40];
  uint32_t w[64];
  uint32_t r[8];
};
__device__ __forceinline__ uint32_t rotv(uint32_t x, int n) { return __builtin_amdgcn_alignbit(x, x, n); }
__device__ __forceinline__ uint32_t xor3v(uint32_t a, uint32_t b, uint32_t c) { return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96); }
__device__ __forceinline__ uint32_t sha_s0(uint32_t x) { return xor3v(rotv(x, 7), rotv(x, 18), x >> 3); }
__device__ __forceinline__ uint32_t sha_s1(uint32_t x) { return xor3v(rotv(x, 17), rotv(x, 19), x >> 10); }
#define VL_SHA_IV {0x6a09e667u, 0xbb67ae85u, 0x3c6ef372u, 0xa54ff53au, 0x510e527fu, 0x9b05688cu, 0x1f83d9abu, 0x5be0cd19u}

// Word `lane` of the padded message state || label || K values, written to T.w by
// each lane (K <= 5: at most four blocks).  The label's first four letters are
// word 8; up to two more (label2, below 256 for one) begin word 9, so word i >=
// 9 holds the last bytes of value word i - 10 and the first ones of i - 9.
// Returns the number of blocks.
__device__ __forceinline__ uint32_t tr_message(RoundLds& T, uint32_t label4, uint32_t label2, int K) {
  const int n = label2 == 0 ? 0 : (label2 < 256 ? 1 : 2);
  const int N = 32 + 4 + n + 32 * K, NB = (N + 9 + 63) / 64;
  auto word = [&](int d) -> uint32_t {
    const uint32_t x = d < 8 * K ? T.v[d < 0 ? 0 : d] : (d == 8 * K ? 0x80u : 0u);
    return __builtin_amdgcn_perm(x, x, 0x00010203u);
  };
  const int i = (int)(threadIdx.x & 63u);
  const uint32_t lo = word(i - 9), hi = i >= 10 ? word(i - 10) : label2;
  uint32_t m = __builtin_amdgcn_alignbit(hi, lo, 8 * n);
  if (i < 8) m = T.st[i & 7];
  if (i == 8) m = label4;
  if (i == 16 * NB - 1) m = N * 8;
  T.w[i] = m;
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  return (uint32_t)NB;
}

// One SHA-256 hash on two lanes four apart: the one in the even bank of four
// lanes has a, b, c, d and forms S0(a) + maj(a, b, c), the one in the odd bank
// has e, f, g, h and forms t1 = S1(e) + ch(e, f, g) + h + wk.  The same
// instructions serve both: rotations by per-lane amounts, and maj(a, b, c) is
// the choice between b and c by ~(a ^ b).  Ten instructions a round instead of
// 14; a wave issues one per four cycles and that bounds a transcript.
struct ShaLane {
  uint32_t odd;          // 1 in the lane of e .. h
  uint32_t r1, r2, r3;   // rotations
  uint32_t m;            // all ones in the lane of a .. d
};
__device__ __forceinline__ ShaLane sha_lane(uint32_t lane) {
  ShaLane L;
  L.odd = (lane >> 2) & 1u;
  L.r1 = L.odd ? 6u : 2u;
  L.r2 = L.odd ? 11u : 13u;
  L.r3 = L.odd ? 25u : 22u;
  L.m = L.odd ? 0u : ~0u;
  return L;
}
// x of the lane four below in odd banks (old elsewhere), or four above in even ones
__device__ __forceinline__ uint32_t sha_to_odd(uint32_t old, uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, 0x114, 0xf, 0xa, false);   // row_shr:4
}
__device__ __forceinline__ uint32_t sha_to_even(uint32_t old, uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)old, (int)x, 0x104, 0xf, 0x5, false);   // row_shl:4
}
// one round: the new a or e replaces s3; u holds h + wk of this round in odd
// lanes and zero in even ones, and leaves as that of the next (its word w).
// An instruction's result is read across lanes three instructions later.
#define VL_SHA_RND(s0, s1, s2, s3, w)                                            \
  "v_alignbit_b32 %[x], %[" s0 "], %[" s0 "], %[r1]\n"                           \
  "v_alignbit_b32 %[y], %[" s0 "], %[" s0 "], %[r2]\n"                           \
  "v_alignbit_b32 %[z], %[" s0 "], %[" s0 "], %[r3]\n"                           \
  "v_bitop3_b32 %[f], %[" s0 "], %[" s1 "], %[m] bitop3:0xd2\n"                  \
  "v_bitop3_b32 %[x], %[x], %[y], %[z] bitop3:0x96\n"                            \
  "v_bitop3_b32 %[f], %[f], %[" s1 "], %[" s2 "] bitop3:0xca\n"                  \
  "v_add3_u32 %[t], %[x], %[f], %[u]\n"                                          \
  "v_add_u32_dpp %[u], %[" s2 "], %[" w "] quad_perm:[0,1,2,3] row_mask:0xf bank_mask:0xa\n" \
  "v_add_u32_dpp %[" s3 "], %[" s3 "], %[t] row_shr:4 row_mask:0xf bank_mask:0xa\n" \
  "v_add_u32_dpp %[" s3 "], %[t], %[t] row_shl:4 row_mask:0xf bank_mask:0x5\n"
__device__ __forceinline__ void sha_four(uint32_t (&s)[4], uint32_t& u, const ShaLane& L, uint32_t w1, uint32_t w2,
                                         uint32_t w3, uint32_t w4) {
  uint32_t x, y, z, f, t;
  asm(VL_SHA_RND("a", "b", "c", "d", "w1") VL_SHA_RND("d", "a", "b", "c", "w2")
      VL_SHA_RND("c", "d", "a", "b", "w3") VL_SHA_RND("b", "c", "d", "a", "w4")
      : [a] "+v"(s[0]), [b] "+v"(s[1]), [c] "+v"(s[2]), [d] "+v"(s[3]), [u] "+v"(u), [x] "=&v"(x), [y] "=&v"(y),
        [z] "=&v"(z), [f] "=&v"(f), [t] "=&v"(t)
      : [r1] "v"(L.r1), [r2] "v"(L.r2), [r3] "v"(L.r3), [m] "v"(L.m), [w1] "v"(w1), [w2] "v"(w2), [w3] "v"(w3),
        [w4] "v"(w4));
}
#undef VL_SHA_RND

// words 2 k, 2 k + 1 of a schedule in the two lanes (p) and 2 k + 1, 2 k + 2 (q),
// a ring of eight of each: the next pair, i = k mod 8, two words in twelve
// instructions
__device__ __forceinline__ void sha_next_pair(uint32_t (&p)[8], uint32_t (&q)[8], int i) {
  p[i] = p[i] + sha_s0(q[i]) + q[(i + 4) & 7] + sha_s1(p[(i + 7) & 7]);
  q[(i + 7) & 7] = sha_to_odd(q[(i + 7) & 7], p[i]);
  q[i] = sha_to_even(0u, p[i]);   // its odd lanes: with the pair after
}

// One block on the lanes' own schedules (small code: 16 rounds and 16 words in a
// loop): w0, p and q as for sha_next_pair, h the chaining value.
__device__ __forceinline__ void sha_block_lanes(const ShaLane& L, uint32_t w0, uint32_t (&p)[8], uint32_t (&q)[8],
                                                uint32_t (&h)[4]) {
  const uint32_t* KK = sha256_k();
  uint32_t s[4], kk[16];
#pragma unroll
  for (int j = 0; j < 4; ++j) s[j] = h[j];
#pragma unroll
  for (int i = 0; i < 16; ++i) kk[i] = KK[i];
#pragma unroll 1
  for (int it = 0; it < 4; ++it) {
    uint32_t w[16], u;
    w[0] = w0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      w[2 * k + 1] = p[k];
      if (k < 7) w[2 * k + 2] = q[k];
    }
#pragma unroll
    for (int i = 0; i < 16; ++i) w[i] += kk[i];
#pragma unroll
    for (int i = 0; i < 16; ++i) kk[i] = KK[(16 * it + 16 + i) & 63];   // on their way during the rounds
    __builtin_amdgcn_sched_barrier(0);
    u = L.odd ? s[3] + w[0] : 0u;
#pragma unroll
    for (int i = 0; i < 16; i += 4) sha_four(s, u, L, w[i + 1], w[i + 2], w[i + 3], w[(i + 4) & 15]);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      sha_next_pair(p, q, i);
      if (i == 0) w0 = q[7];
    }
  }
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j] += s[j];
}

// absorb(label, x_0 .. x_{K-1}) for a label of four to six letters by all 64 lanes of one
// wave, the K <= 5 canonical values in T.v: one block after the other, every
// lane pair the same (once or twice per proof, so small code counts: it is
// fetched for one pass)
constexpr uint32_t kLblFinal4 = 0x66696e61u, kLblFinal1 = 0x6cu;     // "fina", "l"
constexpr uint32_t kLblPart4 = 0x70617274u;                          // "part"
constexpr uint32_t kLblClaim4 = 0x636c6169u, kLblClaim1 = 0x6du;     // "clai", "m"
constexpr uint32_t kLblRfinal4 = 0x7266696eu, kLblRfinal2 = 0x616cu; // "rfin", "al"
constexpr uint32_t kLblSigma4 = 0x7369676du, kLblSigma1 = 0x61u;     // "sigm", "a"
__device__ __forceinline__ void tr_absorb_lanes(RoundLds& T, uint32_t label4, uint32_t label2, int K) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t NB = tr_message(T, label4, label2, K);
  const ShaLane L = sha_lane(lane);
  constexpr uint32_t iv[8] = VL_SHA_IV;
  uint32_t h[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) h[j] = L.odd ? iv[4 + j] : iv[j];
#pragma unroll 1
  for (uint32_t b = 0; b < NB; ++b) {
    uint32_t p[8], q[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      p[k] = T.w[16 * b + 2 * k + L.odd];
      q[k] = T.w[(16 * b + 2 * k + 1 + L.odd) & 63];   // (word 16 of the last one follows in the block)
    }
    sha_block_lanes(L, T.w[16 * b], p, q, h);
  }
  if ((lane & ~4u) == 0)
#pragma unroll
    for (int j = 0; j < 4; ++j) T.st[lane + j] = h[j];
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// the eight words of a pair's digest in its odd lane, read as a candidate
__device__ __forceinline__ Fr sha_candidate(const uint32_t (&h)[4], uint32_t (&g)[8]) {
  Fr x;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    g[j] = sha_to_odd(0u, h[j]);
    g[4 + j] = h[j];
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) x.w[j] = __builtin_amdgcn_perm(g[j], g[j], 0x00010203u);
  x.w[7] &= 0x7fffffffu;
  return x;
}
// the counter that a lane's pair squeezes with
__device__ __forceinline__ uint32_t sha_counter(uint32_t lane) {
  return (lane >> 4) * 8 + ((lane >> 3) & 1u) * 4 + (lane & 3u);
}
// squeeze(label) for a five-letter label by all 64 lanes of one wave: the new
// state in T.st, the element in Montgomery form in T.r; 32 counters at a time,
// of which one in ten is rejected
__device__ __forceinline__ void tr_squeeze_lanes(RoundLds& T, uint32_t label4, uint32_t label1) {
  const uint32_t lane = threadIdx.x & 63u;
  const ShaLane L = sha_lane(lane);
  constexpr uint32_t iv[8] = VL_SHA_IV;
  uint64_t ok = 0;
  uint32_t g[8];
  Fr x;
#pragma unroll 1
  for (uint32_t base = 0; ok == 0; base += 32) {
    const uint32_t c = base + sha_counter(lane);
    // word 8: label4, 9: the last letter and the counter's low bytes (below 2^16), 10: padding
    const uint32_t w9 = (label1 << 24) | ((c & 0xffu) << 16) | (c & 0xff00u), bits = 41 * 8;
    uint32_t p[8], q[8], h[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      p[k] = T.st[2 * k + L.odd];
      q[k] = k < 3 ? T.st[2 * k + 1 + L.odd] : (L.odd ? label4 : T.st[7]);
    }
    p[4] = L.odd ? w9 : label4;
    q[4] = L.odd ? 0x00800000u : w9;
    p[5] = L.odd ? 0u : 0x00800000u;
    q[5] = p[6] = q[6] = 0u;
    p[7] = L.odd ? bits : 0u;
    q[7] = bits;
#pragma unroll
    for (int j = 0; j < 4; ++j) h[j] = L.odd ? iv[4 + j] : iv[j];
    sha_block_lanes(L, T.st[0], p, q, h);
    x = sha_candidate(h, g);
    ok = __ballot(L.odd && fr_lt_p(x));
  }
  const Fr xm = fr_to_mont(x);
  if (lane == (uint32_t)__builtin_ctzll(ok))
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      T.st[j] = g[j];
      T.r[j] = xm.w[j];
    }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
}
// the state as 32 digest bytes, by one lane
__device__ __forceinline__ void tr_put_digest(const RoundLds& T, uint8_t* out) {
#pragma unroll 1
  for (int i = 0; i < 8; ++i)
#pragma unroll
    for (int q = 0; q < 4; ++q) out[4 * i + q] = (uint8_t)(T.st[i] >> (24 - 8 * q));
}

// absorb("round", g(0..K-1)) and squeeze("r") by all 64 lanes of one wave, K =
// 3 or 4: T.v holds the canonical values (8 K words), T.st the state; leaves
// the new state in T.st and the challenge, in Montgomery form, in T.r.  The
// same digests as tr_absorb_frs and tr_squeeze_fixed.
// Bound by the issue of one wave's instructions, 4 cycles each, so lanes share
// what they can: lane i builds message word i; the lane pair of block b < 3
// makes its schedule and the chaining value moves from pair to pair; pair c
// squeezes with counter c, so that a rejected candidate (one in ten) costs
// nothing.  Both hashes pass through the same code.  7.9 us; 10.2
// with a hash in one lane and the schedule word by word.
__device__ __forceinline__ void tr_round(RoundLds& T, int K) {
  const uint32_t lane = threadIdx.x & 63u;
  tr_message(T, 0x726f756eu, 0x64u, K);   // "roun", "d": three blocks
  const uint32_t blk = min(lane & 3u, 2u);
  constexpr uint32_t KK[64] = {VL_SHA256_K};   // literals: scalar loads of them took longer
  ShaLane L = sha_lane(lane);
  asm("" : "+v"(L.r1), "+v"(L.r2), "+v"(L.r3), "+v"(L.m));
  uint32_t w0 = T.w[16 * blk], p[8], q[8], h[4];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    p[k] = T.w[16 * blk + 2 * k + L.odd];
    q[k] = T.w[16 * blk + 2 * k + 1 + L.odd];   // (word 16 of the last one follows below)
  }
  uint32_t base = 0;   // phase 0: absorb; then counters base ..
#pragma unroll 1
  for (uint32_t phase = 0;; ++phase) {
    constexpr uint32_t iv[8] = VL_SHA_IV;
    uint32_t w[64];
    w[0] = w0;
#pragma unroll
    for (int k = 0; k < 32; ++k) {
      const int i = k & 7;
      if (k >= 8) {
        sha_next_pair(p, q, i);
        w[2 * k] = q[(i + 7) & 7];
      } else if (k > 0) {
        w[2 * k] = q[k - 1];
      }
      w[2 * k + 1] = p[i];
    }
#pragma unroll
    for (int i = 0; i < 64; ++i) w[i] += KK[i];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      h[j] = L.odd ? iv[4 + j] : iv[j];
      asm("" : "+v"(h[j]));
    }
#pragma unroll 1
    for (uint32_t b = 0; b < (phase ? 1u : 3u); ++b) {
      uint32_t s[4], u = L.odd ? h[3] + w[0] : 0u;
#pragma unroll
      for (int j = 0; j < 4; ++j) s[j] = h[j];
#pragma unroll
      for (int i = 0; i < 64; i += 4) sha_four(s, u, L, w[i + 1], w[i + 2], w[i + 3], w[(i + 4) & 63]);
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        h[j] += s[j];
        // to the next block's pair (row_shr:1); after the last block lanes 2
        // and 6 hold the digest, and 3 and 7 get it
        if (!phase) h[j] = (uint32_t)__builtin_amdgcn_update_dpp((int)h[j], (int)h[j], 0x111, 0xf, 0xf, false);
      }
    }
    uint32_t d[9];
    if (phase == 0) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        d[j] = (uint32_t)__builtin_amdgcn_readlane((int)h[j], 3);
        d[4 + j] = (uint32_t)__builtin_amdgcn_readlane((int)h[j], 7);
      }
      if (lane == 0)
#pragma unroll
        for (int j = 0; j < 8; ++j) T.st[j] = d[j];
    } else {
      uint32_t g[8];
      const Fr x = sha_candidate(h, g);
      const uint64_t ok = __ballot(L.odd && fr_lt_p(x));
      if (ok) {
        const Fr xm = fr_to_mont(x);
        if (lane == (uint32_t)__builtin_ctzll(ok))
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            T.st[j] = g[j];
            T.r[j] = xm.w[j];
          }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        return;
      }
      base += 32;
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = T.st[j];
    }
    // state || "r", the counter (below 2^16) || padding
    const uint32_t c = base + sha_counter(lane);
    d[8] = 0x72000000u | ((c & 0xffu) << 16) | (c & 0xff00u);
    w0 = d[0];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      p[k] = L.odd ? d[2 * k + 1] : d[2 * k];
      q[k] = L.odd ? d[2 * k + 2] : d[2 * k + 1];
    }
    p[4] = L.odd ? 0x00800000u : d[8];
    q[4] = L.odd ? 0u : 0x00800000u;
    p[5] = p[6] = q[5] = q[6] = 0u;
    p[7] = L.odd ? 37 * 8 : 0u;
    q[7] = 37 * 8;
  }
}

}  // namespace vl
