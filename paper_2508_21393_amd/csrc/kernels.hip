// Device kernels of the matmul-sumcheck prover (gfx950), apart from the
// integer contractions (contract.hip).
//
// Paths and the paper passages they compute:
//   eq_kernel        eq(x, i) tables, eq. (MLE) Lagrange basis, and their
//                    signed-digit pack form for the contractions
//   pass1_kernel     the claim's dot product and round 1 of every product
//                    as partial sums across the GPU
//   rounds_kernel    claim c = C~(u, v), the sumcheck rounds (Sec. II-B.1)
//                    with Fiat-Shamir challenges, and the fold of each round
//   lift/export      integer -> Fr lifting (x < 0 -> p - |x|) and back to
//                    canonical form
//   upload/copy_in   job descriptors to the workspace
#include <cstring>

#include "device.hpp"
#include "rounds_dev.hpp"
#include "sha256.hpp"

namespace vl {

// ---------------------------------------------------------------- eq -------
// Entry i of an eq table is a product of n factors: x_j for bit 1 and 1 - x_j
// for bit 0, b_1 the most significant bit.  A block has kEqBlock = 2^8
// consecutive entries, one per thread: two tables of 16 products over the low
// variables, four lanes multiplying an entry's factors as a tree, and the
// block's product over the others (with the form's constant)
// likewise; then two products an entry.  Bound by that chain of about seven
// products: with n + 4 of them in sequence on a thread of four entries, and 41
// KB of code, the single 64 x 128 x 32 product's tables took 15 us and the 7B
// block's 36, now 5.4 and 23.
struct EqLds {
  uint32_t g[2][16][8];
  uint32_t up[8];
};
// the form an entry is multiplied into: times R once more, as the factors are
// (Montgomery), or out of Montgomery form
enum EqForm { EQ_CANON = 0, EQ_MONT = 1, EQ_R2 = 2 };
// Entry 256 blk + threadIdx.x (or a product without meaning past 2^n), in form
// `form`, then taken `down` forms lower in `low`.
template <typename P>
__device__ __forceinline__ Fr eq_entry(const P& point, uint32_t n, uint32_t blk, uint32_t form, uint32_t down,
                                       EqLds& T, Fr& low) {
  const uint32_t tid = threadIdx.x;
  const uint32_t nu = n > 8 ? n - 8 : 0;
  if (tid < 192) {
    // threads 4 e + k < 128: factor k of group entry e; 128 + m: the block's
    // factor m
    const bool grp = tid < 128;
    const uint32_t e = (tid >> 2) & 15u, k = tid & 3u, m = tid - 128;
    const uint32_t bit = grp ? 4 * (tid >> 6) + k : 8 + m;
    const uint32_t set = grp ? (e >> k) & 1u : (m < 32 ? (blk >> m) & 1u : 0u);
    Fr f = fr_R();
    if (bit < n) {
      const Fr x = point(n - 1 - bit);
      f = set ? x : fr_sub(f, x);
    } else if (!grp && m == nu && form != EQ_MONT) {
      // a product with R^2 (R^3 / R) or with 1
      f = fr_R2();
      if (form == EQ_CANON)
#pragma unroll
        for (int j = 0; j < 8; ++j) f.w[j] = j == 0 ? 1u : 0u;
    }
    const uint32_t width = grp ? 4u : nu + 1;
#pragma unroll 1
    for (uint32_t off = 1; off < width; off <<= 1) {
      Fr o;
#pragma unroll
      for (int j = 0; j < 8; ++j) o.w[j] = __shfl_xor(f.w[j], (int)off, kWave);
      f = fr_mul(f, o);
    }
    if (grp ? k == 0 : m == 0) lds_put(grp ? T.g[tid >> 6][e] : T.up, f);
  }
  __syncthreads();
  Fr e = lds_get(T.g[0][tid & 15u]), out = e;
#pragma unroll 1
  for (uint32_t q = 0; q < 2 + down; ++q) {
    Fr f;
#pragma unroll
    for (int j = 0; j < 8; ++j) f.w[j] = j == 0 ? 1u : 0u;
    if (q < 2) f = lds_get(q ? T.up : T.g[1][(tid >> 4) & 15u]);
    e = fr_mul(e, f);
    if (q < 2) out = e;
  }
  low = e;
  return out;
}

__global__ void __launch_bounds__(kEqBlock) eq_kernel(const EqJob* __restrict__ jobs, uint32_t n_jobs,
                                                      uint32_t n_blocks) {
  __shared__ EqLds T;
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  uint32_t lo = 0, hi = n_jobs;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (jobs[mid].block_begin <= blk) lo = mid; else hi = mid;
  }
  const EqJob& J = jobs[lo];
  const uint32_t b = blk - J.block_begin;
  // the pack holds e R^2 or e R (level 2 or 1), the table e R or e (1 or 0)
  const uint32_t eq_form = J.eq_canon ? EQ_CANON : EQ_MONT;
  const uint32_t form = J.pack ? (J.pack_r2 ? EQ_R2 : EQ_MONT) : eq_form;
  Fr low;
  const uint32_t* pt = J.point;
  const Fr e = eq_entry([&](uint32_t j) { return lds_or_global_fr(pt + 8 * j); }, J.nvars, b, form,
                        J.eq ? form - eq_form : 0u, T, low);
  const uint64_t i = (uint64_t)b * kEqBlock + threadIdx.x;
  if (J.eq && i < (1ull << J.nvars)) store_sol(J.eq, J.eq_ld, i, low);
  if (J.pack && i < J.pack_len) signed_digits(e, J.pack + i * 8);
}

// eq table for a point passed by value (vl_eq_table): no device staging
__global__ void __launch_bounds__(kEqBlock) eq_point_kernel(EqPointArgs a) {
  __shared__ EqLds T;
  Fr low;
  const Fr e = eq_entry([&](uint32_t j) { return lds_or_global_fr(a.pt[j]); }, a.nvars, blockIdx.x, EQ_MONT, 0u,
                        T, low);
  const uint64_t i = (uint64_t)blockIdx.x * kEqBlock + threadIdx.x;
  if (i < (1ull << a.nvars)) store_sol(a.out, a.ld, i, e);
}

// pack form of a caller-provided eq vector (vl_mle_partial_eval)
__global__ void __launch_bounds__(256) pack_kernel(const uint32_t* __restrict__ eq, uint64_t ld,
                                                   uint64_t len, uint32_t* __restrict__ pack) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= len) return;
  signed_digits(fr_to_mont(load_sol(eq, ld, i)), pack + i * 8);
}

// ---------------------------------------------------------------- rounds ----
// A round of product p sums, over the pairs t < h, the quadratic
//     (a_t + X (a_{t+h} - a_t)) (b_t + X (b_{t+h} - b_t))
// by its values at 0 and 1 and its leading coefficient ("points" 0, 1, 2); the
// messages g(0), g(1), g(2) follow from the three sums.  The a~ tables are in
// Montgomery form and the b~ tables in canonical form, so every product, and
// with it every sum and message, is canonical; folding by r in Montgomery form
// keeps both forms.

// LDS sums (ten limb sums each): the claim, three values per product for its
// first round, and the three of the round at hand
constexpr uint32_t kMatAccProd = 1, kMatAccRound = 1 + 3 * VL_MAX_PRODS;
constexpr uint32_t kMatAccWords = 10 * (kMatAccRound + 3);
// in the rounds kernel behind those, twice: the three values of the next round
// with the tables folded by 0, by 1, and their leading coefficients in the
// challenge
constexpr uint32_t kMatAccNext = kMatAccRound + 3, kMatAccNextLen = 9;

// the product at point pt of a pair, from its table entries e[0] (point 2: the
// difference of the pair's) and, to be folded by r, e[1]
struct MatTerm {
  Fr A, B, val;
};
__device__ __forceinline__ MatTerm mat_term(const Fr (&ea)[2], const Fr (&eb)[2], const Fr& r) {
  MatTerm o;
  o.A = fr_fold(r, ea[0], ea[1]);
  o.B = fr_fold(r, eb[0], eb[1]);
  o.val = fr_mul(o.A, o.B);
  return o;
}

// sums of the pass-1 partials into acc (zeroed), by all nw waves of the
// workgroup: value 0 the claim, kMatAccProd + 3 p + q value q of product p
__device__ __forceinline__ void mat_sum_first(const RoundsJob& J, unsigned long long* acc, uint32_t nw) {
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
#pragma unroll 1
  for (uint32_t v = wave; v < kMatAccProd + 3 * J.n_prods; v += nw) {
    const uint32_t p = v ? (v - kMatAccProd) / 3 : 0, q = v ? (v - kMatAccProd) % 3 : 0;
    const uint32_t* part = v ? J.prods[p].g_part + 8 * q : J.c_part;
    const uint32_t n = v ? J.prods[p].g_nparts : J.c_nparts;
    Fr x = fr_zero();
    for (uint32_t i = lane; i < n; i += kWave) x = fr_add(x, ld_rec(part + 24ull * i));
    acc_add(acc, v, x);
  }
}
// sums of wide round rd >= 1 into acc's round values, by waves 0 .. 2
__device__ __forceinline__ void mat_sum_wide(const RoundsJob& J, uint32_t rd, unsigned long long* acc) {
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  if (wave >= 3) return;
  const uint32_t h = 1u << (J.prods[0].n1 - 1 - rd), nb = h / mat_span(h);
  Fr x = fr_zero();
  for (uint32_t i = lane; i < nb; i += kWave) x = fr_add(x, ld_rec(mat_part(J, rd, i) + 8 * wave));
  acc_add(acc, kMatAccRound + wave, x);
}
// The statement, by wave 0: the prover guard (c equals the sum of every
// product's g(0) + g(1)), then the claim and the part claims written (by one
// workgroup) and absorbed.
__device__ __forceinline__ bool mat_claim(const RoundsJob& J, const unsigned long long* acc, RoundLds& T, bool write) {
  const uint32_t lane = threadIdx.x & 63u, n = J.n_prods;
  if (lane < 8) T.st[lane] = J.st[lane];
  // lane p < n: product p's sum; lane 8: c
  const uint32_t v0 = lane < n ? kMatAccProd + 3 * lane : 0;
  uint64_t t[10];
#pragma unroll
  for (int i = 0; i < 10; ++i) t[i] = acc[10 * v0 + i] + (lane < n ? acc[10 * v0 + 10 + i] : 0ull);
  const Fr mine = fr_of_limb_sums(t);
  Fr sum = mine;
#pragma unroll
  for (int j = 0; j < 8; ++j) sum.w[j] = lane < n ? sum.w[j] : 0u;
  sum = fr_add(sum, fr_row_shl<4>(sum));
  sum = fr_add(sum, fr_row_shl<2>(sum));
  sum = fr_add(sum, fr_row_shl<1>(sum));
  if (!fr_eq(readlane_fr(sum, 0), readlane_fr(mine, 8))) return false;
#pragma unroll 1
  for (uint32_t p = 0; p < n; ++p) {   // c, then the sums of products 0 .. n - 2
    if (lane == (p ? p - 1 : 8u)) {
      if (write) put_canon(J.proof + 32 * p, mine);
      lds_put(T.v, mine);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    tr_absorb_lanes(T, p ? kLblPart4 : kLblClaim4, p ? 0u : kLblClaim1, 1);
  }
  return true;
}
// A round's messages from the sums at value v0, and its challenge, by wave 0.
// next: the sums are kMatAccNextLen ones, quadratics in the challenge before,
// T.r.
__device__ __forceinline__ void mat_round(const unsigned long long* acc, uint32_t v0, uint8_t* out, RoundLds& T,
                                          bool write, bool next = false) {
  const uint32_t lane = threadIdx.x & 63u;
  // lane 4 j + k: value k's j-th
  Fr g = acc_point(acc, v0 + (next ? 3 * min(lane >> 2, 2u) : 0), min(lane & 3u, 2u));
  if (next) g = fr_eval2(g, fr_row_shl<4>(g), fr_row_shl<8>(g), fr_vgpr(lds_get(T.r)));
  if (lane < 3) {
    if (write) put_canon(out + 32 * lane, g);
    lds_put(T.v + 8 * lane, g);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  tr_round(T, 3);
}

// Wide round rd >= 1 of product 0 across the GPU, mat_span pairs per block,
// kMatSweepPairs at a time.  Wave 0 of every block first takes round rd - 1's transcript step
// (round 0: also the statement) from the previous launch's sums, so no block
// waits for another and a round is one launch; only the job's first block
// stores proof bytes and io.  Then each thread folds by r_{rd-1} and takes the
// product at one point of a pair; the entries are loaded before the step.
// Bound by the step (about 13 us of 18; the first sweep 25 to 31); with the sums
// by lane shuffles, the squeeze and the statement on one lane it was 30 us, 43
// the first.  256 pairs per block: 22 us.
__global__ void __launch_bounds__(3 * kMatSweepPairs) mat_sweep_kernel(const RoundsJob* __restrict__ jobs,
                                                                       const MatSweep* __restrict__ list,
                                                                       uint32_t n_list, uint32_t n_blocks,
                                                                       uint32_t rd) {
  __shared__ unsigned long long acc[kMatAccWords];
  __shared__ RoundLds T;
  __shared__ int32_t verdict;
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  uint32_t lo = 0, hi = n_list;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (list[mid].block_begin <= blk) lo = mid; else hi = mid;
  }
  const MatSweep& S = list[lo];
  const RoundsJob& J = jobs[S.job];
  if (*reinterpret_cast<volatile const int32_t*>(J.io) != VL_OK) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, pt = tid / kMatSweepPairs;
  const bool write = blk == S.block_begin;
  if (rd == 1 && J.err && *(volatile const int32_t*)J.err) {
    if (write && tid == 0) {
      J.io[0] = (uint32_t)VL_ERR_RANGE;
      *J.status = VL_ERR_RANGE;
    }
    return;
  }
  const RoundsProd& P = J.prods[0];
  const uint64_t ld = P.ld;
  const uint32_t h = 1u << (P.n1 - 1 - rd), span = mat_span(h);   // h is a multiple of span, span of kMatSweepPairs
  uint32_t t = (blk - S.block_begin) * span + tid % kMatSweepPairs;
  const uint32_t end = (blk - S.block_begin + 1) * span;
  Fr ea[2], eb[2];
  auto load = [&]() {
    const uint32_t i0 = pt == 1 ? t + h : t;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      ea[q] = load_sol(P.a, ld, i0 + 2 * q * h);
      eb[q] = load_sol(P.b, ld, i0 + 2 * q * h);
      if (pt == 2) {
        ea[q] = fr_sub(load_sol(P.a, ld, t + h + 2 * q * h), ea[q]);
        eb[q] = fr_sub(load_sol(P.b, ld, t + h + 2 * q * h), eb[q]);
      }
    }
  };
  load();
  for (uint32_t i = tid; i < kMatAccWords; i += 3 * kMatSweepPairs) acc[i] = 0;
  __syncthreads();
  if (rd == 1) {
    mat_sum_first(J, acc, 3 * kMatSweepPairs / kWave);
  } else {
    mat_sum_wide(J, rd - 1, acc);
    if (tid < 8) T.st[tid] = J.io[kMatIoState + 8 * (rd & 1) + tid];
  }
  __syncthreads();
  if (tid < 64) {
    const bool ok = rd > 1 || mat_claim(J, acc, T, write);
    if (lane == 0) verdict = ok ? 1 : 0;
    if (ok) {
      mat_round(acc, rd == 1 ? kMatAccProd : kMatAccRound, J.proof + 32ull * J.n_prods + 96ull * (rd - 1), T, write);
      if (write && lane < 8) {
        J.io[kMatIoState + 8 * ((rd - 1) & 1) + lane] = T.st[lane];
        J.io[kMatIoR + 8 * ((rd - 1) & 1) + lane] = T.r[lane];
      }
      if (lane < 30) acc[10 * kMatAccRound + lane] = 0;
    } else if (write && lane == 0) {
      J.io[0] = (uint32_t)VL_ERR_FALSE_STATEMENT;
      *J.status = VL_ERR_FALSE_STATEMENT;
    }
  }
  __syncthreads();
  if (!verdict) return;
  Fr sum = fr_zero();
#pragma unroll 1
  for (;;) {
    const MatTerm o = mat_term(ea, eb, lds_get(T.r));
    if (pt < 2) {
      const uint32_t i0 = pt == 1 ? t + h : t;
      store_sol(P.a, ld, i0, o.A);
      store_sol(P.b, ld, i0, o.B);
    }
    sum = fr_add(sum, o.val);
    t += kMatSweepPairs;
    if (t >= end) break;   // the same for all threads
    load();                // (other pairs than those stored)
    __syncthreads();       // read by all points before any is stored over
  }
  acc_add(acc, kMatAccRound + pt, sum);
  __syncthreads();
  if (tid < 64) {
    const Fr v = acc_value(acc, kMatAccRound + min(tid, 2u));
    if (tid < 3) st_rec(mat_part(J, rd, blk - S.block_begin) + 8 * tid, v);
  }
}

// Pass 1: the claim's dot product and round 1 of every product as partial
// sums, kPass1Pairs pairs per block, spread over the whole GPU (the rounds
// kernel of a group runs on one CU and only adds the partials).  A thread
// takes one point of its pairs.  Bound by the loads' latency and one product's
// chain; with all three products on a thread and sums by lane shuffles it was
// 12.7 us for the 13B query forward at T 128, now 8.4.
__global__ void __launch_bounds__(kPass1Block) pass1_kernel(const Pass1Job* __restrict__ jobs, uint32_t n_jobs,
                                                            uint32_t n_blocks) {
  __shared__ unsigned long long acc[30];
  const uint32_t blk = blockIdx.x, tid = threadIdx.x, lane = tid & 63u;
  if (blk >= n_blocks) return;
  uint32_t lo = 0, hi = n_jobs;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (jobs[mid].block_begin <= blk) lo = mid; else hi = mid;
  }
  const Pass1Job& J = jobs[lo];
  if (tid < 30) acc[tid] = 0;
  const uint32_t base = (blk - J.block_begin) * kPass1Pairs, end = min(base + kPass1Pairs, J.h);
  // a dot product's entries over all threads, a product's pairs over a third
  const uint32_t step = J.dot ? kPass1Block : kPass1Block / 3, pt = J.dot ? 0 : tid / step;
  Fr g = fr_zero();
#pragma unroll 1
  for (uint32_t t = base + tid % step; t < end; t += step) {
    const uint32_t i0 = pt ? t + J.h : t;
    Fr a = load_sol(J.a, J.a_ld, i0), b = load_sol(J.b, J.b_ld, i0);
    if (pt == 2) {
      a = fr_sub(a, load_sol(J.a, J.a_ld, t));
      b = fr_sub(b, load_sol(J.b, J.b_ld, t));
    }
    g = fr_add(g, fr_mul(a, b));
  }
  __syncthreads();
  acc_add(acc, pt, g);
  __syncthreads();
  if (tid >= 64) return;
  const Fr v = acc_value(acc, min(lane, 2u));
  Fr s[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) s[k] = readlane_fr(v, k);
  if (lane == 0) {
    uint32_t* o = J.out + (uint64_t)(blk - J.block_begin) * 24;
#pragma unroll
    for (int k = 0; k < 3; ++k) st_rec(o + 8 * k, s[k]);
    // persistent mode: count this block for the group's resident rounds
    // workgroup (release: the partials, and everything the earlier
    // kernels of the stream wrote, are visible to whoever sees the count)
    if (J.ready) __hip_atomic_fetch_add(J.ready, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
  }
}

// A long round's tables folded by r in place and its sums added to acc, by all
// threads: the values at 0 and 1 of all pairs t < h, then the leading
// coefficients from the folded entries (small code: three products).
__device__ __noinline__ void mat_fold_long(uint32_t* ga, uint32_t* gb, uint64_t ld, uint32_t h, const uint32_t* rp,
                                           unsigned long long* acc) {
  const Fr r = lds_get(rp);
#pragma unroll 1
  for (uint32_t pt = 0; pt < 3; ++pt) {
    Fr sum = fr_zero();
#pragma unroll 1
    for (uint32_t t = threadIdx.x; t < h; t += kRoundsBlock) {
      const uint32_t i = pt ? t + h : t, i2 = pt < 2 ? i + 2 * h : t;
      Fr A = load_sol(ga, ld, i), B = load_sol(gb, ld, i);
      const Fr dA = fr_sub(load_sol(ga, ld, i2), A), dB = fr_sub(load_sol(gb, ld, i2), B);
      if (pt < 2) {
        A = fr_add(A, fr_mul(r, dA));
        B = fr_add(B, fr_mul(r, dB));
        store_sol(ga, ld, i, A);
        store_sol(gb, ld, i, B);
      } else {
        A = dA;   // (both differences negated)
        B = dB;
      }
      sum = fr_add(sum, fr_mul(A, B));
    }
    acc_add(acc, kMatAccRound + pt, sum);
  }
}

// The rounds of a group, one workgroup each, apart from the wide ones: the
// statement (without wide rounds), then product after product.  The first
// round's sums come from pass 1, or from the last wide round's blocks.  While
// wave 0 hashes round rd, waves 1 .. 7 fold the tables by r_{rd-1} and sum
// round rd + 1 as quadratics in the r_rd not known yet, three products per
// value: of pair t < h they take the entries t, t + 2 h (the value at 0), t + h,
// t + 3 h (at 1) and the differences (the leading coefficient) of the tables
// of 4 h entries.  So a round is the hash and the quadratics at r, with one
// barrier.  A row of 16 lanes takes one of the three values of 16 pairs, a wave
// the same value of four rows.
// Tables of more than kMatLds entries fold in place in global memory, a pair's
// values in one thread (the leading one first, which reads all entries);
// shorter ones are folded from one LDS buffer into the other and a pair's
// values go to different waves.
// That is 21 products a pair of round rd + 1.  Rounds of more than kMatAhead
// pairs (persistent mode, and the later products of a sum) would outlast the
// hash with it: their tables fold after the hash of round rd, 7 products a
// pair on all waves (2^18 inner entries in one workgroup: 2.8 ms, all ahead 7.4).
// Bound by the hash (7.9 of about 10.7 us a round).  With the sums after
// the hash a round took 13 us, before that, with sums by lane shuffles, the
// squeeze and claims on one lane and 183 KB of code, 18, and 30 with 42 groups
// at once; the 64 x 128 x 32 product's rounds 134 us, now 88.  The LDS tables
// hold whole elements (16-byte accesses), and there is one copy of the hash's
// code: a kernel's first pass over code costs as much as several rounds.
__global__ void __launch_bounds__(kRoundsBlock) rounds_kernel(const RoundsJob* __restrict__ jobs) {
  const RoundsJob& J = jobs[blockIdx.x];
  // the rounds are one serial chain per group; when they overlap contraction
  // kernels on the same CUs, their waves go first, and before them the
  // transcript's, which shares its SIMD with another
  if (threadIdx.x < kWave) __builtin_amdgcn_s_setprio(3); else __builtin_amdgcn_s_setprio(2);
  __shared__ alignas(16) uint32_t buf[2][8 * (kMatLds + kMatLds / 2)];   // a, b: two buffers each
  constexpr uint32_t kAcc = 10 * (kMatAccNext + 2 * kMatAccNextLen);
  __shared__ unsigned long long acc[kAcc];
  __shared__ uint32_t rbuf[2][8], fin[2][2][8];              // r_rd by parity; the last pairs
  __shared__ RoundLds T;
  __shared__ int32_t verdict;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;

  if (J.ready) {
    // persistent mode: wait until every pass-1 block of this group has
    // counted itself, at most spin_limit polls.  The polls are relaxed loads
    // and one acquire fence follows the loop (an acquire load per poll would
    // invalidate this XCD's L2 on every poll, under the contraction kernels
    // that share it); the fence pairs with the pass-1 blocks' release
    // increments.
    if (tid == 0) {
      uint32_t polls = 0;
      int32_t ok = 1;
      while (__hip_atomic_load(J.ready, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < J.ready_target) {
        if (++polls > J.spin_limit) {
          ok = 0;
          break;
        }
        __builtin_amdgcn_s_sleep(8);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
      verdict = ok;
    }
    __syncthreads();
    if (!verdict) {
      if (tid == 0) *J.status = VL_ERR_TIMEOUT;
      return;
    }
  }
  const uint32_t wide = J.wide;
  if (wide) {
    // the range flag, the statement and product 0's first rounds were wide
    // launches' work, which left their status in io
    const int32_t st = *reinterpret_cast<volatile const int32_t*>(J.io);
    if (st != VL_OK) {
      if (tid == 0) *J.status = st;
      return;
    }
  } else if (J.err && *(volatile const int32_t*)J.err) {
    if (tid == 0) *J.status = VL_ERR_RANGE;
    return;
  }
  for (uint32_t i = tid; i < kAcc; i += kRoundsBlock) acc[i] = 0;
  __syncthreads();
  mat_sum_first(J, acc, kRoundsBlock / kWave);
  if (wide) {
    mat_sum_wide(J, wide - 1, acc);
    // the state after round wide - 2, the last step a wide launch took
    if (tid < 8) T.st[tid] = J.io[kMatIoState + 8 * (wide & 1) + tid];
  }
  __syncthreads();
  if (!wide) {
    if (wave == 0) {
      const bool ok = mat_claim(J, acc, T, true);
      if (lane == 0) verdict = ok ? 1 : 0;
    }
    __syncthreads();
    if (!verdict) {
      if (tid == 0) *J.status = VL_ERR_FALSE_STATEMENT;
      return;
    }
  }

  uint8_t* out = J.proof + 32ull * J.n_prods;
#pragma unroll 1
  for (uint32_t p = 0; p < J.n_prods; ++p) {
    const RoundsProd& P = J.prods[p];
    uint32_t *const ga = P.a, *const gb = P.b;
    const uint64_t ld = P.ld;
    const uint32_t n1 = P.n1, rd0 = p == 0 && wide ? wide - 1 : 0;
    int at = -1;   // the tables' place: -1 global, else the LDS buffer of kMatLds entries (0) or half of them (1)
    auto get = [&](uint32_t k, uint32_t i) {
      if (at >= 0) return ld_rec(buf[k] + (at ? 8 * kMatLds : 0) + 8 * i);
      return load_sol(k ? gb : ga, ld, i);
    };
    bool fold = false;   // the sums of the round at hand are quadratics; the tables are a round behind
#pragma unroll 1
    for (uint32_t rd = rd0; rd < n1; ++rd) {
      const uint32_t h = rd + 1 < n1 ? 1u << (n1 - 2 - rd) : 0;   // pairs of round rd + 1
      const bool ahead = h <= kMatAhead;
      unsigned long long* const cur = acc + 10 * (kMatAccNext + kMatAccNextLen * (rd & 1));
      unsigned long long* const nxt = acc + 10 * (kMatAccNext + kMatAccNextLen * (~rd & 1));
      // the last round's tables are one pair each, in fin
      const bool lds = fold && h && 4 * h <= kMatLds;
      if (wave == 0) {
        // (one call: its code is large)
        mat_round(fold ? cur : acc, fold ? 0 : (rd == 0 ? kMatAccProd + 3 * p : kMatAccRound), out + 96ull * rd, T, true,
                  fold);
#pragma unroll
        for (uint32_t i = lane; i < 10 * kMatAccNextLen; i += kWave) cur[i] = 0;
        if (!ahead && lane < 30) acc[10 * kMatAccRound + lane] = 0;
        if (lane < 8) rbuf[rd & 1][lane] = T.r[lane];
      } else if (h && ahead) {
        const Fr r = lds_get(rbuf[~rd & 1]);
        const bool split = lds || !fold;   // a pair's values on different waves
        constexpr uint32_t kWaves = kRoundsBlock / kWave - 1, kPtWaves = kWaves / 3;
        const uint32_t chunks = (h + 15) / 16;
        const uint32_t first = 4 * (split ? (wave - 1) / 3 : wave - 1), step = 4 * (split ? kPtWaves : kWaves);
        const bool on = (!split || wave <= 3 * kPtWaves) && first < chunks;
#pragma unroll 1
        for (uint32_t j = 0; on && j < (split ? 1u : 3u); ++j) {
          const uint32_t pt = split ? (wave - 1) % 3 : (j == 0 ? 2 : j - 1);
          Fr sum[3];
          sum[0] = sum[1] = sum[2] = fr_zero();
#pragma unroll 1
          for (uint32_t ch = first + (lane >> 4); ch < chunks; ch += step) {
            const uint32_t t = ch * 16 + (lane & 15u), i0 = pt == 1 ? t + h : t;
            if (t >= h) continue;
            // entries i0 and i0 + 2 h of the tables of round rd (point 2: the
            // differences of the pair's)
            Fr e[2][2];
#pragma unroll
            for (int k = 0; k < 2; ++k)
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                auto entry = [&](uint32_t off) {
                  Fr x = get(k, i0 + off);
                  if (pt == 2) x = fr_sub(get(k, t + h + off), x);
                  return x;
                };
                e[k][q] = entry(2 * q * h);
                if (fold) e[k][q] = fr_fold(r, e[k][q], entry(2 * q * h + 4 * h));
              }
            if (fold && pt < 2) {
              const uint32_t off = at == 0 ? 8 * kMatLds : 0;
#pragma unroll
              for (int q = 0; q < 2; ++q) {
                const uint32_t i = i0 + 2 * q * h;
                if (lds) {
                  st_rec(buf[0] + off + 8 * i, e[0][q]);
                  st_rec(buf[1] + off + 8 * i, e[1][q]);
                } else {
                  store_sol(ga, ld, i, e[0][q]);
                  store_sol(gb, ld, i, e[1][q]);
                }
              }
            }
            sum[0] = fr_add(sum[0], fr_mul(e[0][0], e[1][0]));
            sum[1] = fr_add(sum[1], fr_mul(e[0][1], e[1][1]));
            sum[2] = fr_add(sum[2], fr_mul(fr_sub(e[0][1], e[0][0]), fr_sub(e[1][1], e[1][0])));
          }
#pragma unroll
          for (uint32_t q = 0; q < 3; ++q) acc_add(nxt, 3 * q + pt, sum[q]);
        }
        if (!lds) __threadfence_block();   // the folded entries, for the next round
      } else if (fold && tid < kWave + 4) {   // the last pair of each table
        const uint32_t k = (lane >> 1) & 1u, i = lane & 1u;
        lds_put(fin[k][i], fr_fold(lds_get(rbuf[~rd & 1]), get(k, i), get(k, i + 2)));
      }
      if (lds) at = at == 0 ? 1 : 0;
      __syncthreads();   // r_rd, round rd + 1's sums, the folded entries
      if (!ahead) {
        mat_fold_long(ga, gb, ld, h, rbuf[rd & 1], acc);
        __threadfence_block();
        __syncthreads();   // round rd + 1's sums and tables
      }
      fold = ahead;
    }
    // lane k < 2 of wave 0: the final value of table k, the last challenge
    // folding the remaining pair; a~ out of Montgomery form
    out += 96ull * n1;
    if (wave == 0) {
      const uint32_t k = min(lane, 1u);
      const bool two = n1 > rd0 + 1;
      Fr mine = two ? lds_get(fin[k][0]) : get(k, 0);
      if (n1) mine = fr_fold(lds_get(T.r), mine, two ? lds_get(fin[k][1]) : get(k, 1));
      const Fr canon = fr_from_mont(mine);
      if (k == 0) mine = canon;
      if (lane < 2) {
        put_canon(out + 32 * lane, mine);
        lds_put(T.v + 8 * lane, mine);
      }
      __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
      if (p + 1 < J.n_prods || J.digest) tr_absorb_lanes(T, kLblFinal4, kLblFinal1, 2);
    }
    out += 64;
    __syncthreads();   // the buffers, before the next product's tables
  }
  if (tid == 0) {
    if (J.digest) tr_put_digest(T, J.digest);
    *J.status = VL_OK;
  }
}

// ------------------------------------------------------- chained proofs ----
// M~(x, y) of a chained proof's evaluation step: the pass-1 partials of its
// dot product added (one block per value) and written canonical.
__global__ void __launch_bounds__(256) eval_kernel(const EvalJob* __restrict__ jobs) {
  const EvalJob& J = jobs[blockIdx.x];
  if (J.err && *(volatile const int32_t*)J.err) {
    if (threadIdx.x == 0) *J.status = VL_ERR_RANGE;
    return;
  }
  Fr v[1];
  v[0] = fr_zero();
  for (uint32_t i = threadIdx.x; i < J.nparts; i += 256) v[0] = fr_add(v[0], lds_or_global_fr(J.part + 24ull * i));
  __shared__ uint32_t red[8 * 4];
  wave_sum<1>(v, kWave);
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  if (lane == 0)
#pragma unroll
    for (int j = 0; j < 8; ++j) red[j * 4 + wave] = v[0].w[j];
  __syncthreads();
  if (wave == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) v[0].w[j] = lane < 4 ? red[j * 4 + lane] : 0u;
    wave_sum<1>(v, 4);
    if (lane == 0) {
      put_canon(J.out, v[0]);
      *J.status = VL_OK;
    }
  }
}

// Claim reductions (ReduceJob).  Both phases are sumchecks of
//     sum_k s_k sum_t eq(p_k, t) B_k(t),
// B_k = t_k in phase 1 and the one table M~(r, .) in phase 2.  The challenges
// enter eq(p_k, .) only through a running scalar (see lookup.hip), so a round
// sums the line sum_t eq(p_k's suffix, t) B_k(X, t) by its values at 0 and 1, and
//     g(X) = sum_k sc_k eq1(p_{k,rd}, X) (line_k at X).
// One of the tables and its weights is in Montgomery form and the other
// canonical, so every round value is canonical.  A table W_k starts as
// eq(p_k, .); the weights of a round are the sums of W_k's two halves
// (eq1(p, 0) + eq1(p, 1) = 1), written over its lower half.

// Term (k, pt) of pair t: the fold by r of the entries e (and e' 2 h further
// on) and its product with the weight w0 + w1; two products a term.
struct RedTerm {
  Fr B, w, val;
};
__device__ __forceinline__ RedTerm red_term(const Fr (&e)[2], bool fold, const Fr& r, const Fr& w0, const Fr& w1) {
  RedTerm o;
  o.B = fold ? fr_fold(r, e[0], e[1]) : e[0];
  o.w = fr_add(w0, w1);
  o.val = fr_mul(o.B, o.w);
  return o;
}
// Wave 0's state: lane 4 k + x of each row of 16 has claim k's running scalar
// and that times eq1(p_{k,rd}, x) (row 2 later on, see red_next).
struct RedState {
  Fr sc, sce;
};
__device__ __forceinline__ uint32_t red_claim(const ReduceJob& J, uint32_t lane) { return min((lane & 15u) >> 2, J.K - 1); }
__device__ __forceinline__ void red_set_sce(const ReduceJob& J, uint32_t rd, RedState& s, uint32_t lane) {
  if (rd >= J.n) return;
  Fr om, slope;
  s.sce = fr_mul(s.sc, fr_eq1(lds_or_global_fr(J.pt[red_claim(J, lane)] + 8 * rd), lane & 3u, om, slope));
  if ((lane & 15u) >= 4 * J.K) s.sce = fr_zero();
}
// what round rd starts from (state and running scalars), left by round rd - 1
// in the slot of its parity, and where round rd leaves its challenge: phase 1
// keeps them all
__device__ __forceinline__ uint32_t* red_slot(const ReduceJob& J, uint32_t rd) { return J.io + (rd & 1u ? J.slot : 0u); }
__device__ __forceinline__ uint32_t* red_r(const ReduceJob& J, uint32_t rd) {
  if (J.phase == 1) return J.io + kReduceIoR + 8 * rd;
  return J.io + (rd & 1u ? kReduceIoR : J.slot + kReduceIoR);
}
__device__ __forceinline__ void red_load_state(const ReduceJob& J, uint32_t rd, RedState& s, RoundLds& T, uint32_t lane) {
  const uint32_t k = red_claim(J, lane);
  if (J.phase == 1 && rd == 0) {
#pragma unroll
    for (int j = 0; j < 8; ++j) s.sc.w[j] = J.coef[k][j];
  } else {
    s.sc = lds_or_global_fr(red_slot(J, rd) + kReduceIoSigma + 8 * k);
  }
  if (lane < 8) T.st[lane] = J.phase == 1 && rd == 0 ? J.st[lane] : red_slot(J, rd)[lane];
  red_set_sce(J, rd, s, lane);
}
__device__ __forceinline__ void red_advance(const ReduceJob& J, uint32_t rd, RedState& s, const RoundLds& T, uint32_t lane) {
  Fr om, slope;
  fr_eq1(lds_or_global_fr(J.pt[red_claim(J, lane)] + 8 * rd), 0, om, slope);
  s.sc = fr_mul(s.sc, fr_add(om, fr_mul(slope, fr_vgpr(lds_get(T.r)))));
}
// lane 4 k + x: claim k's line at x, from its sums at 0 and 1
__device__ __forceinline__ Fr red_line(const ReduceJob& J, const unsigned long long* acc, uint32_t lane) {
  return acc_line(acc, 2 * red_claim(J, lane), min(lane & 3u, 2u));
}
// Round rd by wave 0, v its lines' values.  Lanes 0 .. 2 write g(0), g(1), g(2);
// absorbed, r squeezed into T.
__device__ __forceinline__ void red_step(const ReduceJob& J, uint32_t rd, Fr v, const RedState& s, RoundLds& T,
                                         uint32_t lane, bool write = true) {
  v = fr_mul(v, s.sce);
  v = fr_add(fr_add(v, fr_row_shl<4>(v)), fr_add(fr_row_shl<8>(v), fr_row_shl<12>(v)));
  if (lane < 3) {
    if (write) put_canon(J.proof + 96ull * rd + 32 * lane, v);
    lds_put(T.v + 8 * lane, v);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  tr_round(T, 3);
}
// round rd's sums into acc (zeroed), one wave each
__device__ __forceinline__ void red_sum_parts(const ReduceJob& J, uint32_t rd, unsigned long long* acc) {
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t nblocks = (1u << (J.n - 1 - rd)) / kRedSweepPairs;
  if (wave >= 2 * J.K) return;
  Fr v = fr_zero();
  for (uint32_t i = lane; i < nblocks; i += 64) v = fr_add(v, ld_rec(red_part(J, rd, i) + 8 * wave));
  acc_add(acc, wave, v);
}
// the step of wide round rd by wave 0; write: by the one workgroup that stores
// proof bytes and io
__device__ __forceinline__ void red_wide_step(const ReduceJob& J, uint32_t rd, const unsigned long long* acc, RedState& s,
                                              RoundLds& T, uint32_t lane, bool write) {
  red_step(J, rd, red_line(J, acc, lane), s, T, lane, write);
  if (!write) return;
  red_advance(J, rd, s, T, lane);
  uint32_t* io = red_slot(J, rd + 1);
  if (lane < 8) {
    io[lane] = T.st[lane];
    red_r(J, rd)[lane] = T.r[lane];
  }
  if ((lane & 3u) == 0 && lane < 4 * J.K)
#pragma unroll
    for (int j = 0; j < 8; ++j) io[kReduceIoSigma + 2 * lane + j] = s.sc.w[j];
}

// One wide round: the listed jobs, kRedSweepPairs pairs per block; the
// waves take the terms (claim, point) of the pairs in turn.  Tables fold in
// place: every wave reads its terms' entries before any wave writes.
// step: every block first takes round rd - 1's transcript step itself, from the
// previous launch's sums (its first block stores it), so that a round is one
// launch: 22 us instead of 8.3 and 16.2 for a sweep and a step, while
// the launch has no more blocks than CUs (kRedMergeBlocks).
__global__ void __launch_bounds__(2 * kRedSweepPairs * kMaxReduceClaims) reduce_sweep_kernel(
    const ReduceJob* __restrict__ jobs, const MatSweep* __restrict__ list, uint32_t n_list, uint32_t n_blocks,
    uint32_t rd, uint32_t step) {
  __shared__ unsigned long long acc[20 * kMaxReduceClaims + 10];
  __shared__ RoundLds T;
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  uint32_t lo = 0, hi = n_list;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (list[mid].block_begin <= blk) lo = mid; else hi = mid;
  }
  const MatSweep& S = list[lo];
  const ReduceJob& J = jobs[S.job];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, term = tid / kRedSweepPairs, k = term >> 1, pt = term & 1u;
  const uint64_t ld = J.ld, h = 1ull << (J.n - 1 - rd);   // a multiple of kRedSweepPairs
  const uint64_t t = (uint64_t)(blk - S.block_begin) * kRedSweepPairs + tid % kRedSweepPairs;
  const uint64_t i0 = pt ? t + h : t;
  const bool fold = rd > 0, mine = k < J.K;
  Fr e[2], w0 = fr_zero(), w1 = fr_zero(), r = fr_zero();
  e[0] = e[1] = fr_zero();
  uint32_t* tab = nullptr;
  if (mine) {
    tab = J.phase == 1 ? J.b[k] : J.a[0];
    e[0] = load_sol(tab, ld, i0);
    if (fold) e[1] = load_sol(tab, ld, i0 + 2 * h);
    w0 = load_sol(J.w[k], ld, t);
    w1 = load_sol(J.w[k], ld, t + h);
  }
  if (tid < 20 * kMaxReduceClaims + 10) acc[tid] = 0;
  __syncthreads();   // everything read (and acc zeroed)
  if (step) {
    RedState s;
    if (tid < 64) red_load_state(J, rd - 1, s, T, lane);
    red_sum_parts(J, rd - 1, acc);
    __syncthreads();
    if (tid < 64) {
      red_wide_step(J, rd - 1, acc, s, T, lane, blk == S.block_begin);
      if (lane < 20 * kMaxReduceClaims) acc[lane] = 0;
    }
    __syncthreads();
  }
  if (fold) r = step ? lds_get(T.r) : lds_or_global_fr(red_r(J, rd - 1));
  if (mine) {
    const RedTerm o = red_term(e, fold, r, w0, w1);
    if (fold && (J.phase == 1 || k == 0)) store_sol(tab, ld, i0, o.B);
    if (pt == 0) store_sol(J.w[k], ld, t, o.w);
    acc_add(acc, term, o.val);
  }
  __syncthreads();
  if (tid < 64) {
    const Fr v = acc_value(acc, min(tid, 2 * kMaxReduceClaims - 1));
    if (tid < 2 * J.K) st_rec(red_part(J, rd, blk - S.block_begin) + 8 * tid, v);
  }
}

// The transcript step after a wide round, one workgroup per job, where the next
// sweep does not take it.
__global__ void __launch_bounds__(128 * kMaxReduceClaims) reduce_step_kernel(const ReduceJob* __restrict__ jobs,
                                                                            const MatSweep* __restrict__ list,
                                                                            uint32_t rd) {
  __shared__ unsigned long long acc[20 * kMaxReduceClaims + 10];
  __shared__ RoundLds T;
  const ReduceJob& J = jobs[list[blockIdx.x].job];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  if (tid < 20 * kMaxReduceClaims + 10) acc[tid] = 0;
  RedState s;
  if (tid < 64) red_load_state(J, rd, s, T, lane);
  __syncthreads();
  red_sum_parts(J, rd, acc);
  __syncthreads();
  if (tid < 64) red_wide_step(J, rd, acc, s, T, lane, true);
}

// The lines of a later round rd by wave 0 from sums that are linear in
// r_{rd-1}, T.r (acc: a round's sums with the tables folded by 0, then by 1),
// and the scalars' next values, side by side: rows 0 and 1 of 16 lanes have the
// two values, row 2 the scalars.  pts: the claims' points, in LDS.
constexpr uint32_t kRedAccWords = 20 * kMaxReduceClaims;
__device__ __forceinline__ Fr fr_lane(const Fr& x, uint32_t l) {
  Fr r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.w[j] = __shfl(x.w[j], (int)l, kWave);
  return r;
}
__device__ __forceinline__ Fr red_next(const ReduceJob& J, const uint32_t (*pts)[32 * 8], uint32_t rd,
                                       const unsigned long long* acc, RedState& s, const RoundLds& T, uint32_t lane) {
  const bool scalar = lane >= 32;
  const Fr v = red_line(J, acc + (lane & 16u ? kRedAccWords : 0), lane);
  const Fr d = fr_sub(fr_lane(v, lane + 16), v), r = fr_vgpr(lds_get(T.r));
  const uint32_t k = red_claim(J, lane);
  Fr om, slope, om2, slope2;
  fr_eq1(lds_get(pts[k] + 8 * (rd - 1)), 0, om, slope);
  const Fr e = fr_eq1(lds_get(pts[k] + 8 * rd), lane & 3u, om2, slope2);
  const Fr m1 = fr_mul(r, fr_pick(scalar, slope, d));
  s.sc = fr_mul(s.sc, fr_add(om, m1));   // (row 2)
  s.sce = fr_mul(s.sc, e);
  if ((lane & 15u) >= 4 * J.K) s.sce = fr_zero();
  s.sce = fr_lane(s.sce, (lane & 15u) + 32);
  return fr_add(v, m1);
}

// The rounds left after the wide ones, one workgroup per job, and the phase's
// end.  As in the matmul rounds, waves 1 .. 7 sum round rd + 1, as lines in
// r_rd, while wave 0 hashes round rd; a job without wide rounds sums its first
// round before.  Wave 1 + q, 1 + q + 2 K, .. take term q (claim, point), a row
// of 16 lanes 16 pairs.  The tables come from global memory until their first
// fold (at most kLen entries then), the weights until their first sums, and
// live in LDS after that.  With all rounds in this workgroup, both tables
// folded and three products a pair, the 7 tensors of the FFN-up layer took 603
// and 664 us in the two phases; with the sums after the hash the rounds from
// 256 pairs on 160 and 137 us, now 140 and 124.
constexpr uint32_t kRedTailWaves = 8;
__global__ void __launch_bounds__(64 * kRedTailWaves) reduce_kernel(const ReduceJob* __restrict__ jobs) {
  const ReduceJob& J = jobs[blockIdx.x];
  constexpr uint32_t kLen = kRedWidePairs;                                            // entries of the first table buffer
  __shared__ alignas(16) uint32_t buf[kMaxReduceClaims][8 * (kLen + kLen / 2)];       // tables: two buffers each
  __shared__ alignas(16) uint32_t wbuf[kMaxReduceClaims][8 * (kLen / 2 + kLen / 4)];  // weights: two buffers each
  __shared__ unsigned long long acc_s[2][2 * kRedAccWords];                           // a round's sums, by parity
  __shared__ uint32_t rbuf[2][8], fin[kMaxReduceClaims][2][8];                        // r_rd by parity; the last pairs
  __shared__ uint32_t pts[kMaxReduceClaims][32 * 8];
  __shared__ RoundLds T;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
  const uint32_t n = J.n, K = J.K, wide = J.wide, phase = J.phase, ntab = phase == 1 ? K : 1;
  const uint32_t rd0 = wide ? wide - 1 : 0;   // the first round to hash: the last wide one's sums are in its parts
  const uint64_t ld = J.ld;
  int at = -1, wat = -1;   // the tables' and the weights' place: -1 global, else buffer 0 or 1
  auto get = [&](uint32_t k, uint32_t i) {
    if (at >= 0) return ld_rec(buf[k] + (at ? 8 * kLen : 0) + 8 * i);
    return load_sol(phase == 1 ? J.b[k] : J.a[0], ld, i);
  };
  RedState s;
  if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);   // the transcript's wave goes before those it shares its SIMD with
    red_load_state(J, rd0, s, T, lane);
  }
  for (uint32_t i = tid; i < 4 * kRedAccWords; i += 64 * kRedTailWaves) acc_s[i / (2 * kRedAccWords)][i % (2 * kRedAccWords)] = 0;
  for (uint32_t i = tid; i < 8 * n * K; i += 64 * kRedTailWaves) pts[i / (8 * n)][i % (8 * n)] = J.pt[i / (8 * n)][i % (8 * n)];
  __syncthreads();
  if (wide) red_sum_parts(J, rd0, acc_s[rd0 & 1]);
  __syncthreads();
  // rd: the round to hash; tl: the tables' round so far; ready: rd's sums are there
  uint32_t rd = rd0, tl = rd0;
  bool ready = wide > 0;
#pragma unroll 1
  while (rd < n) {
    const bool poly = ready;   // sums of round nx in the challenge r_{nx-1} of the hash at hand
    const uint32_t nx = ready ? rd + 1 : rd, to = ready ? rd : nx;
    const bool fold = tl < to;
    if (wave == 0) {
      if (ready) {
        unsigned long long* const cur = acc_s[rd & 1];
        const Fr v = rd > rd0 ? red_next(J, pts, rd, cur, s, T, lane) : red_line(J, cur, lane);
        red_step(J, rd, v, s, T, lane);
#pragma unroll
        for (uint32_t i = lane; i < 2 * kRedAccWords; i += kWave) cur[i] = 0;
        if (lane < 8) {
          rbuf[rd & 1][lane] = T.r[lane];
          if (phase == 1) J.io[kReduceIoR + 8 * rd + lane] = T.r[lane];   // Montgomery, for eq(r, .)
        }
      }
    } else if (nx < n) {
      const uint32_t h = 1u << (n - 1 - nx), far = poly ? 4 * h : 2 * h;
      const uint32_t groups = (kRedTailWaves - 1) / (2 * K), g = (wave - 1) / (2 * K), term = (wave - 1) % (2 * K);
      const uint32_t k = term >> 1, pt = term & 1u, tab = phase == 1 ? k : 0, chunks = (h + 15) / 16;
      const Fr r = lds_get(rbuf[~to & 1]);
      Fr sum[2];
      sum[0] = sum[1] = fr_zero();
#pragma unroll 1
      for (uint32_t ch = 4 * g + (lane >> 4); g < groups && ch < chunks; ch += 4 * groups) {
        const uint32_t t = ch * 16 + (lane & 15u), i0 = pt ? t + h : t;
        if (t >= h) continue;
        auto entry = [&](uint32_t off) {
          Fr x = get(tab, i0 + off);
          if (fold) {
            x = fr_fold(r, x, get(tab, i0 + off + far));
            if (phase == 1 || k == 0) st_rec(buf[tab] + (at == 0 ? 8 * kLen : 0) + 8 * (i0 + off), x);
          }
          return x;
        };
        const Fr e0 = entry(0);
        Fr w0, w1;
        if (wat >= 0) {
          const uint32_t* w = wbuf[k] + (wat ? 4 * kLen : 0);
          w0 = ld_rec(w + 8 * t);
          w1 = ld_rec(w + 8 * (t + h));
        } else {
          w0 = load_sol(J.w[k], ld, t);
          w1 = load_sol(J.w[k], ld, t + h);
        }
        const Fr w = fr_add(w0, w1), v0 = fr_mul(e0, w);
        if (pt == 0) st_rec(wbuf[k] + (wat == 0 ? 4 * kLen : 0) + 8 * t, w);
        sum[0] = fr_add(sum[0], v0);
        sum[1] = fr_add(sum[1], poly ? fr_mul(entry(2 * h), w) : v0);
      }
      if (g < groups && 4 * g < chunks) {
        acc_add(acc_s[nx & 1], term, sum[0]);
        acc_add(acc_s[nx & 1] + kRedAccWords, term, sum[1]);
      }
    } else if (fold && tid < kWave + 2 * ntab) {   // the last pair of each table
      const uint32_t k = lane >> 1, i = lane & 1u;
      lds_put(fin[k][i], fr_fold(lds_get(rbuf[~to & 1]), get(k, i), get(k, i + 2)));
    }
    if (nx < n) {
      if (fold) at = at == 0 ? 1 : 0;
      tl = to;
      wat = wat == 0 ? 1 : 0;
    }
    rd += ready ? 1 : 0;
    ready = true;
    __syncthreads();   // r, the sums, the folded entries and the next weights
  }
  if (wave != 0) return;
  // lane k < ntab: the last challenge folds the remaining pair of table k
  const uint32_t k1 = min(lane, ntab - 1);
  const bool two = n > 0 && tl + 1 < n;   // the last fold is in fin
  Fr mine = two ? lds_get(fin[k1][0]) : get(k1, 0);
  if (n) mine = fr_fold(lds_get(T.r), mine, two ? lds_get(fin[k1][1]) : get(k1, 1));
  if (phase == 2) mine = fr_from_mont(mine);
  if (lane < ntab) {
    put_canon(J.proof + 96ull * n + 32 * lane, mine);
    lds_put(T.v + 8 * lane, mine);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (phase == 1) {
    // t_k(r) sent and absorbed ("rfinal"); sigma_1 .. sigma_K squeezed for phase 2
    tr_absorb_lanes(T, kLblRfinal4, kLblRfinal2, (int)K);
#pragma unroll 1
    for (uint32_t k = 0; k < K; ++k) {
      tr_squeeze_lanes(T, kLblSigma4, kLblSigma1);
      if (lane < 8) J.io[kReduceIoSigma + 8 * k + lane] = T.r[lane];
    }
    if (lane < 8) J.io[lane] = T.st[lane];
    return;
  }
  tr_absorb_lanes(T, kLblFinal4, kLblFinal1, 1);
  if (lane == 0) {
    if (J.digest) tr_put_digest(T, J.digest);
    if (J.status) *J.status = VL_OK;
  }
}

// ---------------------------------------------------------------- lift ------
template <typename T>
__global__ void __launch_bounds__(256) lift_kernel(const T* __restrict__ src, uint64_t n,
                                                   uint32_t* __restrict__ dst, uint64_t ld) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const int64_t x = (int64_t)src[i];
  const uint64_t mag = x < 0 ? (uint64_t)0 - (uint64_t)x : (uint64_t)x;
  Fr v = fr_zero();
  v.w[0] = (uint32_t)mag;
  v.w[1] = (uint32_t)(mag >> 32);
  if (x < 0) v = fr_sub(fr_zero(), v);
  store_sol(dst, ld, i, fr_to_mont(v));
}

__global__ void __launch_bounds__(256) export_kernel(const uint32_t* __restrict__ src, uint64_t ld,
                                                     uint64_t n, uint32_t* __restrict__ dst) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const Fr c = fr_from_mont(load_sol(src, ld, i));
#pragma unroll
  for (int j = 0; j < 8; ++j) dst[8 * i + j] = c.w[j];
}

// descriptor upload through kernel arguments: the runtime copies the
// arguments at launch, so the host image can be reused at once and nothing
// waits on the stream (also valid inside a captured graph)
__global__ void __launch_bounds__(256) upload_kernel(UploadArgs a) {
  const uint32_t i = threadIdx.x;
  const uint32_t nw = (a.bytes + 3) / 4;
  uint32_t* d = reinterpret_cast<uint32_t*>(a.dst);
  for (uint32_t k = i; k < nw; k += blockDim.x) d[k] = a.words[k];
}

// device copy of a pinned host buffer (src is its device-side address): the
// GPU reads host memory directly, so the copy runs on the caller's stream
// with no copy-engine command, which other streams' copies could queue behind
__global__ void __launch_bounds__(256) copy_in_kernel(u32x4* __restrict__ dst, const u32x4* __restrict__ src,
                                                      uint64_t n16) {
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += (uint64_t)gridDim.x * blockDim.x)
    dst[i] = src[i];
}

__global__ void __launch_bounds__(256) zero_kernel(uint32_t* __restrict__ p, uint64_t n) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = 0;
}

// ---------------------------------------------------------------- launchers -

hipError_t launch_eq(const EqJob* jobs, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(eq_kernel, dim3(n_blocks), dim3(kEqBlock), 0, s, jobs, n_jobs, n_blocks);
  return hipGetLastError();
}

hipError_t launch_eq_point(const EqPointArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(eq_point_kernel, dim3(blocks_for(1ull << a.nvars, kEqBlock)), dim3(kEqBlock), 0, s, a);
  return hipGetLastError();
}

hipError_t launch_pack(const uint32_t* eq, uint64_t ld, uint64_t len, uint32_t* pack,
                       hipStream_t s) {
  if (len == 0) return hipSuccess;
  hipLaunchKernelGGL(pack_kernel, dim3(blocks_for(len, 256)), dim3(256), 0, s, eq, ld, len, pack);
  return hipGetLastError();
}

hipError_t launch_pass1(const Pass1Job* jobs, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(pass1_kernel, dim3(n_blocks), dim3(kPass1Block), 0, s, jobs, n_jobs, n_blocks);
  return hipGetLastError();
}

hipError_t launch_mat_sweep(const RoundsJob* jobs, const MatSweep* list, uint32_t n_list, uint32_t n_blocks,
                            uint32_t round, hipStream_t s) {
  if (!n_blocks) return hipSuccess;
  hipLaunchKernelGGL(mat_sweep_kernel, dim3(n_blocks), dim3(3 * kMatSweepPairs), 0, s, jobs, list, n_list, n_blocks,
                     round);
  return hipGetLastError();
}

hipError_t launch_rounds(const RoundsJob* jobs, uint32_t n_jobs, hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(rounds_kernel, dim3(n_jobs), dim3(kRoundsBlock), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_eval(const EvalJob* jobs, uint32_t n_jobs, hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(eval_kernel, dim3(n_jobs), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_reduce(const ReduceJob* jobs, uint32_t n_jobs, hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_kernel, dim3(n_jobs), dim3(64 * kRedTailWaves), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_reduce_sweep(const ReduceJob* jobs, const MatSweep* list, uint32_t n_list, uint32_t n_blocks,
                               uint32_t round, bool step, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_sweep_kernel, dim3(n_blocks), dim3(2 * kRedSweepPairs * kMaxReduceClaims), 0, s, jobs, list,
                     n_list, n_blocks, round, step ? 1u : 0u);
  return hipGetLastError();
}

hipError_t launch_reduce_step(const ReduceJob* jobs, const MatSweep* list, uint32_t n_list, uint32_t round,
                              hipStream_t s) {
  if (n_list == 0) return hipSuccess;
  hipLaunchKernelGGL(reduce_step_kernel, dim3(n_list), dim3(128 * kMaxReduceClaims), 0, s, jobs, list, round);
  return hipGetLastError();
}

hipError_t launch_lift(const void* src, int dtype, uint64_t n, uint32_t* dst, uint64_t ld,
                       hipStream_t s) {
  if (n == 0) return hipSuccess;
  const dim3 g(blocks_for(n, 256)), b(256);
  switch (dtype) {
    case VL_I16: hipLaunchKernelGGL(lift_kernel<int16_t>, g, b, 0, s, (const int16_t*)src, n, dst, ld); break;
    case VL_I32: hipLaunchKernelGGL(lift_kernel<int32_t>, g, b, 0, s, (const int32_t*)src, n, dst, ld); break;
    case VL_I64: hipLaunchKernelGGL(lift_kernel<int64_t>, g, b, 0, s, (const int64_t*)src, n, dst, ld); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t launch_export(const uint32_t* src, uint64_t ld, uint64_t n, uint32_t* dst, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(export_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, src, ld, n, dst);
  return hipGetLastError();
}

hipError_t launch_upload(void* dst, const void* src, uint64_t bytes, hipStream_t s) {
  const uint8_t* p = reinterpret_cast<const uint8_t*>(src);
  uint8_t* d = reinterpret_cast<uint8_t*>(dst);
  for (uint64_t o = 0; o < bytes; o += kUploadBytes) {
    UploadArgs a;
    a.dst = d + o;
    a.bytes = (uint32_t)((bytes - o) < kUploadBytes ? (bytes - o) : kUploadBytes);
    memcpy(a.words, p + o, a.bytes);
    hipLaunchKernelGGL(upload_kernel, dim3(1), dim3(256), 0, s, a);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_copy_in(void* dst, const void* src, uint64_t bytes, hipStream_t s) {
  if (bytes == 0) return hipSuccess;
  const uint64_t n16 = bytes / 16;
  hipLaunchKernelGGL(copy_in_kernel, dim3((uint32_t)std::min<uint64_t>(blocks_for(n16, 256), 64)), dim3(256), 0, s,
                     reinterpret_cast<u32x4*>(dst), reinterpret_cast<const u32x4*>(src), n16);
  return hipGetLastError();
}

hipError_t launch_zero_words(uint32_t* p, uint64_t n, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(zero_kernel, dim3(blocks_for(n, 256)), dim3(256), 0, s, p, n);
  return hipGetLastError();
}

}  // namespace vl
