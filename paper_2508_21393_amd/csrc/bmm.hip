// Device kernels of the per-head batched matmul sumcheck (vl_bmm_prove).
//
// Attention multiplies one pair of matrices per head (Sec. III-A, eq. (att));
// the H products C_h = A_h B_h are proved with one sumcheck over the head
// variables and the inner variables of
//     C~(rho, u, v) = sum_{h, w} eq(rho, h) A~(h, u, w) B~(h, w, v),
// the multilinear extension of eq. (MLE) over (head, row, column) indices of
// the 3-D tensors, head index most significant.  Head rounds come first: the
// summand is eq(rho, .) a b, of degree 3, sent as g(0..3).  The challenges
// enter eq(rho, .) only through one running scalar (see lookup.hip), so a head
// round sums the quadratic h(X) = sum_t eq(rho's suffix, t) a(X, t) b(X, t) by
// h(0), h(1) and its leading coefficient, and g(X) = scale eq1(rho_rd, X) h(X);
// the inner rounds are the degree-2 rounds of eq. (zk-mle-matmul), the same
// sums without weights, times the scale.
//
//   bmm_start_kernel   the claim c from its pass-1 partials, absorbed; the
//                      suffix tables of eq(rho, .)
//   bmm_sweep_kernel   one round over large tables across the GPU: fold by
//                      the previous challenge and the round's partial sums
//   bmm_step_kernel    one workgroup per job: the round values, the prover
//                      guard (round 1: g(0) + g(1) = c), transcript, challenge
//   bmm_rounds_kernel  one workgroup per job: the remaining rounds and the
//                      final values a_final = A~(r_h, u, r_w),
//                      b_final = B~(r_h, r_w, v)
#include "device.hpp"
#include "rounds_dev.hpp"
#include "sha256.hpp"

namespace vl {

namespace {

// proof byte offset of round rd's values: c, then 4 values per head round
// and 3 per inner round
__device__ __forceinline__ uint64_t bmm_round_off(const BmmJob& J, uint32_t rd) {
  const uint32_t hr = rd < J.nh ? rd : J.nh;
  return 32ull * (1 + 4ull * hr + 3ull * (rd - hr));
}

__device__ __forceinline__ int32_t bmm_io_status(const BmmJob& J) {
  return *reinterpret_cast<volatile const int32_t*>(J.io);
}

// One term of 64 or 16 pairs: the product of the lines a and b at point pt
// (0, 1, or 2 for the leading coefficient), folded by r first, with the
// weight.  a is in Montgomery form and b canonical, so the term is canonical.
// A thread's chain is two folds side by side, the product and the weight.
struct BmmTerm {
  Fr A, B, val;
};
__device__ __forceinline__ BmmTerm bmm_term(const Fr (&ea)[2], const Fr (&eb)[2], bool fold, const Fr& r, bool weigh,
                                            const Fr& w) {
  BmmTerm o;
  o.A = ea[0];
  o.B = eb[0];
  if (fold) {
    o.A = fr_fold(r, ea[0], ea[1]);
    o.B = fr_fold(r, eb[0], eb[1]);
  }
  o.val = fr_mul(o.A, o.B);
  if (weigh) o.val = fr_mul(o.val, w);
  return o;
}
// eq(rho's last m variables, i): bmm_start_kernel leaves the suffix tables in
// E, that of m variables at [2^m, 2^(m+1))
__device__ __forceinline__ Fr bmm_weight(const BmmJob& J, uint32_t m, uint64_t i) {
  return load_sol(J.E, 1ull << J.nh, (1ull << m) + i);
}

// Wave 0's state: the running scalar and, per lane k = lane & 3, that times
// eq1(rho_rd, k) in a head round.
struct BmmState {
  Fr sc, sce;
};
__device__ __forceinline__ void bmm_set_sce(const BmmJob& J, uint32_t rd, BmmState& s, uint32_t lane) {
  s.sce = s.sc;
  if (rd < J.nh) {
    Fr om, slope;
    s.sce = fr_mul(s.sc, fr_eq1(fr_vgpr(lds_or_global_fr(J.rho + 8 * rd)), lane & 3u, om, slope));
  }
}
// the state round rd starts from, left in io by round rd - 1 (or the start) in
// the slot of its parity
__device__ __forceinline__ uint32_t* bmm_slot(const BmmJob& J, uint32_t rd) { return J.io + kBmmIoSlot + 24 * (~rd & 1u); }
__device__ __forceinline__ void bmm_load_state(const BmmJob& J, uint32_t rd, BmmState& s, RoundLds& T, uint32_t lane) {
  const uint32_t* io = bmm_slot(J, rd);
  s.sc = fr_vgpr(lds_or_global_fr(io + kBmmSlotScale));
  if (lane < 8) T.st[lane] = io[lane];
  bmm_set_sce(J, rd, s, lane);
}
// the scalar for round rd + 1, after r is known
__device__ __forceinline__ void bmm_advance(const BmmJob& J, uint32_t rd, BmmState& s, const RoundLds& T, uint32_t lane) {
  if (rd < J.nh) {
    Fr om, slope;
    fr_eq1(fr_vgpr(lds_or_global_fr(J.rho + 8 * rd)), 0, om, slope);
    s.sc = fr_mul(s.sc, fr_add(om, fr_mul(slope, fr_vgpr(lds_get(T.r)))));
  }
  bmm_set_sce(J, rd + 1, s, lane);
}
// Round rd by wave 0: lane k has h(k), forms g(k) and writes it; the values are absorbed and r squeezed into T.  Round 0
// checks the guard g(0) + g(1) = c (false in every lane if it fails).
__device__ __forceinline__ bool bmm_step(const BmmJob& J, uint32_t rd, const Fr& h, const BmmState& s, RoundLds& T,
                                         uint32_t lane, bool write = true) {
  const uint32_t K = rd < J.nh ? 4u : 3u;
  const Fr g = fr_mul(h, s.sce);
  if (rd == 0 && !fr_eq(fr_add(readlane_fr(g, 0), readlane_fr(g, 1)), lds_or_global_fr(J.io + kBmmIoC))) return false;
  if (lane < K) {
    if (write) put_canon(J.proof + bmm_round_off(J, rd) + 32 * lane, g);
    lds_put(T.v + 8 * lane, g);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  tr_round(T, (int)K);
  return true;
}

}  // namespace

// The claim c = C~(rho, u, v) from its pass-1 partials; c is written as the
// first proof element and absorbed.  The other waves turn eq(rho, .) in E into
// the tables of rho's suffixes: the table of m variables is the sum of the two
// halves of the one of m + 1 (eq1(u, 0) + eq1(u, 1) = 1), each thread writing
// over the upper entry it read.
__global__ void __launch_bounds__(256) bmm_start_kernel(const BmmJob* __restrict__ jobs) {
  const BmmJob& J = jobs[blockIdx.x];
  __shared__ RoundLds T;
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  const uint64_t eld = 1ull << J.nh;
  for (uint32_t m = J.nh; m-- > 0;) {
    const uint64_t half = 1ull << m, src = m + 1 == J.nh ? 0 : 2 * half;
    for (uint64_t t = tid; t < half; t += 256)
      store_sol(J.E, eld, half + t, fr_add(load_sol(J.E, eld, src + t), load_sol(J.E, eld, src + half + t)));
    __threadfence_block();
    __syncthreads();
  }
  if (tid >= 64) return;
  if (J.err && *(volatile const int32_t*)J.err) {
    if (lane == 0) {
      J.io[0] = (uint32_t)VL_ERR_RANGE;
      *J.status = VL_ERR_RANGE;
    }
    return;
  }
  Fr c[1];
  c[0] = fr_zero();
  for (uint32_t i = lane; i < J.c_nparts; i += kWave) c[0] = fr_add(c[0], lds_or_global_fr(J.c_part + 24ull * i));
  wave_sum<1>(c, kWave);
  if (lane < 8) T.st[lane] = J.st[lane];
  if (lane == 0) {
    put_canon(J.proof, c[0]);
    lds_put(T.v, c[0]);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  tr_absorb_lanes(T, kLblClaim4, kLblClaim1, 1);
  if (lane < 8) bmm_slot(J, 0)[lane] = T.st[lane];
  if (lane == 0) {
    const Fr one = fr_R();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      J.io[kBmmIoC + i] = c[0].w[i];
      bmm_slot(J, 0)[kBmmSlotScale + i] = one.w[i];
    }
    J.io[0] = (uint32_t)VL_OK;
  }
}

// round rd's sums into acc (zeroed), by waves 0 .. 2
__device__ __forceinline__ void bmm_sum_parts(const BmmJob& J, uint32_t rd, unsigned long long* acc) {
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  if (wave >= 3) return;
  const uint64_t nb = (1ull << (J.nh + J.n1 - 1 - rd)) / kBmmSweepPairs;
  Fr v = fr_zero();
  for (uint64_t i = lane; i < nb; i += 64) v = fr_add(v, ld_rec(bmm_part(J, rd, i) + 8 * wave));
  acc_add(acc, wave, v);
}
// the step of wide round rd by wave 0; write: by the one workgroup that stores
// proof bytes and io
__device__ __forceinline__ bool bmm_wide_step(const BmmJob& J, uint32_t rd, const unsigned long long* acc, BmmState& s,
                                              RoundLds& T, uint32_t lane, bool write) {
  if (!bmm_step(J, rd, acc_point(acc, 0, lane & 3u), s, T, lane, write)) {
    if (write && lane == 0) {
      J.io[0] = (uint32_t)VL_ERR_FALSE_STATEMENT;
      *J.status = VL_ERR_FALSE_STATEMENT;
    }
    return false;
  }
  if (write) {
    uint32_t* io = bmm_slot(J, rd + 1);
    if (lane < 8) {
      io[lane] = T.st[lane];
      io[kBmmSlotR + lane] = T.r[lane];
    }
    bmm_advance(J, rd, s, T, lane);
    if (lane == 0)
#pragma unroll
      for (int i = 0; i < 8; ++i) io[kBmmSlotScale + i] = s.sc.w[i];
  }
  return true;
}

// One wide round: every job of the round's list, kBmmSweepPairs pairs per
// block, the waves in three groups by point.  Round rd > 0 first folds the
// tables by the previous challenge, in place: every wave has read the block's
// entries before any wave writes.  Each block writes its three sums.
// step: every block first takes round rd - 1's transcript step itself, from the
// previous launch's sums (its first block stores it), so that a round is one
// launch.  That pays while the launch has no more blocks than CUs
// (kBmmMergeBlocks): 21 to 30 us instead of 12 and 15.5 for a sweep and a step.
// Bound by the chain of a thread (four products) and of the step.
__global__ void __launch_bounds__(3 * kBmmSweepPairs) bmm_sweep_kernel(const BmmJob* __restrict__ jobs,
                                                                       const BmmSweep* __restrict__ list,
                                                                       uint32_t n_list, uint32_t n_blocks,
                                                                       uint32_t rd, uint32_t step) {
  __shared__ unsigned long long acc[50];   // three values; acc_point reads two past its base
  __shared__ RoundLds T;
  __shared__ uint32_t dead_s;
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  uint32_t lo = 0, hi = n_list;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (list[mid].block_begin <= blk) lo = mid; else hi = mid;
  }
  const BmmSweep& S = list[lo];
  const BmmJob& J = jobs[S.job];
  if (bmm_io_status(J) != VL_OK) return;
  const uint32_t tid = threadIdx.x, lane = tid & 63u, pt = tid / kBmmSweepPairs;
  const uint32_t nv = J.nh + J.n1;
  const uint64_t ld = 1ull << nv, h = 1ull << (nv - 1 - rd);   // at least kBmmWidePairs, a multiple of the block's
  const uint64_t t = (uint64_t)(blk - S.block_begin) * kBmmSweepPairs + tid % kBmmSweepPairs;
  const uint64_t i0 = pt == 1 ? t + h : t;
  const bool fold = rd > 0, head = rd < J.nh;
  Fr ea[2], eb[2];
  ea[0] = load_sol(J.a, ld, i0);
  eb[0] = load_sol(J.b, ld, i0);
  if (fold) {
    ea[1] = load_sol(J.a, ld, i0 + 2 * h);
    eb[1] = load_sol(J.b, ld, i0 + 2 * h);
  }
  if (pt == 2) {
    ea[0] = fr_sub(load_sol(J.a, ld, t + h), ea[0]);
    eb[0] = fr_sub(load_sol(J.b, ld, t + h), eb[0]);
    if (fold) {
      ea[1] = fr_sub(load_sol(J.a, ld, t + 3 * h), ea[1]);
      eb[1] = fr_sub(load_sol(J.b, ld, t + 3 * h), eb[1]);
    }
  }
  Fr w = fr_zero();
  if (head) w = bmm_weight(J, J.nh - 1 - rd, t >> J.n1);
  if (tid < 50) acc[tid] = 0;
  if (tid == 0) dead_s = 0;
  __syncthreads();   // everything read (and acc zeroed)
  if (step) {
    BmmState s;
    if (tid < 64) bmm_load_state(J, rd - 1, s, T, lane);
    bmm_sum_parts(J, rd - 1, acc);
    __syncthreads();
    if (tid < 64) {
      const bool ok = bmm_wide_step(J, rd - 1, acc, s, T, lane, blk == S.block_begin);
      if (lane < 50) acc[lane] = 0;
      if (lane == 0 && !ok) dead_s = 1;
    }
    __syncthreads();
    if (dead_s) return;
  }
  Fr r = fr_zero();
  if (fold) r = step ? lds_get(T.r) : lds_or_global_fr(bmm_slot(J, rd) + kBmmSlotR);
  const BmmTerm o = bmm_term(ea, eb, fold, r, head, w);
  if (fold && pt < 2) {
    store_sol(J.a, ld, i0, o.A);
    store_sol(J.b, ld, i0, o.B);
  }
  acc_add(acc, pt, o.val);
  __syncthreads();
  if (tid < 64) {
    const Fr v = acc_value(acc, min(tid, 2u));
    if (tid < 3) st_rec(bmm_part(J, rd, blk - S.block_begin) + 8 * tid, v);
  }
}

// The transcript step after a wide round, one workgroup per job, where the next
// sweep does not take it.
__global__ void __launch_bounds__(192) bmm_step_kernel(const BmmJob* __restrict__ jobs,
                                                       const BmmSweep* __restrict__ list, uint32_t rd) {
  __shared__ unsigned long long acc[50];
  __shared__ RoundLds T;
  const BmmJob& J = jobs[list[blockIdx.x].job];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  if (bmm_io_status(J) != VL_OK) return;
  if (tid < 50) acc[tid] = 0;
  BmmState s;
  if (tid < 64) bmm_load_state(J, rd, s, T, lane);
  __syncthreads();
  bmm_sum_parts(J, rd, acc);
  __syncthreads();
  if (tid < 64) bmm_wide_step(J, rd, acc, s, T, lane, true);
}

// The messages of a later round rd by wave 0, from sums that are quadratics in
// r_{rd-1}, T.r (acc: nine, as in the matmul rounds), and the scalar's next
// value, side by side: lane 4 j + k < 12 takes value k's j-th coefficient, lane
// 12 + k the scalar times eq1(rho_rd, k).  rho: in LDS.
__device__ __forceinline__ Fr bmm_next(const BmmJob& J, const uint32_t* rho, uint32_t rd, const unsigned long long* acc,
                                       BmmState& s, const RoundLds& T, uint32_t lane) {
  const uint32_t k = lane & 3u;
  const bool scalar = (lane & 15u) >= 12;
  const Fr v0 = acc_point(acc, 3 * min((lane >> 2) & 3u, 2u), k);
  const Fr v1 = fr_row_shl<4>(v0), v2 = fr_row_shl<8>(v0), r = fr_vgpr(lds_get(T.r));
  Fr om = fr_R(), slope = fr_zero(), e, d;
  if (rd <= J.nh) fr_eq1(lds_get(rho + 8 * (rd - 1)), 0, om, slope);
  const Fr m1 = fr_mul(r, fr_pick(scalar, slope, v2));
  const Fr m2 = fr_mul(fr_pick(scalar, s.sc, r), fr_add(m1, fr_pick(scalar, om, fr_sub(fr_sub(v1, v0), v2))));
  s.sc = m2;   // in the scalar's lanes
  s.sce = m2;
  if (rd < J.nh) {
    e = fr_eq1(lds_get(rho + 8 * rd), k, om, d);
    s.sce = fr_mul(m2, e);
  }
  s.sce = fr_row_shl<12>(s.sce);
  return fr_add(v0, m2);
}

// The rounds left after the wide ones, one workgroup per job, then the final
// values.  As in the matmul rounds (kernels.hip), waves 1 .. 6 sum round rd + 1
// while wave 0 hashes round rd, as quadratics in r_rd, once that has at most
// kBmmAhead pairs: it takes up to nine products a pair's value, after the hash
// at most four, and the sums of 256 pairs would outlast the hash.  The first
// round's sums and the larger ones' come before their hash.  The tables come
// from global memory until their first fold (at most kBmmLds entries then) and
// live in LDS after it.  With the pairs' points on one thread and 183 KB of code
// a round took 30 us, with the sums after the hash 16, now 11.4 (the last nine
// rounds and the end of a product 116 to 119 us).
constexpr uint32_t kBmmTailWaves = 8;
__global__ void __launch_bounds__(64 * kBmmTailWaves) bmm_rounds_kernel(const BmmJob* __restrict__ jobs) {
  const BmmJob& J = jobs[blockIdx.x];
  constexpr uint32_t kLen = kBmmLds;                 // entries of the first LDS buffer
  __shared__ alignas(16) uint32_t buf[2][8 * (kLen + kLen / 2)];   // a, b: two buffers each
  __shared__ unsigned long long acc_s[2][90];              // a round's nine sums, by parity
  __shared__ uint32_t rbuf[2][8], fin[2][2][8];            // r_rd by parity; the last pairs
  __shared__ uint32_t rho[32 * 8];
  __shared__ RoundLds T;
  __shared__ uint32_t dead_s;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
  const int32_t st0 = bmm_io_status(J);
  if (st0 != VL_OK) {
    if (tid == 0) *J.status = st0;
    return;
  }
  const uint32_t nh = J.nh, n1 = J.n1, nv = nh + n1, wide = J.wide;
  const uint32_t rd0 = wide ? wide - 1 : 0;   // the first round to hash: the last wide one's sums are in its parts
  const uint64_t ld = 1ull << nv;
  const uint32_t *const ga = J.a, *const gb = J.b;
  int at = -1;   // the tables' place: -1 global, else the LDS buffer of length kLen (0) or kLen / 2 (1)
  auto get = [&](uint32_t k, uint32_t i) {
    if (at >= 0) return ld_rec(buf[k] + (at ? 8 * kLen : 0) + 8 * i);
    return load_sol(k ? gb : ga, ld, i);
  };
  auto put = [&](uint32_t k, uint32_t i, const Fr& x) { st_rec(buf[k] + (at == 0 ? 8 * kLen : 0) + 8 * i, x); };
  BmmState s;
  if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);   // the transcript's wave goes before those it shares its SIMD with
    bmm_load_state(J, rd0, s, T, lane);
  }
  if (tid < 180) acc_s[tid / 90][tid % 90] = 0;
  if (tid < 8 * nh) rho[tid] = J.rho[tid];
  if (tid == 0) dead_s = 0;
  __syncthreads();
  if (wide) bmm_sum_parts(J, rd0, acc_s[rd0 & 1]);
  __syncthreads();
  // rd: the round to hash; tl: the tables' round so far; ready: rd's sums are there
  uint32_t rd = rd0, tl = rd0;
  bool ready = wide > 0;
#pragma unroll 1
  while (rd < nv) {
    const bool poly = ready;   // sums of round nx in the challenge r_{nx-1} of the hash at hand
    const uint32_t nx = ready ? rd + 1 : rd, to = ready ? rd : nx;
    const bool sum_it = nx < nv && (!ready || (1u << (nv - 1 - nx)) <= kBmmAhead);
    const bool last = ready && nx == nv;
    const bool fold = (sum_it || last) && tl < to;
    if (wave == 0) {
      if (ready) {
        unsigned long long* const cur = acc_s[rd & 1];
        const Fr h = rd > rd0 ? bmm_next(J, rho, rd, cur, s, T, lane) : acc_point(cur, 0, lane & 3u);
        const bool ok = bmm_step(J, rd, h, s, T, lane);
#pragma unroll
        for (uint32_t i = lane; i < 90; i += kWave) cur[i] = 0;
        if (lane < 8) rbuf[rd & 1][lane] = T.r[lane];
        if (lane == 0 && !ok) {
          dead_s = 1;
          *J.status = VL_ERR_FALSE_STATEMENT;
        }
      }
    } else if (sum_it) {
      const uint32_t h = 1u << (nv - 1 - nx);   // pairs of round nx
      const uint32_t far = poly ? 4 * h : 2 * h;   // the fold's other entry
      const bool head = nx < nh;
      const Fr r = lds_get(rbuf[~to & 1]);
      // waves 1, 4, .. the values at 0, 2, 5, .. at 1, the others the leading
      // coefficients, a row of 16 lanes 16 pairs
      constexpr uint32_t kPtWaves = (kBmmTailWaves - 1) / 3;
      const uint32_t chunks = (h + 15) / 16, pt = (wave - 1) % 3, first = 4 * ((wave - 1) / 3);
      const bool on = wave <= 3 * kPtWaves && first < chunks;
      Fr sum[3];
      sum[0] = sum[1] = sum[2] = fr_zero();
#pragma unroll 1
      for (uint32_t ch = first + (lane >> 4); on && ch < chunks; ch += 4 * kPtWaves) {
        const uint32_t t = ch * 16 + (lane & 15u), i0 = pt == 1 ? t + h : t;
        if (t >= h) continue;
        Fr e[2][2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
          auto entry = [&](uint32_t off) {
            Fr x = get(k, i0 + off);
            if (pt == 2) x = fr_sub(get(k, t + h + off), x);
            if (fold) {
              Fr y = get(k, i0 + off + far);
              if (pt == 2) y = fr_sub(get(k, t + h + off + far), y);
              x = fr_fold(r, x, y);
              if (pt < 2) put(k, i0 + off, x);
            }
            return x;
          };
          e[k][0] = entry(0);
          e[k][1] = poly ? entry(2 * h) : e[k][0];
        }
        if (head) {
          const Fr w = bmm_weight(J, nh - 1 - nx, t >> n1);
          e[0][0] = fr_mul(e[0][0], w);
          e[0][1] = fr_mul(e[0][1], w);
        }
        const Fr sum1 = sum[1];
        sum[0] = fr_add(sum[0], fr_mul(e[0][0], e[1][0]));
        sum[1] = sum[0];   // (a constant)
        if (poly) {
          sum[1] = fr_add(sum1, fr_mul(e[0][1], e[1][1]));
          sum[2] = fr_add(sum[2], fr_mul(fr_sub(e[0][1], e[0][0]), fr_sub(e[1][1], e[1][0])));
        }
      }
      unsigned long long* const dst = acc_s[nx & 1];
      if (on)
#pragma unroll
        for (uint32_t q = 0; q < 3; ++q) acc_add(dst, 3 * q + pt, sum[q]);
    } else if (fold && tid < kWave + 4) {   // the last pair of each table
      const uint32_t k = (lane >> 1) & 1u, i = lane & 1u;
      lds_put(fin[k][i], fr_fold(lds_get(rbuf[~to & 1]), get(k, i), get(k, i + 2)));
    }
    if (sum_it && fold) at = at == 0 ? 1 : 0;
    if (sum_it) tl = to;
    rd += ready ? 1 : 0;
    ready = !ready || sum_it;
    __syncthreads();   // r, the sums and the folded entries
    if (dead_s) return;
  }
  if (wave != 0) return;
  // lane k < 2: the final value of table k, the last challenge folding the
  // remaining pair
  const uint32_t k = min(lane, 1u);
  const bool two = nv > 0 && tl + 1 < nv;   // the last fold is in fin
  Fr mine = two ? lds_get(fin[k][0]) : get(k, 0);
  if (nv > 0) {
    mine = fr_fold(lds_get(T.r), mine, two ? lds_get(fin[k][1]) : get(k, 1));
  } else {
    // no rounds at all (one head, inner dimension 1): the guard is a b = c
    const Fr a = readlane_fr(mine, 0), b = readlane_fr(mine, 1);
    if (!fr_eq(fr_mul(fr_vgpr(a), b), lds_or_global_fr(J.io + kBmmIoC))) {
      if (lane == 0) *J.status = VL_ERR_FALSE_STATEMENT;
      return;
    }
  }
  const Fr canon = fr_from_mont(mine);
  if (k == 0) mine = canon;
  if (lane < 2) {
    put_canon(J.proof + bmm_round_off(J, nv) + 32 * lane, mine);
    lds_put(T.v + 8 * lane, mine);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (J.digest) {
    tr_absorb_lanes(T, kLblFinal4, kLblFinal1, 2);
    if (lane == 0) tr_put_digest(T, J.digest);
  }
  if (lane == 0) *J.status = VL_OK;
}

hipError_t launch_bmm_start(const BmmJob* jobs, uint32_t n_jobs, hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(bmm_start_kernel, dim3(n_jobs), dim3(256), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_bmm_sweep(const BmmJob* jobs, const BmmSweep* list, uint32_t n_list, uint32_t n_blocks,
                            uint32_t round, bool step, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(bmm_sweep_kernel, dim3(n_blocks), dim3(3 * kBmmSweepPairs), 0, s, jobs, list, n_list, n_blocks,
                     round, step ? 1u : 0u);
  return hipGetLastError();
}

hipError_t launch_bmm_step(const BmmJob* jobs, const BmmSweep* list, uint32_t n_list, uint32_t round,
                           hipStream_t s) {
  if (n_list == 0) return hipSuccess;
  hipLaunchKernelGGL(bmm_step_kernel, dim3(n_list), dim3(192), 0, s, jobs, list, round);
  return hipGetLastError();
}

hipError_t launch_bmm_rounds(const BmmJob* jobs, uint32_t n_jobs, hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(bmm_rounds_kernel, dim3(n_jobs), dim3(64 * kBmmTailWaves), 0, s, jobs);
  return hipGetLastError();
}

}  // namespace vl
