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
__device__ __forceinline__ void bmm_load_state(const BmmJob& J, uint32_t rd, BmmState& s, RoundLds& T, uint32_t lane) {
  s.sc = fr_vgpr(lds_or_global_fr(J.io + kBmmIoScale));
  if (lane < 8) {
    T.st[lane] = J.io[kBmmIoState + lane];
    T.r[lane] = J.io[kBmmIoR + lane];
  }
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
// Round rd by wave 0: acc holds the limb sums of h(0), h(1), h2.  Lane k forms
// g(k) and writes it; the values are absorbed and r squeezed into T.  Round 0
// checks the guard g(0) + g(1) = c (false in every lane if it fails).
__device__ __forceinline__ bool bmm_step(const BmmJob& J, uint32_t rd, const unsigned long long* acc, const BmmState& s,
                                         RoundLds& T, uint32_t lane) {
  const uint32_t K = rd < J.nh ? 4u : 3u;
  const Fr g = fr_mul(acc_point(acc, 0, lane & 3u), s.sce);
  if (rd == 0 && !fr_eq(fr_add(readlane_fr(g, 0), readlane_fr(g, 1)), lds_or_global_fr(J.io + kBmmIoC))) return false;
  if (lane < K) {
    put_canon(J.proof + bmm_round_off(J, rd) + 32 * lane, g);
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
  if (lane < 8) J.io[kBmmIoState + lane] = T.st[lane];
  if (lane == 0) {
    const Fr one = fr_R();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      J.io[kBmmIoC + i] = c[0].w[i];
      J.io[kBmmIoScale + i] = one.w[i];
    }
    J.io[0] = (uint32_t)VL_OK;
  }
}

// One wide round: every job of the round's list, kBmmSweepPairs pairs per
// block, the waves in three groups by point.  Round rd > 0 first folds the
// tables by the previous challenge, in place: every wave has read the block's
// entries before any wave writes.  Each block writes its three sums.  Few
// pairs (at most 32,768 in the 7B attention layer): bound by a thread's chain
// and the launch, which a thread per pair and four points made longer (18 to
// 35 us a launch, now 12 to 20).
__global__ void __launch_bounds__(3 * kBmmSweepPairs) bmm_sweep_kernel(const BmmJob* __restrict__ jobs,
                                                                       const BmmSweep* __restrict__ list,
                                                                       uint32_t n_list, uint32_t n_blocks,
                                                                       uint32_t rd) {
  __shared__ unsigned long long acc[50];   // three values; acc_point reads two past its base
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
  const uint32_t tid = threadIdx.x, pt = tid / kBmmSweepPairs;
  const uint32_t nv = J.nh + J.n1;
  const uint64_t ld = 1ull << nv, h = 1ull << (nv - 1 - rd);   // at least kBmmWidePairs, a multiple of the block's
  const uint64_t t = (uint64_t)(blk - S.block_begin) * kBmmSweepPairs + tid % kBmmSweepPairs;
  const uint64_t i0 = pt == 1 ? t + h : t;
  const bool fold = rd > 0, head = rd < J.nh;
  const Fr r = lds_or_global_fr(J.io + kBmmIoR);
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
  __syncthreads();   // everything read (and acc zeroed)
  const BmmTerm o = bmm_term(ea, eb, fold, r, head, w);
  if (fold && pt < 2) {
    store_sol(J.a, ld, i0, o.A);
    store_sol(J.b, ld, i0, o.B);
  }
  acc_add(acc, pt, o.val);
  __syncthreads();
  if (tid < 64) {
    const Fr v = acc_point(acc, min(tid, 2u), 0);
    if (tid < 3) st_rec(J.part + (uint64_t)(blk - S.block_begin) * 32 + 8 * tid, v);
  }
}

// The transcript step after a wide round, one workgroup per job: wave k adds
// the blocks' value k, wave 0 runs the round's step.
__global__ void __launch_bounds__(192) bmm_step_kernel(const BmmJob* __restrict__ jobs,
                                                       const BmmSweep* __restrict__ list, uint32_t rd) {
  __shared__ unsigned long long acc[50];
  __shared__ RoundLds T;
  const BmmJob& J = jobs[list[blockIdx.x].job];
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
  if (bmm_io_status(J) != VL_OK) return;
  const uint64_t h = 1ull << (J.nh + J.n1 - 1 - rd);
  const uint32_t nblocks = (uint32_t)((h + kBmmSweepPairs - 1) / kBmmSweepPairs);
  if (tid < 50) acc[tid] = 0;
  BmmState s;
  if (wave == 0) bmm_load_state(J, rd, s, T, lane);
  Fr v = fr_zero();
  for (uint32_t i = lane; i < nblocks; i += 64) v = fr_add(v, ld_rec(J.part + 32ull * i + 8 * wave));
  __syncthreads();
  acc_add(acc, wave, v);
  __syncthreads();
  if (wave != 0) return;
  if (!bmm_step(J, rd, acc, s, T, lane)) {
    if (lane == 0) {
      J.io[0] = (uint32_t)VL_ERR_FALSE_STATEMENT;
      *J.status = VL_ERR_FALSE_STATEMENT;
    }
    return;
  }
  if (lane < 8) {
    J.io[kBmmIoState + lane] = T.st[lane];
    J.io[kBmmIoR + lane] = T.r[lane];
  }
  bmm_advance(J, rd, s, T, lane);
  if (lane == 0)
#pragma unroll
    for (int i = 0; i < 8; ++i) J.io[kBmmIoScale + i] = s.sc.w[i];
}

// The rounds left after the wide ones, one workgroup per job, then the final
// values.  The tables come from global memory until their first fold (at most
// 2 kBmmWidePairs entries then) and live in LDS after it, folded from one
// buffer into the other.  The rows of 16 lanes of waves 1 .. 11 take the terms
// of 16 pairs at a time; wave 0 runs the transcript.  With the pairs' points
// on one thread and 183 KB of code a round took 30 us, now about 19.
constexpr uint32_t kBmmTailWaves = 12;
__global__ void __launch_bounds__(64 * kBmmTailWaves) bmm_rounds_kernel(const BmmJob* __restrict__ jobs) {
  const BmmJob& J = jobs[blockIdx.x];
  constexpr uint32_t kLen = kBmmWidePairs;                 // entries of the first LDS buffer
  __shared__ uint32_t buf[2][8 * (kLen + kLen / 2)];       // a, b: two buffers each
  __shared__ unsigned long long acc[50];
  __shared__ RoundLds T;
  __shared__ uint32_t dead_s;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
  const int32_t st0 = bmm_io_status(J);
  if (st0 != VL_OK) {
    if (tid == 0) *J.status = st0;
    return;
  }
  const uint32_t nh = J.nh, n1 = J.n1, nv = nh + n1, wide = J.wide;
  const uint64_t ld = 1ull << nv;
  const uint32_t *const ga = J.a, *const gb = J.b;
  bool pending = wide > 0;
  int at = -1;   // the tables' place: -1 global, else the LDS buffer of length kLen (0) or kLen / 2 (1)
  auto get = [&](uint32_t k, uint32_t i) {
    if (at >= 0) return load_sol(buf[k] + (at ? 8 * kLen : 0), at ? kLen / 2 : kLen, i);
    return load_sol(k ? gb : ga, ld, i);
  };
  auto put = [&](uint32_t k, uint32_t i, const Fr& x) {
    store_sol(buf[k] + (at == 0 ? 8 * kLen : 0), at == 0 ? kLen / 2 : kLen, i, x);
  };
  BmmState s;
  if (wave == 0) bmm_load_state(J, wide, s, T, lane);
  if (tid < 50) acc[tid] = 0;
  if (tid == 0) dead_s = 0;
  __syncthreads();
#pragma unroll 1
  for (uint32_t rd = wide; rd < nv; ++rd) {
    const uint32_t h = 1u << (nv - 1 - rd);
    const bool head = rd < nh;
    if (wave == 0) {
      if (rd > wide) bmm_advance(J, rd - 1, s, T, lane);
    } else {
      const uint32_t chunks = (h + 15) / 16, units = 3 * chunks;   // 16 pairs at one point
      const Fr r = lds_get(T.r);
#pragma unroll 1
      for (uint32_t q0 = 4 * (wave - 1); q0 < units; q0 += 4 * (kBmmTailWaves - 1)) {
        const uint32_t q = q0 + (lane >> 4), pt = q / chunks, t = (q % chunks) * 16 + (lane & 15u);
        const bool take = q < units;
        BmmTerm o;
        o.A = o.B = o.val = fr_zero();
        if (take && t < h) {
          const uint32_t i0 = pt == 1 ? t + h : t, d = pt == 2 ? h : 0;
          Fr ea[2], eb[2];
          auto entry = [&](uint32_t tab, uint32_t off) {
            Fr x = get(tab, i0 + d + off);
            if (pt == 2) x = fr_sub(x, get(tab, t + off));
            return x;
          };
          ea[0] = entry(0, 0);
          eb[0] = entry(1, 0);
          if (pending) {
            ea[1] = entry(0, 2 * h);
            eb[1] = entry(1, 2 * h);
          }
          Fr w = fr_zero();
          if (head) w = bmm_weight(J, nh - 1 - rd, t >> n1);
          o = bmm_term(ea, eb, pending, r, head, w);
          if (pending && pt < 2) {
            put(0, i0, o.A);
            put(1, i0, o.B);
          }
        }
        acc_add(acc, pt, o.val, take);
      }
    }
    if (pending) at = at == 0 ? 1 : 0;
    __syncthreads();   // the sums, and the folded entries
    if (wave == 0) {
      const bool ok = bmm_step(J, rd, acc, s, T, lane);
      if (lane < 30) acc[lane] = 0;
      if (lane == 0 && !ok) {
        dead_s = 1;
        *J.status = VL_ERR_FALSE_STATEMENT;
      }
    }
    __syncthreads();   // r and the zeroed sums
    if (dead_s) return;
    pending = true;
  }
  const Fr r = lds_get(T.r);
  if (wave != 0) return;
  // lane k < 2: the final value of table k, the last challenge folding the
  // remaining pair
  const uint32_t k = min(lane, 1u);
  Fr mine = get(k, 0);
  if (pending) {
    mine = fr_fold(r, mine, get(k, 1));
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
                            uint32_t round, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(bmm_sweep_kernel, dim3(n_blocks), dim3(3 * kBmmSweepPairs), 0, s, jobs, list, n_list, n_blocks,
                     round);
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
