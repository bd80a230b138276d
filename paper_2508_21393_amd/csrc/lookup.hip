// Device kernels of the lookup argument (vl_lookup_prove).
//
// Protocol 1 proves that every entry s_i of a secret tensor lies in a public
// table T through the identity of eq. (rational-function): at a random beta,
// sum_i 1/(beta + s_i) = sum_j m_j/(beta + t_j), with m_j the multiplicity of
// t_j.  Eq. (lookup-sumcheck) turns this and the two inverse relations into
// one sum over the entries x = (x_H, x_L) of
//     alpha A eq(u, .) (S + beta) + A + (N/D) alpha^2 B eq(u_L, .) (T + beta)
//     - (N/D) B m,
// whose value is alpha + alpha^2.  Because the table is small (N rows) and
// every entry is one of its rows, A_i = B_{j(i)}: the N inverses are the only
// ones computed (a batch inversion per chunk of rows), and A is gathered.
//
//   lookup_tables_kernel T + beta and B = 1 / (T + beta), one record per row;
//                        eq tables of u's suffixes
//   lookup_hist_kernel   multiplicities and the membership check of every entry
//   lookup_mult_kernel   m in the field, partial sums of B m
//   lookup_start_kernel  the constant K of the high rounds, the status
//   lookup_sweep/step    the first rounds across the GPU, then a one-block
//                        transcript step
//   lookup_rounds_kernel the remaining rounds in one workgroup, and the
//                        final values A(r), S(r), B(r_L), T(r_L), m(r_L)
// Every table is in Montgomery form; round values are converted to
// canonical form for the proof.  m is kept as M' = c2 m (never sent;
// m(r_L) is recovered as 2^nH M'(r_L)).
//
// A round's polynomial.  With challenges r_0 .. r_{rd-1} bound, eq(u, .) is
// eq1(u_rd, X) eq(u_{rd+1} .., t) prod_k eq1(u_k, r_k), eq1(u, X) =
// u X + (1 - u)(1 - X): the last factor is one running scalar and the middle
// one a table of u's suffix that no challenge changes.  So no eq table is
// folded, and the products are summed as the quadratic
//     h(X) = sum_t eq(suffix, t) A(X, t) (S + beta)(X, t)
// through h(0), h(1) and its leading coefficient h2 (three products and
// three weights a pair instead of four points of a degree-3 product of three
// folded tables); the linear A and the quadratic B M' go into
// q(X) = sum_t A(X, t) - B(X, t) M'(X, t).  Then
//     g(X) = scale eq1(u_rd, X) h(X) + q(X) (+ the high rounds' constant).
// While low bits are bound the rows' terms c1 B eq(u_L, .) (T + beta) add a
// second such product, with the same weights and its own running scalar.
#include <type_traits>

#include "device.hpp"
#include "modinv.hpp"
#include "rounds_dev.hpp"
#include "sha256.hpp"

namespace vl {

namespace {

__device__ __forceinline__ int64_t lk_entry(const void* p, int dt, uint64_t i) {
  return dt == VL_I16 ? (int64_t)reinterpret_cast<const int16_t*>(p)[i]
                      : (int64_t)reinterpret_cast<const int32_t*>(p)[i];
}

// canonical field element of a signed integer
__device__ __forceinline__ Fr fr_of_int(int64_t v) {
  const uint64_t mag = v < 0 ? (uint64_t)0 - (uint64_t)v : (uint64_t)v;
  Fr r = fr_zero();
  r.w[0] = (uint32_t)mag;
  r.w[1] = (uint32_t)(mag >> 32);
  return v < 0 ? fr_neg(r) : r;
}

// Montgomery form of x + gamma y + beta (gamma, beta Montgomery)
__device__ __forceinline__ Fr compress_mont(int64_t x, int64_t y, bool two, const Fr& gamma, const Fr& beta) {
  Fr v = fr_of_int(x);
  if (two) v = fr_add(v, fr_mul(gamma, fr_of_int(y)));   // Montgomery x canonical: canonical
  return fr_add(fr_mul(v, fr_R2()), beta);
}

struct FrMod30 {
  static constexpr int L = 9;
  static constexpr int kBatches = 25;                    // (49 * 256 + 57) / 17 = 741 divsteps
  static constexpr uint32_t inv30 = 1u;                  // p = 1 mod 2^30
  __device__ __forceinline__ static uint32_t limb(int i) {
    switch (i) {
      case 0: return 0x00000001u; case 1: return 0x3ffffffcu; case 2: return 0x3fe5bfefu;
      case 3: return 0x2f6900bfu; case 4: return 0x21d80553u; case 5: return 0x27602026u;
      case 6: return 0x17d48333u; case 7: return 0x29d4ca67u; default: return 0x000073edu;
    }
  }
};
// x^-1, Montgomery in and out (0 for 0): the inverse of the integer x R is
// x^-1 / R, and two products by R^2 give x^-1 R
__device__ Fr fr_inv_mont(const Fr& x) {
  int32_t l[9], d[9];
  words_to_30<8, 9>(x.w, l);
  modinv30<FrMod30>(l, d);
  add_2m30<FrMod30>(d);            // below 4 p, which needs 257 bits
  uint32_t w[9];
  limbs30_to_words<9, 9>(d, w);
  Fr r;
  uint32_t borrow = 0, top = w[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) r.w[j] = w[j];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    Fr t;
    borrow = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) t.w[j] = sbb32(r.w[j], p_limb(j), borrow, borrow);
    const bool ge = top >= borrow;
#pragma unroll
    for (int j = 0; j < 8; ++j) r.w[j] = ge ? t.w[j] : r.w[j];
    top = ge ? top - borrow : top;
  }
  return fr_mul(fr_mul(r, fr_R2()), fr_R2());
}

__device__ __forceinline__ Fr lk_fr(const uint32_t (&w)[8]) {
  Fr r;
#pragma unroll
  for (int j = 0; j < 8; ++j) r.w[j] = w[j];
  return r;
}

__device__ __forceinline__ int32_t lk_io_status(const LookupJob& J) {
  return *reinterpret_cast<volatile const int32_t*>(J.io);
}

// eq of u's last m variables at t (m <= lk_nlo(n))
__device__ __forceinline__ Fr lk_weight(const LookupJob& J, uint32_t m, uint64_t t) {
  return load_sol(J.W + 8 * ((1ull << m) - 1), 1ull << m, t);
}

// the table row of entry i (padding entries are row 0; rows out of the
// table, whose entries have set the flag, are clamped)
__device__ __forceinline__ const uint32_t* lk_row(const LookupJob& J, uint64_t i) {
  int64_t j = i < J.D ? lk_entry(J.x, J.dtype, i) - J.t0 : 0;
  const int64_t N = 1ll << J.nL;
  j = j < 0 ? 0 : (j >= N ? N - 1 : j);
  return J.rec + 16 * (uint64_t)j;
}

// v += {h(0), h(1), h2} of one product of lines, weighted: (w x0) y0, (w x1) y1,
// (w x1 - w x0)(y1 - y0), five products
__device__ __forceinline__ void lk_weighted(const Fr& w, const Fr& x0, const Fr& x1, const Fr& y0, const Fr& y1,
                                            Fr (&v)[5]) {
  const Fr w0 = fr_mul(w, x0), w1 = fr_mul(w, x1);
  v[0] = fr_add(v[0], fr_mul(w0, y0));
  v[1] = fr_add(v[1], fr_mul(w1, y1));
  v[2] = fr_add(v[2], fr_mul(fr_sub(w1, w0), fr_sub(y1, y0)));
}

// One of the nine terms of a pair in a low round: product `role` (0: A Sb,
// 1: B T, 2: B M') at point pt (0, 1, or 2 for the leading coefficient).  A
// wave takes one term of 64 pairs, so that every wave runs the same four
// products (two folds, the product, the weight) and sums one value.  ex, ey:
// the tables' entries {e, e'} whose fold e + r (e' - e) is the line's value at
// the point (for pt 2 the differences of the two points').
struct LkTerm {
  Fr X, Y, val;
};
__device__ __forceinline__ LkTerm lk_term(const Fr (&ex)[2], const Fr (&ey)[2], bool fold, const Fr& r, const Fr& w) {
  LkTerm o;
  o.X = ex[0];
  o.Y = ey[0];
  if (fold) {
    o.X = fr_fold(r, ex[0], ex[1]);
    o.Y = fr_fold(r, ey[0], ey[1]);
  }
  o.val = fr_mul(fr_mul(o.X, o.Y), w);
  return o;
}
// the weight of role 2, whose product enters q negated
__device__ __forceinline__ Fr fr_minus_one() { return fr_neg(fr_R()); }

// State of the rounds held by wave 0: lane 4 g + k (g < 3, k < 4) has group
// g's running scalar, g = 0: alpha prod eq1(u_j, r_j) over the rounds so far,
// 1: c1 prod over the low rounds, 2: one; and e = eq1(u_rd, k) times it.  The
// scalars are canonical, so that they take the values, which are in Montgomery
// form, to canonical ones.
struct LkState {
  Fr sc, sce;
  Fr kc;       // the next high round's constant 2^(nH - rd - 1) K
};
__device__ __forceinline__ void lk_set_sce(const LookupJob& J, uint32_t rd, LkState& s, uint32_t lane) {
  Fr om, slope;
  const Fr e = fr_eq1(fr_vgpr(lds_or_global_fr(J.u + 8 * rd)), lane & 3u, om, slope), m = fr_mul(s.sc, e);
#pragma unroll
  for (int j = 0; j < 8; ++j) s.sce.w[j] = lane < 8 ? m.w[j] : s.sc.w[j];
}
// the state round rd starts from, left in io by round rd - 1 (or the start) in
// the slot of its parity
__device__ __forceinline__ uint32_t* lk_slot(const LookupJob& J, uint32_t rd) { return J.io + kLkIoSlot + kLkSlotWords * (~rd & 1u); }
__device__ __forceinline__ void lk_load_state(const LookupJob& J, uint32_t rd, LkState& s, RoundLds& T, uint32_t lane) {
  const uint32_t g = lane >> 2, *io = lk_slot(J, rd);
  s.sc = lds_or_global_fr(io + kLkSlotScale + 8 * min(g, 2u));
  s.kc = lds_or_global_fr(io + kLkSlotK);
  if (lane < 8) {
    T.st[lane] = io[lane];
    T.r[lane] = io[kLkSlotR + lane];
  }
  if (rd < J.nH + J.nL) lk_set_sce(J, rd, s, lane);
}

// Round rd by wave 0 (all lanes): acc holds the limb sums of the nine values
// {A Sb: h(0), h(1), h2; B T: the same; q(0), q(1), q2}.  Lanes 0 .. 11 form
// the three quadratics at 0 .. 3 and scale them, lanes 0 .. 3 add them to g(k)
// and write the canonical values; these are absorbed and r squeezed into T.
// Round 0 checks the guard g(0) + g(1) = alpha + alpha^2 (false in every lane
// if it fails).
__device__ __forceinline__ bool lk_step(const LookupJob& J, uint32_t rd, const unsigned long long* acc, LkState& s,
                                        RoundLds& T, uint32_t lane, bool write = true) {
  const uint32_t g = min(lane >> 2, 2u), k = lane & 3u;
  Fr v = acc_point(acc, 3 * g, k);
  if (rd == 0 && J.gather && g == 0) {   // A Sb = 1 at every entry, and the weights add up to 1
    // h(0) = h(1) = 1 were not summed: the quadratic has 1, 1, 2 - 1 and 3 - 2 of them
    v = fr_add(v, fr_R());
  }
  v = fr_mul(v, s.sce);
  v = fr_add(v, fr_add(fr_row_shl<4>(v), fr_row_shl<8>(v)));   // lanes 0 .. 3
  if (rd < J.nH) v = fr_add(v, s.kc);
  if (rd == 0 && !fr_eq(fr_add(readlane_fr(v, 0), readlane_fr(v, 1)), fr_from_mont(lk_fr(J.claim)))) return false;
  if (lane < 4) {
    if (write) put_canon(J.proof + 128ull * rd + 32 * lane, v);
    lds_put(T.v + 8 * lane, v);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  tr_round(T, 4);
  return true;
}
// the running scalars and the constant for round rd + 1, after r is known
__device__ __forceinline__ void lk_advance(const LookupJob& J, uint32_t rd, LkState& s, const RoundLds& T, uint32_t lane) {
  Fr om, slope;
  fr_eq1(fr_vgpr(lds_or_global_fr(J.u + 8 * rd)), 0, om, slope);
  const Fr f = fr_add(om, fr_mul(slope, fr_vgpr(lds_get(T.r)))), m = fr_mul(s.sc, f);
  const bool use = lane < 4 || (lane < 8 && rd >= J.nH);
#pragma unroll
  for (int j = 0; j < 8; ++j) s.sc.w[j] = use ? m.w[j] : s.sc.w[j];
  s.kc = fr_half(s.kc);
  if (rd + 1 < J.nH + J.nL) lk_set_sce(J, rd + 1, s, lane);
}

// the block's sums of v = {h(0), h(1), h2, q(0), q(1)} of a high round to the
// nine values of out (72 words); the h sums times *hi (the weight the block's
// pairs share), if given
__device__ __forceinline__ void lk_block_out(const Fr (&v)[5], const Fr* hi, uint32_t* out) {
  __shared__ uint32_t red[5 * 10 * 4];
  const Fr t = block_sum_lanes<5, 4>(v, red);
  if (threadIdx.x < 64) {
    const uint32_t k = threadIdx.x;
    Fr o = t;
    if (hi) {
      const Fr m = fr_mul(t, *hi);
#pragma unroll
      for (int j = 0; j < 8; ++j) o.w[j] = k < 3 ? m.w[j] : t.w[j];
    }
    if (k < 5) st_rec(out + 8 * (k < 3 ? k : k + 3), o);
    if (k >= 5 && k < 9) st_rec(out + 8 * (k == 8 ? 8 : k - 2), fr_zero());
  }
}

template <typename Get>
__device__ __forceinline__ uint32_t lk_find(Get begin_of, uint32_t n, uint32_t blk) {
  uint32_t lo = 0, hi = n;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (begin_of(mid) <= blk) lo = mid; else hi = mid;
  }
  return lo;
}

}  // namespace

// Multiplicities and membership.  An entry outside the table (or, with two
// columns, whose second value differs from the table's) sets the job's flag.
// Tables of up to 2^kLookupLdsVars rows: a block of 1024 threads counts
// J.hist_chunk entries (below 2^16) in 16-bit counters in LDS and writes them
// to its slice of J.hist; the multiplicity kernel adds the slices.  (One global
// atomic per entry: 8.4 M activations took 400 us, this 61 beside the tables.)
// Larger tables: 32-bit global atomics on J.hist, zeroed before.
__global__ void __launch_bounds__(1024) lookup_hist_kernel(const LookupJob* __restrict__ jobs, uint32_t n_jobs,
                                                           uint32_t n_blocks) {
  extern __shared__ uint32_t cnt[];
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  const LookupJob& J = jobs[lk_find([&](uint32_t k) { return jobs[k].hist_begin; }, n_jobs, blk)];
  const uint32_t part = blk - J.hist_begin;
  const uint64_t N = 1ull << J.nL;
  const bool lds = J.nL <= kLookupLdsVars;
  const uint32_t words = (uint32_t)((N + 1) / 2);
  if (lds) {
    for (uint32_t k = threadIdx.x; k < words; k += 1024) cnt[k] = 0;
    __syncthreads();
  }
  const uint64_t i0 = (uint64_t)part * J.hist_chunk, i1 = min(i0 + J.hist_chunk, J.D);
  bool bad = false;
  for (uint64_t i = i0 + threadIdx.x; i < i1; i += 1024) {
    const int64_t j = lk_entry(J.x, J.dtype, i) - J.t0;
    bool ok = j >= 0 && j < (int64_t)N;
    if (ok && J.y) ok = lk_entry(J.y, J.dtype_y, i) == (int64_t)J.tb[j];
    if (!ok) bad = true;
    else if (lds) atomicAdd(cnt + (j >> 1), 1u << (16 * (j & 1)));
    else atomicAdd(J.hist + j, 1u);
  }
  if (bad) *reinterpret_cast<volatile int32_t*>(J.flag) = 1;
  if (lds) {
    __syncthreads();
    uint32_t* out = J.hist + (uint64_t)part * words;
    for (uint32_t k = threadIdx.x; k < words; k += 1024) out[k] = cnt[k];
  }
}

// The tables that need nothing but the descriptors, in one launch.
// Rows: the record {B_j, T_j + beta} of row j, T_j = t0 + j + gamma tb_j and
// B_j its inverse by division steps (modinv.hpp).  Each thread takes
// J.inv_chunk rows with one inversion (prefix products, back-substitution):
// one row while that keeps the SIMDs in their first wave.  A zero T_j + beta
// (beta at a pole, probability N / p) sets the flag.
__device__ __forceinline__ void lk_inv_rows(const LookupJob& J, uint32_t blk) {
  const uint64_t N = 1ull << J.nL;
  const uint64_t ch = (uint64_t)blk * 256 + threadIdx.x;
  const uint64_t j0 = ch * J.inv_chunk, j1 = min(j0 + J.inv_chunk, N);
  if (j0 >= N) return;
  const Fr gamma = lk_fr(J.gamma), beta = lk_fr(J.beta);
  Fr acc = fr_R();
  for (uint64_t j = j0; j < j1; ++j) {
    const Fr tb = compress_mont(J.t0 + (int64_t)j, J.tb ? J.tb[j] : 0, J.tb != nullptr, gamma, beta);
    if (fr_is_zero(tb)) *reinterpret_cast<volatile int32_t*>(J.flag) = 1;
    st_rec(J.rec + 16 * j + 8, tb);
    st_rec(J.rec + 16 * j, acc);      // prefix product, replaced below
    acc = fr_mul(acc, tb);
  }
  Fr inv = fr_inv_mont(acc);
  for (uint64_t jj = j1; jj > j0; --jj) {
    const uint64_t j = jj - 1;
    const Fr b = fr_mul(inv, ld_rec(J.rec + 16 * j));
    inv = fr_mul(inv, ld_rec(J.rec + 16 * j + 8));
    st_rec(J.rec + 16 * j, b);
  }
}

// eq tables of u's suffixes: J.W holds the tables of the last m variables for
// m = 0 .. nlo at 8 (2^m - 1) words, J.EH those of the last m of the first
// n - nlo variables for m = 0 .. n - nlo - 1 in the same layout (the suffix of
// a round with more than nlo variables left is the product of the two).  One
// thread per entry.
__device__ __forceinline__ void lk_eq_entries(const LookupJob& J, uint32_t blk) {
  const uint32_t n = J.nH + J.nL, nlo = lk_nlo(n);
  uint64_t e = (uint64_t)blk * 256 + threadIdx.x;
  uint32_t* base = J.W;
  uint32_t end = n;                       // the suffix ends before variable `end`
  if (e >= (2ull << nlo) - 1) {
    e -= (2ull << nlo) - 1;
    base = J.EH;
    end = n - nlo;
    if (e >= (1ull << end) - 1) return;   // m < n - nlo
  }
  const uint32_t m = 63 - __clzll((unsigned long long)(e + 1));
  const uint64_t t = e + 1 - (1ull << m);
  Fr v = fr_R();
  for (uint32_t k = 0; k < m; ++k) {
    const Fr u = lds_or_global_fr(J.u + 8 * (end - m + k));
    const Fr f = ((t >> (m - 1 - k)) & 1u) ? u : fr_sub(fr_R(), u);
    v = k == 0 ? f : fr_mul(v, f);
  }
  store_sol(base + 8 * ((1ull << m) - 1), 1ull << m, t, v);
}

__global__ void __launch_bounds__(256) lookup_tables_kernel(const LookupJob* __restrict__ jobs, uint32_t n_jobs,
                                                            uint32_t n_blocks) {
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  const LookupJob& J = jobs[lk_find([&](uint32_t k) { return jobs[k].tab_begin; }, n_jobs, blk)];
  const uint32_t b = blk - J.tab_begin;
  if (b < J.inv_blocks) lk_inv_rows(J, b);
  else lk_eq_entries(J, b - J.inv_blocks);
}

// M'_j = c2 m_j, the counts added over the blocks of the count kernel (the
// padding entries count on row 0), and per block the sum of B_j M'_j
__global__ void __launch_bounds__(256) lookup_mult_kernel(const LookupJob* __restrict__ jobs, uint32_t n_jobs,
                                                          uint32_t n_blocks) {
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  const LookupJob& J = jobs[lk_find([&](uint32_t k) { return jobs[k].mult_begin; }, n_jobs, blk)];
  const uint64_t N = 1ull << J.nL, Dp = 1ull << (J.nH + J.nL);
  const uint64_t j = (uint64_t)(blk - J.mult_begin) * 256 + threadIdx.x;
  Fr g[1];
  g[0] = fr_zero();
  if (j < N) {
    uint32_t c = 0;
    if (J.nL <= kLookupLdsVars) {
      const uint64_t words = (N + 1) / 2;
      const uint32_t sh = 16 * (j & 1);
      for (uint32_t b = 0; b < J.hist_blocks; ++b) c += (J.hist[b * words + (j >> 1)] >> sh) & 0xffffu;
    } else {
      c = J.hist[j];
    }
    if (j == 0) c += (uint32_t)(Dp - J.D);
    Fr m = fr_zero();
    m.w[0] = c;
    m = fr_mul(fr_mul(lk_fr(J.c2), fr_R2()), m);   // c2 m in Montgomery form (c2 R^2 times the count)
    store_sol(J.M, N, j, m);
    g[0] = fr_mul(ld_rec(J.rec + 16 * j), m);
  }
  __shared__ uint32_t red[10 * 4];
  const Fr t = block_sum_lanes<1, 4>(g, red);
  if (threadIdx.x == 0) st_rec(J.kpart + 8ull * (blk - J.mult_begin), t);
}

// Entries materialised (jobs without the gathering sweeps): Sb_i = T_j + beta
// and A_i = B_j of the entry's row.  One thread per padded entry.
__global__ void __launch_bounds__(256) lookup_prep_kernel(const LookupJob* __restrict__ jobs, uint32_t n_jobs,
                                                          uint32_t n_blocks) {
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  const LookupJob& J = jobs[lk_find([&](uint32_t k) { return jobs[k].prep_begin; }, n_jobs, blk)];
  if (J.gather) return;
  const uint64_t i = (uint64_t)(blk - J.prep_begin) * 256 + threadIdx.x;
  const uint64_t Dp = 1ull << (J.nH + J.nL);
  if (i >= Dp) return;
  const uint32_t* rec = lk_row(J, i);
  store_sol(J.A, Dp, i, ld_rec(rec));
  store_sol(J.S, Dp, i, ld_rec(rec + 8));
}

// Status, the first round's constant 2^(nH - 1) K of the high rounds with
// K = c1 - sum_j B_j M'_j (the table rows' terms summed over x_L;
// sum_j eq(u_L, j) = 1 and B_j (T_j + beta) = 1), and the rounds' state.
__global__ void __launch_bounds__(64) lookup_start_kernel(const LookupJob* __restrict__ jobs) {
  const LookupJob& J = jobs[blockIdx.x];
  const uint32_t lane = threadIdx.x;
  if (*reinterpret_cast<volatile const int32_t*>(J.flag)) {
    if (lane == 0) {
      J.io[0] = (uint32_t)VL_ERR_FALSE_STATEMENT;
      *J.status = VL_ERR_FALSE_STATEMENT;
    }
    return;
  }
  Fr s[1];
  s[0] = fr_zero();
  for (uint32_t i = lane; i < J.nkparts; i += kWave) s[0] = fr_add(s[0], lds_or_global_fr(J.kpart + 8ull * i));
  wave_sum<1>(s, kWave);
  if (lane == 0) {
    Fr K = fr_sub(lk_fr(J.c1), s[0]);
    for (uint32_t i = 0; i + 1 < J.nH; ++i) K = fr_double(K);
    const Fr alpha = fr_from_mont(lk_fr(J.alpha)), c1 = fr_from_mont(lk_fr(J.c1)), one = fr_one_raw();
    K = fr_from_mont(K);
    uint32_t* io = lk_slot(J, 0);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      io[kLkSlotK + i] = K.w[i];
      io[i] = J.st[i];
      io[kLkSlotScale + i] = alpha.w[i];
      io[kLkSlotScale + 8 + i] = c1.w[i];
      io[kLkSlotScale + 16 + i] = one.w[i];
    }
    J.io[0] = (uint32_t)VL_OK;
  }
}

// One wide round in which a high index bit is bound: only A and Sb depend on
// it.  A block takes lk_span(h) pairs (one common eq factor of the high
// variables), 256 at a time.  Bound by the field products, about 300
// instructions each:
//   kFirst    round 0 of a gathering job: A and Sb are looked up in the row
//             records (64 bytes each, in L2) instead of stored tables, and
//             h(0) = h(1) = 1 because A Sb = 1 at every entry: 2 products a pair
//   kSecond   round 1: the four entries looked up, folded by r_0 and stored
//   kFold     later rounds: folded in place (each thread reads and writes
//             only its own entries): 9 products a pair (262 and 149 us for the
//             largest kSecond and kFold sweeps of 2^23 entries with 10, now 245 and
//             143)
//   kPlain    round 0 of stored tables
enum { kFirst = 0, kSecond = 1, kFold = 2, kPlain = 3 };
template <int MODE>
__global__ void __launch_bounds__(256) lookup_sweep_kernel(const LookupJob* __restrict__ jobs,
                                                           const LookupSweep* __restrict__ list, uint32_t n_list,
                                                           uint32_t n_blocks, uint32_t rd) {
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  const LookupSweep& L = list[lk_find([&](uint32_t k) { return list[k].block_begin; }, n_list, blk)];
  const LookupJob& J = jobs[L.job];
  if (MODE != kFirst && lk_io_status(J) != VL_OK) return;   // the first sweep may run beside the start kernel
  const uint32_t n = J.nH + J.nL, m = n - 1 - rd, nlo = lk_nlo(n);
  const uint64_t h = 1ull << m, span = lk_span(h);
  const uint64_t base = (uint64_t)(blk - L.block_begin) * span;
  const uint64_t ld = J.gather ? 1ull << (n - 1) : 1ull << n;
  Fr v[5];
#pragma unroll
  for (int k = 0; k < 5; ++k) v[k] = fr_zero();
  const Fr r = MODE == kSecond || MODE == kFold ? lds_or_global_fr(lk_slot(J, rd) + kLkSlotR) : fr_zero();
#pragma unroll 1
  for (uint64_t t = base + threadIdx.x; t < h && t < base + span; t += 256) {
    const Fr w = m > nlo ? lk_weight(J, nlo, t & ((1ull << nlo) - 1)) : lk_weight(J, m, t);
    if (MODE == kFirst) {
      const uint32_t *p0 = lk_row(J, t), *p1 = lk_row(J, t + h);
      const Fr a0 = ld_rec(p0), a1 = ld_rec(p1), s0 = ld_rec(p0 + 8), s1 = ld_rec(p1 + 8);
      v[2] = fr_add(v[2], fr_mul(w, fr_mul(fr_sub(a1, a0), fr_sub(s1, s0))));
      v[3] = fr_add(v[3], a0);
      v[4] = fr_add(v[4], a1);
      continue;
    }
    Fr a0, a1, s0, s1;
    if (MODE == kSecond) {
      const uint32_t *p0 = lk_row(J, t), *p1 = lk_row(J, t + h), *p2 = lk_row(J, t + 2 * h), *p3 = lk_row(J, t + 3 * h);
      a0 = fr_fold(r, ld_rec(p0), ld_rec(p2));
      a1 = fr_fold(r, ld_rec(p1), ld_rec(p3));
      s0 = fr_fold(r, ld_rec(p0 + 8), ld_rec(p2 + 8));
      s1 = fr_fold(r, ld_rec(p1 + 8), ld_rec(p3 + 8));
    } else {
      a0 = load_sol(J.A, ld, t);
      a1 = load_sol(J.A, ld, t + h);
      s0 = load_sol(J.S, ld, t);
      s1 = load_sol(J.S, ld, t + h);
      if (MODE == kFold) {
        a0 = fr_fold(r, a0, load_sol(J.A, ld, t + 2 * h));
        a1 = fr_fold(r, a1, load_sol(J.A, ld, t + 3 * h));
        s0 = fr_fold(r, s0, load_sol(J.S, ld, t + 2 * h));
        s1 = fr_fold(r, s1, load_sol(J.S, ld, t + 3 * h));
      }
    }
    if (MODE != kPlain) {
      store_sol(J.A, ld, t, a0);
      store_sol(J.A, ld, t + h, a1);
      store_sol(J.S, ld, t, s0);
      store_sol(J.S, ld, t + h, s1);
    }
    lk_weighted(w, a0, a1, s0, s1, v);
    v[3] = fr_add(v[3], a0);
    v[4] = fr_add(v[4], a1);
  }
  Fr hi = fr_R();
  if (m > nlo) hi = load_sol(J.EH + 8 * ((1ull << (m - nlo)) - 1), 1ull << (m - nlo), base >> nlo);
  lk_block_out(v, m > nlo ? &hi : nullptr, lk_part(J, rd, blk - L.block_begin));
}

// round rd's nine sums into acc (zeroed), one wave each
__device__ __forceinline__ void lk_sum_parts(const LookupJob& J, uint32_t rd, unsigned long long* acc) {
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t nblocks = lk_round_blocks(J.nH + J.nL, J.nH, rd);
  Fr v = fr_zero();
  for (uint32_t i = lane; i < nblocks; i += 64) v = fr_add(v, ld_rec(lk_part(J, rd, i) + 8 * wave));
  acc_add(acc, wave, v);
}
// the step of wide round rd by wave 0; write: by the one workgroup that stores
// proof bytes and io
__device__ __forceinline__ bool lk_wide_step(const LookupJob& J, uint32_t rd, const unsigned long long* acc, LkState& s,
                                             RoundLds& T, uint32_t lane, bool write) {
  if (!lk_step(J, rd, acc, s, T, lane, write)) {
    if (write && lane == 0) {
      J.io[0] = (uint32_t)VL_ERR_FALSE_STATEMENT;
      *J.status = VL_ERR_FALSE_STATEMENT;
    }
    return false;
  }
  if (write) {
    uint32_t* io = lk_slot(J, rd + 1);
    if (lane < 8) {
      io[lane] = T.st[lane];
      io[kLkSlotR + lane] = T.r[lane];
    }
    lk_advance(J, rd, s, T, lane);
    if ((lane & 3u) == 0 && lane < 12)
#pragma unroll
      for (int i = 0; i < 8; ++i) io[kLkSlotScale + 2 * lane + i] = s.sc.w[i];
    if (lane == 0)
#pragma unroll
      for (int i = 0; i < 8; ++i) io[kLkSlotK + i] = s.kc.w[i];
  }
  return true;
}

// One wide round in which a low index bit is bound, every table: 64 pairs a
// block, one wave per term (lk_term).  Few pairs: bound by a thread's chain of
// five products and by fetching the kernel's code, so the code is small.  The
// tables fold in place: every wave has read the block's entries before any
// wave writes.
// step: every block first takes round rd - 1's transcript step itself, from the
// previous launch's sums (its first block stores it), so that a round is one
// launch: 26 us instead of 11.5 and 16.5, while the launch has no more
// blocks than CUs (kLookupMergeBlocks).
__global__ void __launch_bounds__(64 * kLkTerms) lookup_sweep_low_kernel(const LookupJob* __restrict__ jobs,
                                                                         const LookupSweep* __restrict__ list,
                                                                         uint32_t n_list, uint32_t n_blocks,
                                                                         uint32_t rd, uint32_t step) {
  __shared__ unsigned long long acc[110];   // nine values; acc_point reads two past its base
  __shared__ RoundLds T;
  __shared__ uint32_t dead_s;
  const uint32_t blk = blockIdx.x;
  if (blk >= n_blocks) return;
  const LookupSweep& L = list[lk_find([&](uint32_t k) { return list[k].block_begin; }, n_list, blk)];
  const LookupJob& J = jobs[L.job];
  if (lk_io_status(J) != VL_OK) return;
  const uint32_t wave = threadIdx.x >> 6, lane = threadIdx.x & 63u;
  const uint32_t role = wave / 3, pt = wave % 3;
  const uint32_t n = J.nH + J.nL, m = n - 1 - rd, nlo = lk_nlo(n);
  const uint64_t h = 1ull << m;
  const uint64_t t = (uint64_t)(blk - L.block_begin) * kLookupLowPairs + lane;   // h is a multiple of 64 here
  const uint64_t ldA = J.gather ? 1ull << (n - 1) : 1ull << n, ldN = 1ull << J.nL;
  const bool fold = role == 0 ? rd > 0 : rd > J.nH;
  auto get = [&](uint32_t k, uint64_t i) {   // table k: A, Sb, B, T + beta, M'
    if (k == 2 || k == 3) return ld_rec(J.rec + 16 * i + (k == 3 ? 8 : 0));
    return load_sol(k == 0 ? J.A : (k == 1 ? J.S : J.M), k == 4 ? ldN : ldA, i);
  };
  auto put = [&](uint32_t k, uint64_t i, const Fr& x) {
    if (k == 2 || k == 3) st_rec(J.rec + 16 * i + (k == 3 ? 8 : 0), x);
    else store_sol(k == 0 ? J.A : (k == 1 ? J.S : J.M), k == 4 ? ldN : ldA, i, x);
  };
  const uint32_t tx = role == 0 ? 0 : 2, ty = role == 0 ? 1 : role + 2;
  const uint64_t i0 = pt == 1 ? t + h : t;
  Fr ex[2], ey[2];
  ex[0] = get(tx, i0);
  ey[0] = get(ty, i0);
  if (fold) {
    ex[1] = get(tx, i0 + 2 * h);
    ey[1] = get(ty, i0 + 2 * h);
  }
  if (pt == 2) {
    ex[0] = fr_sub(get(tx, t + h), ex[0]);
    ey[0] = fr_sub(get(ty, t + h), ey[0]);
    if (fold) {
      ex[1] = fr_sub(get(tx, t + 3 * h), ex[1]);
      ey[1] = fr_sub(get(ty, t + 3 * h), ey[1]);
    }
  }
  if (threadIdx.x < 110) acc[threadIdx.x] = 0;
  if (threadIdx.x == 0) dead_s = 0;
  __syncthreads();   // everything read (and acc zeroed)
  if (step) {
    LkState s;
    if (wave == 0) lk_load_state(J, rd - 1, s, T, lane);
    lk_sum_parts(J, rd - 1, acc);
    __syncthreads();
    if (wave == 0) {
      const bool ok = lk_wide_step(J, rd - 1, acc, s, T, lane, blk == L.block_begin);
      acc[lane] = 0;
      if (lane < 46) acc[64 + lane] = 0;
      if (lane == 0 && !ok) dead_s = 1;
    }
    __syncthreads();
    if (dead_s) return;
  }
  const Fr r = step ? lds_get(T.r) : lds_or_global_fr(lk_slot(J, rd) + kLkSlotR);
  const Fr w = role == 2 ? fr_minus_one() : m > nlo ? fr_mul(lk_weight(J, nlo, t & ((1ull << nlo) - 1)),
                                load_sol(J.EH + 8 * ((1ull << (m - nlo)) - 1), 1ull << (m - nlo), t >> nlo))
                       : lk_weight(J, m, t);
  const LkTerm o = lk_term(ex, ey, fold, r, w);
  if (fold && pt < 2) {
    if (role != 2) put(tx, i0, o.X);
    put(ty, i0, o.Y);
  }
  acc_add(acc, wave, o.val);
  if (role == 0 && pt < 2) acc_add(acc, 6 + pt, o.X);
  __syncthreads();
  if (wave == 0) {
    const Fr v = acc_point(acc, min(lane, 8u), 0);
    if (lane < 9) st_rec(lk_part(J, rd, blk - L.block_begin) + 8 * lane, v);
  }
}

// The transcript step after a wide round, one workgroup per job, where the next
// sweep does not take it.
__global__ void __launch_bounds__(64 * 9) lookup_step_kernel(const LookupJob* __restrict__ jobs,
                                                             const LookupSweep* __restrict__ list, uint32_t rd) {
  __shared__ unsigned long long acc[110];   // nine values; acc_point reads two past its base
  __shared__ RoundLds T;
  const LookupJob& J = jobs[list[blockIdx.x].job];
  const uint32_t tid = threadIdx.x, lane = tid & 63u;
  if (lk_io_status(J) != VL_OK) return;
  if (tid < 110) acc[tid] = 0;
  LkState s;
  if (tid < 64) lk_load_state(J, rd, s, T, lane);
  __syncthreads();
  lk_sum_parts(J, rd, acc);
  __syncthreads();
  if (tid < 64) lk_wide_step(J, rd, acc, s, T, lane, true);
}

// The remaining rounds in one workgroup, then the final values.  The tables
// come from global memory until their first fold (at most 2^kLookupTailVars
// entries then) and live in LDS after it, folded from one buffer into the
// other.  The rows of 16 lanes of waves 1 .. 11 take the terms
// (lk_term) of 16 pairs at a time, so that short rounds leave no wave with
// idle lanes beside another on its SIMD (with a wave per term the last rounds
// took 25 us instead of 20); wave 0
// runs the transcript and moves the running scalars on while the others work.
// A round is a chain of one term (about 1700 instructions), the values (900)
// and the hash (4700), 4 cycles each.
constexpr uint32_t kTailWaves = 12;
__global__ void __launch_bounds__(64 * kTailWaves) lookup_rounds_kernel(const LookupJob* __restrict__ jobs) {
  const LookupJob& J = jobs[blockIdx.x];
  constexpr uint32_t kLen = 1u << (kLookupTailVars - 1);   // entries of the first LDS buffer
  __shared__ alignas(16) uint32_t buf[5][8 * (kLen + kLen / 2)];   // A, Sb, B, T, M': two buffers each
  __shared__ unsigned long long acc[110];   // nine values; acc_point reads two past its base
  __shared__ RoundLds T;
  __shared__ uint32_t dead_s;
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = tid & 63u;
  const int32_t st0 = lk_io_status(J);
  if (st0 != VL_OK) {
    if (tid == 0) *J.status = st0;
    return;
  }
  const uint32_t nH = J.nH, n = nH + J.nL, wide = J.wide;
  const uint64_t ldA = J.gather ? 1ull << (n - 1) : 1ull << n, ldN = 1ull << J.nL;
  uint32_t *const gA = J.A, *const gS = J.S, *const gM = J.M, *const gR = J.rec;
  bool pending = wide > 0;
  // where the tables' entries are: -1 global, else the LDS buffer of length
  // kLen (0) or kLen / 2 (1); tables 0, 1 fold every round, 2 .. 4 in low ones
  int atA = -1, atB = -1;
  auto get = [&](uint32_t k, uint32_t i) {
    const int w = k < 2 ? atA : atB;
    if (w >= 0) return ld_rec(buf[k] + (w ? 8 * kLen : 0) + 8 * i);
    if (k == 2 || k == 3) return ld_rec(gR + 16 * (uint64_t)i + (k == 3 ? 8 : 0));
    return load_sol(k == 0 ? gA : (k == 1 ? gS : gM), k == 4 ? ldN : ldA, i);
  };
  auto put = [&](uint32_t k, uint32_t i, const Fr& x) {
    const bool w = (k < 2 ? atA : atB) == 0;
    st_rec(buf[k] + (w ? 8 * kLen : 0) + 8 * i, x);
  };
  LkState s;
  if (wave == 0) {
    __builtin_amdgcn_s_setprio(3);   // the transcript's wave goes before those it shares its SIMD with
    lk_load_state(J, wide, s, T, lane);
  }
  if (tid < 110) acc[tid] = 0;
  if (tid == 0) dead_s = 0;
  __syncthreads();
#pragma unroll 1
  for (uint32_t rd = wide; rd < n; ++rd) {
    const uint32_t h = 1u << (n - 1 - rd);
    const bool low = rd >= nH, fold_rows = pending && rd > nH;
    if (wave == 0) {
      if (rd > wide) lk_advance(J, rd - 1, s, T, lane);
    } else {
      // units of 16 pairs of one term, one per row of lanes
      const uint32_t chunks = (h + 15) / 16, units = (low ? kLkTerms : 3) * chunks;
      const Fr r = lds_get(T.r);
#pragma unroll 1
      for (uint32_t q0 = 4 * (wave - 1); q0 < units; q0 += 4 * (kTailWaves - 1)) {
        const uint32_t q = q0 + (lane >> 4), c = q / chunks, role = c / 3, pt = c % 3;
        const uint32_t t = (q % chunks) * 16 + (lane & 15u);
        const uint32_t tx = role == 0 ? 0 : 2, ty = role == 0 ? 1 : role + 2;
        const bool take = q < units, fold = role == 0 ? pending : fold_rows;
        LkTerm o;
        o.X = o.Y = o.val = fr_zero();
        if (take && t < h) {
          Fr w = fr_minus_one();
          if (role < 2) w = lk_weight(J, n - 1 - rd, t);
          // entries i0 (pt 2: those of t + h less those of t), and 2 h further on
          const uint32_t i0 = pt == 1 ? t + h : t, d = pt == 2 ? h : 0;
          Fr ex[2], ey[2];
          auto entry = [&](uint32_t tab, uint32_t off) {
            Fr x = get(tab, i0 + d + off);
            if (pt == 2) x = fr_sub(x, get(tab, t + off));
            return x;
          };
          ex[0] = entry(tx, 0);
          ey[0] = entry(ty, 0);
          if (fold) {
            ex[1] = entry(tx, 2 * h);
            ey[1] = entry(ty, 2 * h);
          }
          o = lk_term(ex, ey, fold, r, w);
          if (fold && pt < 2) {
            if (role != 2) put(tx, i0, o.X);
            put(ty, i0, o.Y);
          }
        }
        acc_add(acc, c, o.val, take);
        const bool lin = take && role == 0 && pt < 2;
        if (__ballot(lin)) acc_add(acc, 6 + pt, o.X, lin);
      }
    }
    if (pending) atA = atA == 0 ? 1 : 0;
    if (fold_rows) atB = atB == 0 ? 1 : 0;
    __syncthreads();   // the sums, and the folded entries
    if (wave == 0) {
      const bool ok = lk_step(J, rd, acc, s, T, lane);
      acc[lane] = 0;
      if (lane < 26) acc[64 + lane] = 0;
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
  // lane k < 5: the final value of table k (the last challenge bound a high
  // bit, which leaves B, T and M' alone, or a low bit)
  const uint32_t k = min(lane, 4u);
  const bool folds = pending && (k < 2 || n - 1 >= J.nH);
  Fr mine = get(k, 0);
  if (folds) mine = fr_fold(r, mine, get(k, 1));
  Fr v[5];
#pragma unroll
  for (int q = 0; q < 5; ++q) v[q] = readlane_fr(mine, q);
  if (n == 0) {
    // no rounds (one entry, one row): the guard is the summand itself
    const Fr f = fr_add(fr_add(fr_mul(fr_mul(lk_fr(J.alpha), v[0]), v[1]), v[0]),
                        fr_sub(fr_mul(fr_mul(lk_fr(J.c1), v[2]), v[3]), fr_mul(v[2], v[4])));
    if (!fr_eq(f, lk_fr(J.claim))) {
      if (lane == 0) *J.status = VL_ERR_FALSE_STATEMENT;
      return;
    }
  }
  // the values sent: A, S = Sb - beta, B, T and m(r_L) = M'(r_L) / c2 = 2^nH M'(r_L)
  const Fr shifted = fr_sub(mine, lk_fr(J.beta));
  if (k == 1 || k == 3) mine = shifted;
  if (k == 4)
    for (uint32_t i = 0; i < nH; ++i) mine = fr_double(mine);
  mine = fr_from_mont(mine);
  if (lane < 5) {
    put_canon(J.proof + 128ull * n + 32 * lane, mine);
    lds_put(T.v + 8 * lane, mine);
  }
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  if (J.digest) {
    tr_absorb_lanes(T, kLblFinal4, kLblFinal1, 5);
    if (lane == 0) tr_put_digest(T, J.digest);
  }
  if (lane == 0) *J.status = VL_OK;
}

hipError_t launch_lookup_hist(const LookupJob* jobs, uint32_t n_jobs, uint32_t n_blocks, uint32_t lds_bytes,
                              hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_hist_kernel, dim3(n_blocks), dim3(1024), lds_bytes, s, jobs, n_jobs, n_blocks);
  return hipGetLastError();
}

hipError_t launch_lookup_tables(const LookupJob* jobs, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_tables_kernel, dim3(n_blocks), dim3(256), 0, s, jobs, n_jobs, n_blocks);
  return hipGetLastError();
}

hipError_t launch_lookup_mult(const LookupJob* jobs, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_mult_kernel, dim3(n_blocks), dim3(256), 0, s, jobs, n_jobs, n_blocks);
  return hipGetLastError();
}

hipError_t launch_lookup_prep(const LookupJob* jobs, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_prep_kernel, dim3(n_blocks), dim3(256), 0, s, jobs, n_jobs, n_blocks);
  return hipGetLastError();
}

hipError_t launch_lookup_start(const LookupJob* jobs, uint32_t n_jobs, hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_start_kernel, dim3(n_jobs), dim3(kWave), 0, s, jobs);
  return hipGetLastError();
}

hipError_t launch_lookup_sweep(const LookupJob* jobs, const LookupSweep* list, uint32_t n_list, uint32_t n_blocks,
                               uint32_t round, LookupSweepKind kind, bool step, hipStream_t s) {
  if (n_blocks == 0) return hipSuccess;
  const dim3 g(n_blocks), b(256);
  switch (kind) {
    case LK_FIRST: hipLaunchKernelGGL(lookup_sweep_kernel<kFirst>, g, b, 0, s, jobs, list, n_list, n_blocks, round); break;
    case LK_SECOND: hipLaunchKernelGGL(lookup_sweep_kernel<kSecond>, g, b, 0, s, jobs, list, n_list, n_blocks, round); break;
    case LK_FOLD: hipLaunchKernelGGL(lookup_sweep_kernel<kFold>, g, b, 0, s, jobs, list, n_list, n_blocks, round); break;
    case LK_PLAIN: hipLaunchKernelGGL(lookup_sweep_kernel<kPlain>, g, b, 0, s, jobs, list, n_list, n_blocks, round); break;
    default:
      hipLaunchKernelGGL(lookup_sweep_low_kernel, g, dim3(64 * kLkTerms), 0, s, jobs, list, n_list, n_blocks, round,
                         step ? 1u : 0u);
      break;
  }
  return hipGetLastError();
}

hipError_t launch_lookup_step(const LookupJob* jobs, const LookupSweep* list, uint32_t n_list, uint32_t round,
                              hipStream_t s) {
  if (n_list == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_step_kernel, dim3(n_list), dim3(64 * 9), 0, s, jobs, list, round);
  return hipGetLastError();
}

hipError_t launch_lookup_rounds(const LookupJob* jobs, uint32_t n_jobs, hipStream_t s) {
  if (n_jobs == 0) return hipSuccess;
  hipLaunchKernelGGL(lookup_rounds_kernel, dim3(n_jobs), dim3(64 * kTailWaves), 0, s, jobs);
  return hipGetLastError();
}

}  // namespace vl
