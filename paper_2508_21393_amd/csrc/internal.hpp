// Internal job descriptors shared by the kernels and the host orchestration.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/verilora.h"
#include "contract_job.hpp"
#include "fr.hpp"

namespace vl {


// An eq table to build: out[i] = prod_j (x_j or 1 - x_j), i < 2^nvars, plus
// its "pack" form used by the integer contractions (see contract kernel).
constexpr uint32_t kEqBlock = 256;
struct EqJob {
  uint32_t nvars;
  uint32_t pack_len;          // entries to emit into pack (8 signed digits each)
  uint32_t block_begin;       // prefix sum of blocks (kEqBlock entries each) over jobs in a launch
  uint32_t pack_r2;           // 1: pack holds e * R^2 (contractions land in Montgomery
                              // form); 0: e * R (they land in canonical form)
  uint32_t eq_canon;          // 1: eq holds canonical values, 0: Montgomery form
  uint32_t pad_;
  const uint32_t* point;      // device: nvars Montgomery elements x_j (8 words each)
  uint32_t* eq;               // SoL output, may be null
  uint64_t eq_ld;
  uint32_t* pack;             // pack_len * 8 words, may be null
};

// eq table of a point passed by value (at most 20 variables)
struct EqPointArgs {
  uint32_t nvars;
  uint32_t pad_;
  uint32_t* out;
  uint64_t ld;
  uint32_t pt[20][8];         // Montgomery
};

// A slice of a host image copied to device memory by a kernel launch.
constexpr uint32_t kUploadBytes = 3072;   // multiple of 4 (blob sizes are multiples of 256)
struct UploadArgs {
  void* dst;
  uint32_t bytes;
  uint32_t pad_;
  uint32_t words[kUploadBytes / 4];
};

// Round 1 of one product (or the claim's dot product: c = sum_i eqU[i] t[i]
// after a contraction of C by columns, c = sum_j eqV[j] s[j] after one by rows)
// as per-block partial sums, computed across the GPU before the rounds.
constexpr uint32_t kPass1Pairs = 512;   // pairs (entries for the dot) per block
constexpr uint32_t kPass1Block = 768;
struct Pass1Job {
  const uint32_t* a;          // SoL table (eqU or eqV for the claim)
  const uint32_t* b;          // SoL table (t or s for the claim)
  uint64_t a_ld, b_ld;
  uint32_t h;                 // pairs (t, t + h), or entries of the dot product
  uint32_t dot;               // 1: sum_i a[i] b[i]; 0: the sums of round 1 (values at 0, 1, leading coefficient)
  uint32_t block_begin;       // prefix sum of blocks within a launch
  uint32_t pad_;
  uint32_t* out;              // 3 elements (24 words) per block
  uint32_t* ready;            // persistent mode: the group's readiness counter, else null
};

struct RoundsProd {
  uint32_t* a;
  uint32_t* b;
  uint64_t ld;
  uint32_t n1;
  uint32_t g_nparts;          // pass-1 partials of round 1 (3 elements each)
  const uint32_t* g_part;
};

// Wide rounds: a group whose first product's half-table has at least
// kMatWidePairs pairs in round 2 sums that product's first `wide` rounds
// across the GPU before its rounds workgroup starts: round 1 in pass 1 as
// always, each later one in a launch of mat_sweep_kernel (fold by the previous
// challenge, the round's partial sums, kMatSweepPairs pairs per block) whose
// every block first takes the previous round's transcript step from the
// previous launch's partials; the rounds workgroup takes the last wide
// round's step.  io (in the descriptor blob, so every call starts from
// zeros): [0] status, [8..23] transcript state after round k in slot k & 1,
// [24..39] r_k in slot k & 1 (Montgomery).  The partials lie in entries of the
// a~ table that the round folds away (mat_part).
constexpr uint32_t kMatSweepPairs = 128;      // pairs that a sweep block takes at a time
// blocks of a wide round at the most: every block takes the transcript step, so
// beyond one per CU they take more pairs each (2^20 inner entries: the first
// sweeps with 2048, 1024 and 512 blocks 224, 105 and 49 us, so 71, 38 and 28)
constexpr uint32_t kMatSweepBlocks = 256;
inline __host__ __device__ uint32_t mat_span(uint32_t pairs) {   // pairs per block (pairs: a power of two)
  const uint32_t s = pairs / kMatSweepBlocks;
  return s < kMatSweepPairs ? kMatSweepPairs : s;
}
// a group goes wide from this many pairs of its second round on, in calls of few
// groups (wide_rounds): a wide round takes 18 to 20 us, the first 25 to 31
constexpr uint32_t kMatWidePairs = 512;
// rounds of at most this many pairs are summed ahead of their challenge in the
// rounds workgroup (two products of 4096 inner entries: 415 us with 256 here,
// 441 with 512; much longer rounds three times as long ahead)
constexpr uint32_t kMatAhead = 256;
constexpr uint32_t kMatLds = 512;             // entries of the rounds workgroup's LDS tables
constexpr uint32_t kMatMaxWide = 16;          // n1 <= 20 needs at most 11
constexpr uint32_t kMatIoState = 8, kMatIoR = 24, kMatIoWords = 48;
struct MatSweep {
  uint32_t job;               // index in the launch's RoundsJob array
  uint32_t block_begin;       // prefix sum of sweep blocks within the launch
};
// int16 row contractions of large asynchronous calls: chunk factor, and the
// matrix bytes a call must stream to use it
constexpr uint32_t kRows16LongChunks = 16;
constexpr double kRows16LongMinBytes = 1e9;

// The sumcheck rounds of one group, run by one workgroup.
struct RoundsJob {
  uint32_t st[8];             // transcript state (digest words) after squeezing u and v
  uint32_t n_prods;
  uint32_t n0;
  uint8_t* proof;             // device proof bytes of this group
  int32_t* status;            // device status word of this group
  uint8_t* digest;            // device 32 bytes or null
  const int32_t* err;         // range flag of this group's contractions
  const uint32_t* c_part;     // pass-1 partials of c (element 0 of each)
  uint32_t c_nparts;
  uint32_t ready_target;      // persistent mode: pass-1 blocks of this group
  const uint32_t* ready;      // persistent mode: readiness counter, else null
  uint32_t spin_limit;        // polls of `ready` before giving up (VL_ERR_TIMEOUT)
  uint32_t wide;              // product 0's rounds summed by wide launches (0: none, else >= 2)
  uint32_t* io;               // wide rounds: status, transcript states, challenges
  RoundsProd prods[VL_MAX_PRODS];
};

// A matrix MLE value M~(x, y) from the pass-1 partial sums of its dot
// product (a chained proof's evaluation at a random point): the partials are
// added and the canonical value written as 32 proof bytes.
struct EvalJob {
  const uint32_t* part;       // pass-1 partials (element 0 of each is used)
  uint32_t nparts;
  uint32_t pad_;
  uint8_t* out;               // 32 bytes, canonical little-endian
  const int32_t* err;         // range flag of the contraction
  int32_t* status;            // VL_OK, or VL_ERR_RANGE
};

// One phase of a claim reduction (several claims M~(x_k, y_k) = v_k on one
// matrix turned into one):
//  phase 1: a sumcheck over the row variables of
//           sum_k rho_k sum_i eq(x_k, i) t_k(i),  t_k(i) = sum_j M[i][j] eq(y_k, j),
//           weights w[k] = eq(x_k, .) (Montgomery), tables b[k] = t_k
//           (canonical); then the values t_k(r) are sent and absorbed,
//           sigma_1..sigma_K squeezed; r (Montgomery), sigma and the state go
//           to io
//  phase 2: a sumcheck over the column variables of
//           sum_j M~(r, j) sum_k sigma_k eq(y_k, j),
//           weights w[k] = eq(y_k, .) (canonical), table a[0] = M~(r, .)
//           (Montgomery); then M~(r, s) is sent
// The first `wide` rounds run as GPU-wide sweeps; a round's step is taken by the
// next sweep's blocks, by a launch of its own before larger sweeps, and for the
// last of them by the workgroup that runs the rest.
constexpr int kMaxClaims = 3;
constexpr uint32_t kMaxReduceClaims = kMaxClaims;
constexpr uint32_t kRedSweepPairs = 128;     // pairs per sweep block (two threads per claim each)
// rounds with at least this many pairs run wide (shorter ones are summed ahead
// in the workgroup, where one of 256 pairs of three claims would outlast the
// hash)
constexpr uint32_t kRedWidePairs = 256;
constexpr uint32_t kRedMergeBlocks = 256;
constexpr uint32_t kRedPartWords = 16 * kMaxReduceClaims;
struct ReduceJob {
  uint32_t st[8];             // phase 1: transcript state after the rho squeezes
  uint32_t coef[kMaxClaims][8];   // phase 1: rho_k, Montgomery
  uint32_t phase;             // 1 or 2
  uint32_t K;                 // claims
  uint32_t n;                 // rounds (row or column variables)
  uint32_t wide;
  uint32_t slot;              // io words before the second slot
  uint32_t pad_;
  uint64_t ld;                // table stride, 2^n
  uint32_t* a[1];
  uint32_t* b[kMaxClaims];
  uint32_t* w[kMaxClaims];
  const uint32_t* pt[kMaxClaims];   // the points x_k or y_k, Montgomery (their eq jobs')
  uint32_t* part;             // round 0's sums, 2 K elements per block
  uint32_t* io;               // two slots (below)
  uint8_t* proof;             // this phase's proof bytes
  uint8_t* digest;            // phase 2: final state of the reduction's branch
  int32_t* status;            // phase 2: VL_OK when done
};
// io: [state: 8][running scalars, then sigma: kMaxClaims x 8][r: n_rows x 8],
// then a second slot [state][running scalars][r: 8]; wide round rd leaves its
// state and scalars in the first for odd rd, in the second for even rd, and phase
// 2 its challenge too (phase 1's r have been read by then)
constexpr uint32_t kReduceIoSigma = 8, kReduceIoR = 8 + 8 * kMaxClaims;
constexpr uint32_t reduce_io_slot(uint32_t n_rows) { return kReduceIoR + 8 * (n_rows ? n_rows : 1); }
constexpr uint32_t reduce_io_words(uint32_t n_rows) { return reduce_io_slot(n_rows) + kReduceIoR + 8; }

// One per-head batched product (vl_bmm_prove): C_h = A_h B_h for h < H as
// one sumcheck over (head, inner) variables of
//     sum_{h, w} eq(rho, h) a[h, w] b[h, w],  a[h, w] = A~(h, u, w),
//     b[h, w] = B~(h, w, v),
// head variables first (rounds of degree 3, weighted with the eq table of
// rho's suffix), then the inner ones (degree 2, times the head rounds'
// scalar).  Tables: E = eq(rho, .) (2^nh entries, Montgomery, replaced by the
// suffixes' tables), a (Montgomery) and b (canonical) over 2^(nh + n1)
// entries, head index most significant, so every round value is canonical.
// The first `wide` rounds run as GPU-wide sweeps (bmm_sweep_kernel, one launch
// per round); a round's transcript step is taken by the next sweep's blocks, by
// a launch of its own (bmm_step_kernel) before sweeps of more than
// kBmmMergeBlocks blocks, and for the last of them by the workgroup that runs
// the rest (bmm_rounds_kernel).  io holds the state handed between the
// launches.
constexpr uint32_t kBmmSweepPairs = 256;     // pairs per sweep block (three threads each)
// rounds with at least this many pairs run wide (one of 512 or 256 takes 22 us,
// in one workgroup 28)
constexpr uint32_t kBmmWidePairs = 256;
constexpr uint32_t kBmmMergeBlocks = 256;
constexpr uint32_t kBmmLds = 1024;           // entries of the rounds workgroup's LDS tables
constexpr uint32_t kBmmAhead = 128;          // rounds with at most this many are summed ahead in the rounds workgroup
constexpr uint32_t kBmmMaxWide = 24;
// io words: [0] status (VL_OK while running), [8, 16) the claim c (canonical),
// [16, 40) and [40, 64) what round rd leaves for the next, by parity: the
// transcript state, the challenge r and the running scalar (Montgomery)
constexpr uint32_t kBmmIoC = 8, kBmmIoSlot = 16, kBmmSlotR = 8, kBmmSlotScale = 16, kBmmIoWords = 64;
struct BmmJob {
  uint32_t st[8];             // transcript state after squeezing rho, u, v
  uint8_t nh, n1;             // head and inner variables
  uint8_t wide;               // rounds done by the sweep/step launches
  uint8_t pad_;
  uint32_t c_nparts;
  const uint32_t* rho;        // Montgomery (the point of E's eq job; its index until fill_blob)
  const uint32_t* c_part;     // pass-1 partials of the claim's dot product
  uint32_t* E;                // ld 2^nh
  uint32_t* a;                // ld 2^(nh + n1)
  uint32_t* b;
  uint32_t* part;             // round 0's sums: 3 elements per block
  uint32_t* io;
  uint8_t* proof;             // device-writable proof bytes
  uint8_t* digest;            // 32 bytes or null
  int32_t* status;            // device-writable status word
  const int32_t* err;         // range flag of the job's contractions
};
// a job's part in one wide round: its blocks start at block_begin
struct BmmSweep {
  uint32_t job;
  uint32_t block_begin;
};

// One lookup argument (vl_lookup_prove, Protocol 1 with the sum of
// eq. (lookup-sumcheck)): every entry (x_i[, y_i]) of a secret tensor is a
// row (t0 + j[, tb_j]) of a table of N = 2^nL rows.  S is padded to
// D' = 2^(nH + nL) entries with the table's first row.  Tables (Montgomery):
// over the rows the records {B = 1/(beta + T), T + beta} and M' = c2 m; over
// the padded entries A = 1/(beta + S) and Sb = S + beta, which are the
// entries' rows' records: with nH >= 2 and wide rounds the first two rounds
// look them up (gather) and store them folded, from half the entries on.
// Rounds bind the high index bits first (only A and Sb depend on them; the
// rows' terms add a constant per round), then the low bits.  The first `wide`
// rounds run as GPU-wide sweeps and a one-block transcript step.
// rounds with at least this many pairs run wide: a wide round of 256 pairs takes
// 26 us with its step, the eight rounds of 128 pairs and fewer in one workgroup
// 160 to 170 together
constexpr uint32_t kLookupWidePairs = 256;
constexpr uint32_t kLookupTailVars = 9;       // log2 of the entries the one-workgroup rounds start from, at most
constexpr uint32_t kLookupLowPairs = 64;       // pairs per block of a low round's sweep
constexpr uint32_t kLkTerms = 9;               // terms of a low round's pair: three products at three points
constexpr uint32_t kLookupPartWords = 72;      // a sweep block's nine sums
constexpr uint32_t kLookupMaxWide = 32;
constexpr uint32_t kLookupLdsVars = 16;        // tables of up to 2^16 rows are counted in LDS
// variables of the low factor of an eq suffix: its table's entries (2^11)
// stay in L1 while a sweep block passes over them
constexpr uint32_t kLookupLoVars = 11;
inline __host__ __device__ uint32_t lk_nlo(uint32_t n) {
  return n == 0 ? 0 : (n - 1 < kLookupLoVars ? n - 1 : kLookupLoVars);
}
// pairs per block of a high round's sweep with h pairs: as many as the low
// eq factor covers, down to one per thread to keep two blocks per CU
inline __host__ __device__ uint64_t lk_span(uint64_t h) {
  uint64_t s = 1ull << kLookupLoVars;
  while (s > 256 && h / s < 512) s >>= 1;
  return s;
}
inline __host__ __device__ uint32_t lk_round_blocks(uint32_t n, uint32_t nH, uint32_t rd) {
  const uint64_t h = 1ull << (n - 1 - rd), s = rd >= nH ? kLookupLowPairs : lk_span(h);
  return (uint32_t)((h + s - 1) / s);
}
// low rounds whose sweep has at most this many blocks take the step of the round
// before (where every job of that round goes on with one)
constexpr uint32_t kLookupMergeBlocks = 256;
// io words: [0] status, then two slots of what round rd leaves for the next, by
// parity: [0, 8) state, [8, 16) r, [16, 24) the next high round's constant,
// [24, 48) the running scalars
constexpr uint32_t kLkIoSlot = 8, kLkSlotR = 8, kLkSlotK = 16, kLkSlotScale = 24, kLkSlotWords = 48;
constexpr uint32_t kLkIoWords = kLkIoSlot + 2 * kLkSlotWords;
struct LookupJob {
  uint32_t st[8];             // transcript state after gamma, beta, alpha, u
  uint32_t gamma[8], beta[8], alpha[8], c1[8], c2[8];   // Montgomery (c1 = alpha^2 N / D', c2 = N / D')
  uint32_t claim[8];          // alpha + alpha^2, Montgomery
  const void* x;              // D entries, dtype
  const void* y;              // second column or null
  const int32_t* tb;          // table's second column or null
  int32_t dtype, dtype_y;
  int32_t t0;
  uint32_t gather;            // 1: rounds 0 and 1 look A and Sb up
  uint64_t D;
  uint32_t nH, nL;
  uint32_t wide;
  uint32_t hist_begin;        // block prefixes: histogram launch,
  uint32_t prep_begin;        // preparation launch (padded entries; none with gather),
  uint32_t tab_begin;         // table launch: inv_blocks of row chunks, then the eq entries
  uint32_t mult_begin;        // multiplicity launch (one table row per thread)
  uint32_t inv_blocks;
  uint32_t nkparts;           // multiplicity-launch blocks (partials of sum_j B_j m_j)
  uint32_t hist_chunk, hist_blocks;   // entries per histogram block, blocks
  uint32_t inv_chunk;         // table rows per thread of the table launch
  const uint32_t* u;          // the point u, Montgomery (8 words each)
  uint32_t* hist;             // counts: N / 2 words per block (16-bit), or N words zeroed by the plan
  uint32_t* A;                // ld D' (D' / 2 with gather)
  uint32_t* S;
  uint32_t* W;                // eq of u's last m <= lk_nlo variables, at 8 (2^m - 1) words
  uint32_t* EH;               // eq of the last m of the other variables
  uint32_t* rec;              // row records {B, T + beta}, 16 words each
  uint32_t* M;                // ld N
  uint32_t* kpart;
  uint32_t* part;             // sweep partials
  uint32_t* io;
  int32_t* flag;              // set when an entry is not in the table
  uint8_t* proof;
  uint8_t* digest;
  int32_t* status;
};
enum LookupSweepKind { LK_FIRST, LK_SECOND, LK_FOLD, LK_PLAIN, LK_LOW, LK_KINDS };
struct LookupSweep {
  uint32_t job;
  uint32_t block_begin;
};

// Where block b of wide round rd leaves its sums.  A sweep that takes the step
// of round rd - 1 itself has every block read that round's sums while others
// may already be storing their own, so the two rounds' places are apart: from
// the first fold on, a round's sums lie in the entries of a table's first
// plane (or records) that its block b, and no other, folds away in it, which
// the next round leaves alone.
inline __host__ __device__ uint32_t* mat_part(const RoundsJob& J, uint32_t rd, uint32_t b) {   // rd >= 1
  const uint32_t h = 1u << (J.prods[0].n1 - 1 - rd);
  return J.prods[0].a + 2ull * h + (uint64_t)mat_span(h) * b;
}
inline __host__ __device__ uint32_t* red_part(const ReduceJob& J, uint32_t rd, uint32_t b) {
  if (rd == 0) return J.part + kRedPartWords * b;
  return (J.phase == 1 ? J.b[0] : J.a[0]) + (2u << (J.n - 1 - rd)) + kRedSweepPairs * b;
}
static_assert(kRedPartWords <= kRedSweepPairs, "a block's sums fit its folded entries");
inline __host__ __device__ uint32_t* bmm_part(const BmmJob& J, uint32_t rd, uint64_t b) {
  return rd == 0 ? J.part + 24 * b : J.a + (2ull << (J.nh + J.n1 - 1 - rd)) + kBmmSweepPairs * b;
}
// (a lookup's first low round folds no records: its sums go behind those of the
// last high round, which its sweep reads)
inline __host__ __device__ uint64_t lk_part_block(uint32_t n, uint32_t nH, uint32_t rd, uint64_t b) {   // rd <= nH
  return b + (rd == nH && rd > 0 ? lk_round_blocks(n, nH, rd - 1) : 0u);
}
inline __host__ __device__ uint32_t* lk_part(const LookupJob& J, uint32_t rd, uint64_t b) {
  if (rd <= J.nH) return J.part + kLookupPartWords * lk_part_block(J.nH + J.nL, J.nH, rd, b);
  return J.rec + 16 * ((2ull << (J.nH + J.nL - 1 - rd)) + kLookupLowPairs * b);
}

// host launchers (kernels.hip)
hipError_t launch_eval(const EvalJob* jobs_dev, uint32_t n_jobs, hipStream_t s);
hipError_t launch_reduce(const ReduceJob* jobs_dev, uint32_t n_jobs, hipStream_t s);
hipError_t launch_reduce_sweep(const ReduceJob* jobs_dev, const MatSweep* list_dev, uint32_t n_list, uint32_t n_blocks,
                               uint32_t round, bool step, hipStream_t s);
hipError_t launch_reduce_step(const ReduceJob* jobs_dev, const MatSweep* list_dev, uint32_t n_list, uint32_t round,
                              hipStream_t s);
hipError_t launch_eq(const EqJob* jobs_dev, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s);
hipError_t launch_contract(int kind, const ContractJob* jobs_dev, uint32_t n_jobs, uint32_t n_tasks,
                           hipStream_t s);
hipError_t launch_finish(const FinishJob* jobs_dev, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s);
hipError_t launch_pass1(const Pass1Job* jobs_dev, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s);
hipError_t launch_rounds(const RoundsJob* jobs_dev, uint32_t n_jobs, hipStream_t s);
hipError_t launch_mat_sweep(const RoundsJob* jobs_dev, const MatSweep* list_dev, uint32_t n_list, uint32_t n_blocks,
                            uint32_t round, hipStream_t s);

hipError_t launch_lift(const void* src, int dtype, uint64_t n, uint32_t* dst, uint64_t ld, hipStream_t s);
hipError_t launch_export(const uint32_t* src, uint64_t ld, uint64_t n, uint32_t* dst, hipStream_t s);
hipError_t launch_eq_point(const EqPointArgs& a, hipStream_t s);
hipError_t launch_pack(const uint32_t* eq, uint64_t ld, uint64_t len, uint32_t* pack, hipStream_t s);
hipError_t launch_upload(void* dst, const void* src, uint64_t bytes, hipStream_t s);
hipError_t launch_zero_words(uint32_t* p, uint64_t n_words, hipStream_t s);
// batched products (bmm.hip)
hipError_t launch_bmm_start(const BmmJob* jobs_dev, uint32_t n_jobs, hipStream_t s);
hipError_t launch_bmm_sweep(const BmmJob* jobs_dev, const BmmSweep* list_dev, uint32_t n_list, uint32_t n_blocks,
                            uint32_t round, bool step, hipStream_t s);
hipError_t launch_bmm_step(const BmmJob* jobs_dev, const BmmSweep* list_dev, uint32_t n_list, uint32_t round,
                           hipStream_t s);
hipError_t launch_bmm_rounds(const BmmJob* jobs_dev, uint32_t n_jobs, hipStream_t s);
// lookup arguments (lookup.hip)
hipError_t launch_lookup_hist(const LookupJob* jobs_dev, uint32_t n_jobs, uint32_t n_blocks, uint32_t lds_bytes,
                              hipStream_t s);
hipError_t launch_lookup_tables(const LookupJob* jobs_dev, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s);
hipError_t launch_lookup_mult(const LookupJob* jobs_dev, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s);
hipError_t launch_lookup_prep(const LookupJob* jobs_dev, uint32_t n_jobs, uint32_t n_blocks, hipStream_t s);
hipError_t launch_lookup_start(const LookupJob* jobs_dev, uint32_t n_jobs, hipStream_t s);
hipError_t launch_lookup_sweep(const LookupJob* jobs_dev, const LookupSweep* list_dev, uint32_t n_list,
                               uint32_t n_blocks, uint32_t round, LookupSweepKind kind, bool step, hipStream_t s);
hipError_t launch_lookup_step(const LookupJob* jobs_dev, const LookupSweep* list_dev, uint32_t n_list,
                              uint32_t round, hipStream_t s);
hipError_t launch_lookup_rounds(const LookupJob* jobs_dev, uint32_t n_jobs, hipStream_t s);
// Hyrax: generators and fixed-base tables of windows W for m generators;
// commitments of R rows of an int16/int32/int64 matrix in n_split column
// slices of chunk columns (partials: R n_split XYZZ points)
// slices of a row that one wave sums (eight per quad of lanes), and the most
// slices the final kernel takes without a pass of runs before it; the runs' sums take
// R ceil(n_split / kHyraxRun) points behind the slices
constexpr uint32_t kHyraxRun = 128, kHyraxMaxFinal = 256;
hipError_t launch_hyrax_setup(uint32_t m, uint32_t W, uint32_t* table, hipStream_t s);
hipError_t launch_hyrax_commit(const void* M, int dtype, uint64_t ld, uint32_t R, uint32_t m, uint32_t W,
                               const uint32_t* table, uint32_t n_split, uint32_t chunk, uint32_t lanes,
                               uint32_t* partials, bool with_runs, uint32_t* commits, hipStream_t s);
// bytes (a multiple of 16, both pointers 16-byte aligned) from pinned host
// memory, given by its device-side address
hipError_t launch_copy_in(void* dst, const void* src_dev, uint64_t bytes, hipStream_t s);


}  // namespace vl
