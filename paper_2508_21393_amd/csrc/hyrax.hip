// Device kernels of the Hyrax commitments (vl_hyrax_setup, vl_hyrax_commit).
//
// A Hyrax commitment to the multilinear extension of an R x m matrix M (rows
// indexed by the first variables) is one Pedersen vector commitment per row,
// C_i = sum_j M[i][j] G_j, over generators G_j of G1 that nobody knows a
// relation between (Sec. II-A's polynomial commitments; the paper's
// implementation uses Hyrax, whose commitment time dominates its wall clock,
// Table t2).  The entries of the committed tensors are small signed integers,
// so each entry is recoded into signed base-256 digits d_w in [-128, 128],
// M[i][j] = sum_w d_w 256^w, and the commitment becomes a sum of table points:
//     C_i = sum_j sum_w sign(d_w) T_j,w[|d_w|],  T_j,w[k] = k 256^w G_j,
// one mixed addition per nonzero digit (fixed-base precomputation; the
// tables are public parameters computed once per generator count).
//
//   hyrax_gen_kernel     G_j by try-and-increment hashing to the curve and
//                        cofactor clearing (one thread per generator)
//   hyrax_table_kernel   T_j,w[k] for k = 1..128 (one thread per point)
//   hyrax_commit_kernel  one lane per (row, column slice): the sum of the
//                        table points of its entries
//   hyrax_sum_kernel     sums of runs of a row's slices
//   hyrax_final_kernel   a row's slices summed by a group of lanes, in affine
//                        coordinates, encoded as 96 canonical bytes
#include "device.hpp"
#include "fq.hpp"

namespace vl {

namespace {

constexpr uint32_t kHyraxDigits = 128;       // table points per (generator, window)
constexpr uint32_t kPointWords = 24;         // affine point: x, y of 12 limbs
constexpr uint32_t kZWords = 48;             // XYZZ point

__device__ __forceinline__ void store_point(uint32_t* dst, const G1a& a) {
  u32x4* d = reinterpret_cast<u32x4*>(dst);
#pragma unroll
  for (int v = 0; v < 3; ++v) d[v] = u32x4{a.x.w[4 * v], a.x.w[4 * v + 1], a.x.w[4 * v + 2], a.x.w[4 * v + 3]};
#pragma unroll
  for (int v = 0; v < 3; ++v) d[3 + v] = u32x4{a.y.w[4 * v], a.y.w[4 * v + 1], a.y.w[4 * v + 2], a.y.w[4 * v + 3]};
}

__device__ __forceinline__ G1a load_point(const uint32_t* src) {
  const u32x4* s = reinterpret_cast<const u32x4*>(src);
  G1a a;
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    const u32x4 t = s[v];
    a.x.w[4 * v] = t.x; a.x.w[4 * v + 1] = t.y; a.x.w[4 * v + 2] = t.z; a.x.w[4 * v + 3] = t.w;
  }
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    const u32x4 t = s[3 + v];
    a.y.w[4 * v] = t.x; a.y.w[4 * v + 1] = t.y; a.y.w[4 * v + 2] = t.z; a.y.w[4 * v + 3] = t.w;
  }
  return a;
}

__device__ __forceinline__ uint64_t table_index(uint32_t j, uint32_t W, uint32_t w, uint32_t k) {
  return (((uint64_t)j * W + w) * kHyraxDigits + (k - 1)) * kPointWords;
}

// G_j (one thread per generator); a generator no counter below 256 yields
// (probability 2^-256) is left as zero words, which the table kernel and
// every later check treat as invalid
__global__ void __launch_bounds__(64) hyrax_gen_kernel(uint32_t m, uint32_t W, uint32_t* table) {
  const uint32_t j = blockIdx.x * 64 + threadIdx.x;
  if (j >= m) return;
  G1a G;
  if (!hyrax_generator(j, G)) {
    G.x = fq_zero();
    G.y = fq_zero();
  }
  store_point(table + table_index(j, W, 0, 1), G);
}

// T_j,w[k] = (k 256^w) G_j for k = 1..128; block (j, w), thread k - 1.  The
// entry (w = 0, k = 1) is G_j itself, written by the generator kernel.
__global__ void __launch_bounds__(128) hyrax_table_kernel(uint32_t m, uint32_t W, uint32_t* table) {
  const uint32_t jw = blockIdx.x;
  const uint32_t j = jw / W, w = jw % W, k = threadIdx.x + 1;
  if (j >= m || (w == 0 && k == 1)) return;
  const G1a G = load_point(table + table_index(j, W, 0, 1));
  const uint64_t s = (uint64_t)k << (8 * w);
  store_point(table + table_index(j, W, w, k), g1_to_affine(g1_mul_u64(G, s)));
}

// Points of the commitment kernels: XYZZ coordinates as lazily reduced Fl
// elements (fq.hpp) in Montgomery form with R' = 2^392.  The table holds
// x 2^384 and y 2^384; shifting the words by 4 and 2 bits while they are cut
// into limbs gives 2^-4 x and 2^-6 y in R' form, a point of the curve that
// (x, y) -> (u^2 x, u^3 y) with u = 2^-2 maps G1 to, where the same formulas
// add; the final kernel maps the sum back.  Invariants of a finite point:
// X below 9q < 2^384 with limbs below 2^28 + 16; Y, ZZ, ZZZ below 2q with
// limbs below 2^28.  Infinity: ZZ = 0 (all limbs).
#if defined(__HIP_DEVICE_COMPILE__)
typedef u32x4 __attribute__((aligned(4))) u32x4a;   // workspace accesses assume word alignment only
struct G1l {
  Fl X, Y, ZZ, ZZZ;
};

__device__ __forceinline__ Fl fl_zero() {
  Fl r;
#pragma unroll
  for (int i = 0; i < 14; ++i) r.l[i] = 0;
  return r;
}
__device__ __forceinline__ bool fl_all_zero(const Fl& a) {
  uint32_t z = 0;
#pragma unroll
  for (int i = 0; i < 14; ++i) z |= a.l[i];
  return z == 0;
}
__device__ __forceinline__ Fl fl_one() {   // 2^392 mod q
  constexpr uint32_t w[12] = {0x0347fcb8u, 0x19d80000u, 0x6d2002b1u, 0x12e00cdeu, 0xa2090c72u, 0x37669f83u,
                              0xda0f73e0u, 0x09b09b42u, 0x8f1297bbu, 0xa7c515d9u, 0xfcfa012cu, 0x0577a659u};
  return fl_split<0>(w);
}
__device__ __forceinline__ Fl fl_small(uint32_t v) {
  Fl r = fl_zero();
  r.l[0] = v;
  return r;
}

// X3 = R^2 - PPP - 2Q (limb bounds 2^28 each): below 9q, one carry pass
__device__ __forceinline__ Fl x3_of(const Fl& rr, const Fl& ppp, const Fl& q) {
  Fl r;
#pragma unroll
  for (int i = 0; i < 14; ++i) r.l[i] = rr.l[i] + (kq_limb<7, 3>(i) - ppp.l[i] - 2 * q.l[i]);
  return fl_carry1(r);
}

// 2 P (dbl-2008-s-1 with a = 0)
__device__ __forceinline__ G1l g1l_dbl(const G1l& p) {
  Fl U, M3;
#pragma unroll
  for (int i = 0; i < 14; ++i) U.l[i] = 2 * p.Y.l[i];
  const Fl V = fl_sqr(U);
  const Fl W = fl_mul(U, V);
  const Fl S = fl_mul(p.X, V);
  const Fl x2 = fl_sqr(p.X);
#pragma unroll
  for (int i = 0; i < 14; ++i) M3.l[i] = 3 * x2.l[i];
  G1l r;
  r.X = x3_of(fl_sqr(M3), fl_zero(), S);
  r.Y = fl_mul2_add(M3, fl_sub<16, 2>(S, r.X), fl_neg<4, 1>(W), p.Y);
  r.ZZ = fl_mul(V, p.ZZ);
  r.ZZZ = fl_mul(W, p.ZZZ);
  return r;
}

// p += (x, y), the affine point given by its limbs (values below 16q, limbs
// below 2^28 and 2^29): madd-2008-s, 8 products and 2 squarings with 9
// reductions (R (Q - X3) and -Y PPP share one).  An equal point doubles p, an
// opposite one gives infinity.
__device__ __forceinline__ void g1l_madd(G1l& p, const Fl& x, const Fl& y) {
  if (fl_all_zero(p.ZZ)) {
    const Fl one = fl_one();
    p.X = fl_mul(x, one);
    p.Y = fl_mul(y, one);
    p.ZZ = one;
    p.ZZZ = one;
    return;
  }
  const Fl P = fl_sub<16, 2>(fl_mul(x, p.ZZ), p.X);     // limbs below 4 2^28, below 18q
  const Fl R = fl_sub<4, 1>(fl_mul(y, p.ZZZ), p.Y);     // below 3 2^28, below 6q
  const Fl PP = fl_sqr(P);
  const Fl RR = fl_sqr(R);
  if (__builtin_expect(fl_is_zero(PP), 0)) {
    if (fl_is_zero(RR)) {
      p = g1l_dbl(p);
    } else {
      p.ZZ = fl_zero();
      p.ZZZ = fl_zero();
    }
    return;
  }
  const Fl PPP = fl_mul(P, PP);
  const Fl Q = fl_mul(p.X, PP);
  p.ZZ = fl_mul(p.ZZ, PP);
  p.ZZZ = fl_mul(p.ZZZ, PPP);
  p.X = x3_of(RR, PPP, Q);
  p.Y = fl_mul2_add(R, fl_sub<16, 2>(Q, p.X), fl_neg<4, 1>(p.Y), PPP);
}

__device__ __forceinline__ void store_fl(uint32_t* dst, const Fl& a) {
  Fl t = a;     // all limbs below 2^28 for the packing
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < 13; ++i) {
    const uint32_t s = t.l[i] + c;
    t.l[i] = s & kM28;
    c = s >> 28;
  }
  t.l[13] += c;
  const Fq w = fl_pack(t);
  u32x4a* d = reinterpret_cast<u32x4a*>(dst);
#pragma unroll
  for (int v = 0; v < 3; ++v) d[v] = u32x4a{w.w[4 * v], w.w[4 * v + 1], w.w[4 * v + 2], w.w[4 * v + 3]};
}
__device__ __forceinline__ Fl load_fl(const uint32_t* src) {
  uint32_t w[12];
  const u32x4a* s = reinterpret_cast<const u32x4a*>(src);
#pragma unroll
  for (int v = 0; v < 3; ++v) {
    const u32x4 t = s[v];
    w[4 * v] = t.x; w[4 * v + 1] = t.y; w[4 * v + 2] = t.z; w[4 * v + 3] = t.w;
  }
  return fl_split<0>(w);
}
// a point in 48 words (each value is below 2^384)
__device__ __forceinline__ void store_l(uint32_t* dst, const G1l& p) {
  store_fl(dst, p.X);
  store_fl(dst + 12, p.Y);
  store_fl(dst + 24, p.ZZ);
  store_fl(dst + 36, p.ZZZ);
}
__device__ __forceinline__ G1l g1l_infinity() {
  G1l p;
  p.X = p.Y = p.ZZ = p.ZZZ = fl_zero();
  return p;
}
// A point on four neighbouring lanes: lane q of the quad has X, Y, ZZ or ZZZ.
template <int CTRL>   // the limbs of lane (CTRL >> 2 q) & 3 of the quad
__device__ __forceinline__ Fl quad(const Fl& a) {
  Fl r;
#pragma unroll
  for (int i = 0; i < 14; ++i) r.l[i] = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)a.l[i], CTRL, 0xf, 0xf, true);
  return r;
}
__device__ __forceinline__ Fl fl_sel(bool c, const Fl& a, const Fl& b) {
  Fl r;
#pragma unroll
  for (int i = 0; i < 14; ++i) r.l[i] = c ? a.l[i] : b.l[i];
  return r;
}
// a + o (add-2008-s) on quads: four products deep, each of the 14 products of
// the formulas in one of the lanes.  Bounds as in g1l_madd, but for Y: two
// reduced products, below 4q, carried to limbs below 2^28.
__device__ __forceinline__ Fl quad_add(const Fl& a, const Fl& o, uint32_t q) {
  // a.X o.ZZ = U1, a.Y o.ZZZ = S1, a.ZZ o.X = U2, a.ZZZ o.Y = S2
  const Fl m1 = fl_mul(a, quad<0x4e>(o));
  const Fl d = fl_sub<4, 1>(quad<0x4e>(m1), m1);   // lane 0: P = U2 - U1, lane 1: R = S2 - S1
  // P^2, R^2, ZZ ZZ, ZZZ ZZZ
  const Fl m2 = fl_mul(fl_sel(q < 2, d, a), fl_sel(q < 2, d, o));
  const Fl pp = quad<0x00>(m2);
  // P PP = PPP, U1 PP = Q, ZZ ZZ PP
  const Fl m3 = fl_mul(fl_sel(q == 0, d, fl_sel(q == 1, quad<0x00>(m1), m2)), pp);
  const Fl ppp = quad<0x00>(m3), qq = quad<0x55>(m3);
  const Fl x3 = x3_of(quad<0x55>(m2), ppp, qq);
  // R (Q - X3), -S1 PPP, -, ZZZ ZZZ PPP
  const Fl m4 = fl_mul(fl_sel(q == 0, quad<0x55>(d), fl_sel(q == 1, fl_neg<4, 1>(m1), m2)),
                       fl_sel(q == 0, fl_sub<16, 2>(qq, x3), ppp));
  const Fl y0 = quad<0x00>(m4), y1 = quad<0x55>(m4);
  Fl r;
  uint32_t c = 0;
#pragma unroll
  for (int i = 0; i < 14; ++i) {
    const uint32_t t = y0.l[i] + y1.l[i] + c;
    const uint32_t y = i < 13 ? t & kM28 : t;
    c = t >> 28;
    r.l[i] = q == 0 ? x3.l[i] : (q == 1 ? y : (q == 2 ? m3.l[i] : m4.l[i]));
  }
  // infinity on either side, equal and opposite points
  uint32_t za = 0, zo = 0;
#pragma unroll
  for (int i = 0; i < 14; ++i) {
    za |= a.l[i];
    zo |= o.l[i];
  }
  za = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)za, 0xaa, 0xf, 0xf, true);
  zo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)zo, 0xaa, 0xf, 0xf, true);
  const bool same_x = za && zo && fl_is_zero(pp);
  if (__builtin_expect(__ballot(same_x) != 0, 0)) {
    G1l p;
    p.X = quad<0x00>(a);
    p.Y = quad<0x55>(a);
    p.ZZ = quad<0xaa>(a);
    p.ZZZ = quad<0xff>(a);
    const bool equal = fl_is_zero(quad<0x55>(m2));
    const G1l t = g1l_dbl(p);
    const Fl v = fl_sel(q == 0, t.X, fl_sel(q == 1, t.Y, fl_sel(q == 2, t.ZZ, t.ZZZ)));
#pragma unroll
    for (int i = 0; i < 14; ++i) r.l[i] = same_x ? (equal ? v.l[i] : 0u) : r.l[i];
  }
  return fl_sel(zo == 0, a, fl_sel(za == 0, o, r));
}
// The sum of partials[(s0 + k) R + i] for quad gl of the G quads of a row
// (k = gl, gl + G, ... < n), then over those quads (xor distances stride G / 2
// .. stride of lanes): every quad of the row ends with the sum.
__device__ __forceinline__ Fl sum_slices(const uint32_t* partials, uint64_t R, uint64_t i, uint32_t s0, uint32_t n,
                                         uint32_t gl, uint32_t G, uint32_t stride) {
  const uint32_t q = threadIdx.x & 3u, nl = (n + G - 1) / G;
  auto load = [&](uint32_t k) {
    return k < n ? load_fl(partials + ((uint64_t)(s0 + k) * R + i) * kZWords + 12 * q) : fl_zero();
  };
  Fl acc = load(gl);
  uint32_t k = gl + G, off = (G >> 1) * stride;
#pragma unroll 1
  for (uint32_t it = 1; it < nl || off >= stride; ++it) {
    Fl o;
    if (it < nl) {
      o = load(k);
      k += G;
    } else {
#pragma unroll
      for (int j = 0; j < 14; ++j) o.l[j] = __shfl_xor(acc.l[j], (int)off);
      off >>= 1;
    }
    acc = quad_add(acc, o, q);
  }
  return acc;
}
#endif

// digit w of v's signed base-256 recoding given the carry into window w:
// d in [-128, 127] below the top window (carry out when the byte plus carry
// is >= 128), the top digit in [-128, 128]; sum_w d_w 256^w = v
template <int WD>
__device__ __forceinline__ int digit_of(int64_t v, uint32_t w, int carry, int& cout) {
  if (w + 1 < (uint32_t)WD) {
    const int x = (int)(((uint64_t)v >> (8 * w)) & 0xffu) + carry;
    cout = x >= 128 ? 1 : 0;
    return x - (cout << 8);
  }
  cout = 0;
  return (int)(v >> (8 * (WD - 1))) + carry;
}

// A lane's nonzero terms (entry t, window w, digit d) in order.  Every
// madd of the commitment loop is executed by the whole wave, so a lane must
// not spend an iteration on a zero digit while the others add: each lane
// walks its own entries to its next nonzero digit (quantised weights mostly
// have a zero top digit), and the loop runs as many iterations as the lane
// with the most nonzero terms.  Entry t + 1 is loaded while entry t is in
// use.
template <typename T>
struct NonzeroTerms {
  static constexpr int WD = (int)sizeof(T);
  const T* row;
  uint32_t j0, cnt;       // the lane's entries j0 + t, t < cnt
  uint32_t t, w;          // the next term to examine
  int c;                  // carry into window w
  int64_t v;              // entry t
  T vn;                   // entry t + 1

  __device__ __forceinline__ T load(uint32_t k) const {
    return row[j0 + min(k, max(cnt, 1u) - 1)];   // clamped: always in the slice
  }
  __device__ __forceinline__ void init(const T* r, uint32_t j0_, uint32_t cnt_) {
    row = r; j0 = j0_; cnt = cnt_; t = 0; w = 0; c = 0;
    v = (int64_t)load(0);
    vn = load(1);
  }
  __device__ __forceinline__ bool next(int& d, uint32_t& j, uint32_t& win) {
    while (t < cnt) {
      int co;
      const int x = digit_of<WD>(v, w, c, co);
      const uint32_t jj = j0 + t, ww = w;
      if (w + 1 < (uint32_t)WD) {
        c = co;
        ++w;
      } else {
        w = 0;
        c = 0;
        ++t;
        v = (int64_t)vn;
        vn = load(t + 1);
      }
      if (x != 0) {
        d = x;
        j = jj;
        win = ww;
        return true;
      }
    }
    return false;
  }
};

// Lane t = s R + i sums M[i][j] G_j over the slice j in [s chunk, (s + 1)
// chunk) of columns, so the lanes of a wave take neighbouring rows of one
// slice and look up the same generators' points together.  Each iteration
// finds every lane's next nonzero term and loads its table point (a lane
// without one loads the slice's first point and adds nothing), then adds the
// current points.  Bound by the integer issue rate: about 4700 instructions
// of 4 cycles a mixed addition (3542 of them multiply-adds), no LDS, no
// cross-lane step.  With a wave per (row, slice), 32-bit limbs and carries
// (about 7900 instructions an addition and a butterfly over the lanes) a
// 4096 x 4096 int16 commitment took 4.82 ms, with this 2.99 ms.
#if defined(__HIP_DEVICE_COMPILE__)
template <typename T>
__device__ __forceinline__ G1l slice_sum(const T* row, uint32_t jb, uint32_t cnt, uint32_t W,
                                         const uint32_t* __restrict__ table) {
  const uint32_t* safe = table + table_index(jb, W, 0, 1);
  NonzeroTerms<T> ts;
  ts.init(row, jb, cnt);
  int dn = 0;
  uint32_t jn = 0, wn = 0;
  bool have = ts.next(dn, jn, wn);
  G1a nxt = load_point(have ? table + table_index(jn, W, wn, (uint32_t)abs(dn)) : safe);
  G1l acc = g1l_infinity();
  while (__ballot(have) != 0) {
    const G1a cur = nxt;
    const int d = have ? dn : 0;
    have = ts.next(dn, jn, wn);
    nxt = load_point(have ? table + table_index(jn, W, wn, (uint32_t)abs(dn)) : safe);
    if (d != 0) {
      const Fl x = fl_split<4>(cur.x.w);
      Fl y = fl_split<2>(cur.y.w);
      const Fl ny = fl_neg<8, 1>(y);
#pragma unroll
      for (int k = 0; k < 14; ++k) y.l[k] = d < 0 ? ny.l[k] : y.l[k];
      g1l_madd(acc, x, y);
    }
  }
  return acc;
}
#endif

template <typename T>
__global__ void __launch_bounds__(256, 2) hyrax_commit_kernel(const T* __restrict__ M, uint64_t ld, uint32_t R,
                                                              uint32_t m, uint32_t W,
                                                              const uint32_t* __restrict__ table, uint32_t n_split,
                                                              uint32_t chunk, uint32_t* partials) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint64_t task = (uint64_t)blockIdx.x * 256 + threadIdx.x;
  if (task >= (uint64_t)R * n_split) return;
  const uint32_t sl = (uint32_t)(task / R), i = (uint32_t)(task % R);
  const uint32_t jb = sl * chunk;
  store_l(partials + task * kZWords, slice_sum(M + (uint64_t)i * ld, jb, min(chunk, m - jb), W, table));
#endif
}

// The same for slices shared by `lanes` lanes (a power of two in 4 .. 64),
// where the caller's split or workspace gives too few slices to fill the GPU: a
// workgroup has 256 / lanes rows, whose lanes' sums it adds by quads through
// LDS (64 lanes: three additions a quad, then four levels over the quads).
// Bound like the kernel above: 16 x 11008 in one slice 2.2 ms, 119 on one lane
// each; 4096 x 4096 in a workspace for one slice 3.3 ms, 46 on one lane each.
template <typename T>
__global__ void __launch_bounds__(256, 2) hyrax_commit_cut_kernel(const T* __restrict__ M, uint64_t ld, uint32_t R,
                                                                  uint32_t m, uint32_t W,
                                                                  const uint32_t* __restrict__ table, uint32_t chunk,
                                                                  uint32_t lanes, uint32_t* partials) {
#if defined(__HIP_DEVICE_COMPILE__)
  __shared__ alignas(16) uint32_t sums[256 * kZWords];
  const uint32_t rows = 256 / lanes, groups = (R + rows - 1) / rows;
  const uint32_t sl = blockIdx.x / groups, i0 = blockIdx.x % groups * rows;
  const uint32_t jb = sl * chunk, len = min(chunk, m - jb), per = (len + lanes - 1) / lanes;
  const uint32_t part = threadIdx.x / rows, i = i0 + threadIdx.x % rows;   // neighbouring lanes: rows
  const uint32_t j0 = part * per, cnt = i < R && j0 < len ? min(per, len - j0) : 0;
  // (a lane without entries is given the slice's first one, of which it takes none)
  const G1l acc = slice_sum(M + (uint64_t)min(i, R - 1) * ld, cnt ? jb + j0 : jb, cnt, W, table);
  store_l(sums + threadIdx.x * kZWords, acc);
  __syncthreads();
  const uint32_t G = lanes / 4, wrows = 16 / G;   // quads per row, rows per wave
  const uint32_t wave = threadIdx.x >> 6, qd = (threadIdx.x >> 2) & 15u, q = threadIdx.x & 3u, gl = qd / wrows;
  const uint32_t row = wave * wrows + qd % wrows;
  const Fl sum = sum_slices(sums, rows, row, 0, lanes, gl, G, 4 * wrows);
  if (gl == 0 && i0 + row < R) store_fl(partials + ((uint64_t)sl * R + i0 + row) * kZWords + 12 * q, sum);
#endif
}

// Runs of `run` slices of a row summed by the 16 quads of one wave each: slice
// s' of out is the sum of slices s' run .. s' run + run - 1.
__global__ void __launch_bounds__(64) hyrax_sum_kernel(uint32_t R, uint32_t n_split, uint32_t run,
                                                       const uint32_t* __restrict__ partials, uint32_t* out) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t i = blockIdx.x % R, s = blockIdx.x / R;
  const uint32_t s0 = s * run;
  const Fl acc = sum_slices(partials, R, i, s0, min(run, n_split - s0), threadIdx.x >> 2, 16, 4);
  if (threadIdx.x < 4) store_fl(out + ((uint64_t)s * R + i) * kZWords + 12 * threadIdx.x, acc);
#endif
}

// C_i = the sum of row i's slices by a group of G quads (a power of two up to
// 16; a wave has 16 / G rows), as 96 canonical bytes (24 words).  Every lane
// inverts its row's ZZ ZZZ by division steps (modinv.hpp), so rows share
// nothing.  A chain of additions and one inversion of about 30 us.  An
// addition on one lane is 14 products deep, 11 us alone and more where the
// waves of a CU fetch its 60 KB of code at different places: the two kernels
// took 264 us for a 16 x 11008 matrix and 359 for 4096 x 4096, with the
// quads (four deep) 160 and 139.
__global__ void __launch_bounds__(64) hyrax_final_kernel(uint32_t R, uint32_t n_split, uint32_t G,
                                                         const uint32_t* __restrict__ partials, uint32_t* commits) {
#if defined(__HIP_DEVICE_COMPILE__)
  const uint32_t rows = 16 / G, qd = threadIdx.x >> 2, q = threadIdx.x & 3u;
  const uint64_t i = (uint64_t)blockIdx.x * rows + qd % rows;
  const uint32_t gl = qd / rows;
  const Fl acc = sum_slices(partials, R, min(i, (uint64_t)R - 1), 0, n_split, gl, G, 4 * rows);
  // lane 0 x = 2^4 X / ZZ, lane 1 y = 2^6 Y / ZZZ (the other two like lane 1)
  const Fl X = quad<0x54>(acc), Z = quad<0xaa>(acc), ZZZ = quad<0xff>(acc);
  const bool inf = fl_all_zero(Z);
  // 1 / (ZZ ZZZ) in R' form: the inverse of the integer a R' is a^-1 / R', and
  // a product with R'^3 gives a^-1 R'
  const Fq inv = fq_inv_raw(fl_pack(fl_mul(Z, ZZZ)));
  constexpr uint32_t r3[12] = {0xd1f7b890u, 0x22294cc4u, 0x56c9f3afu, 0xc0ccb5bau, 0xd975ccb5u, 0x89a8c5c0u,
                               0x6c968b4cu, 0x922672eau, 0xa691de8cu, 0x7c835652u, 0xbbb98497u, 0x141ab424u};
  Fl f = fl_split<0>(inv.w);
#pragma unroll 1
  for (uint32_t k = 0; k < 4; ++k) {   // one product's code, out of Montgomery form with the last
    Fl g = fl_sel(k == 0, fl_split<0>(r3), fl_sel(k == 1, fl_sel(q == 0, ZZZ, Z), X));
    if (k == 3) g = fl_small(q == 0 ? 16 : 64);
    f = fl_mul(f, g);
  }
  if (i >= R || gl != 0 || q >= 2) return;
  const Fq c = fq_reduce_once(fl_pack(f));
  uint32_t* out = commits + i * 24 + 12 * q;
#pragma unroll
  for (int k = 0; k < 12; ++k) out[k] = inf ? 0u : c.w[k];
#endif
}

}  // namespace

hipError_t launch_hyrax_setup(uint32_t m, uint32_t W, uint32_t* table, hipStream_t s) {
  hipLaunchKernelGGL(hyrax_gen_kernel, dim3(blocks_for(m, 64)), dim3(64), 0, s, m, W, table);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(hyrax_table_kernel, dim3((uint32_t)((uint64_t)m * W)), dim3(kHyraxDigits), 0, s, m, W, table);
  return hipGetLastError();
}

hipError_t launch_hyrax_commit(const void* M, int dtype, uint64_t ld, uint32_t R, uint32_t m, uint32_t W,
                               const uint32_t* table, uint32_t n_split, uint32_t chunk, uint32_t lanes,
                               uint32_t* partials, bool with_runs, uint32_t* commits, hipStream_t s) {
  auto commit = [&](auto* src) {
    using T = std::remove_const_t<std::remove_pointer_t<decltype(src)>>;
    if (lanes == 1) {
      const uint64_t tasks = (uint64_t)R * n_split;
      hipLaunchKernelGGL(hyrax_commit_kernel<T>, dim3((uint32_t)((tasks + 255) / 256)), dim3(256), 0, s, src, ld, R, m, W,
                         table, n_split, chunk, partials);
    } else {
      hipLaunchKernelGGL(hyrax_commit_cut_kernel<T>, dim3(blocks_for(R, 256 / lanes) * n_split), dim3(256), 0, s, src, ld,
                         R, m, W, table, chunk, lanes, partials);
    }
  };
  switch (dtype) {
    case VL_I16: commit(reinterpret_cast<const int16_t*>(M)); break;
    case VL_I32: commit(reinterpret_cast<const int32_t*>(M)); break;
    default: commit(reinterpret_cast<const int64_t*>(M)); break;
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // Many slices are first summed in runs of 128 (eight per quad of a wave);
  // the runs' sums go behind the slices (with_runs: there is room for them).
  if (with_runs && n_split > kHyraxMaxFinal) {
    const uint32_t runs = (n_split + kHyraxRun - 1) / kHyraxRun;
    uint32_t* sums = partials + (uint64_t)R * n_split * kZWords;
    hipLaunchKernelGGL(hyrax_sum_kernel, dim3(R * runs), dim3(64), 0, s, R, n_split, kHyraxRun, partials, sums);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    partials = sums;
    n_split = runs;
  }
  // as many quads per row as one wave on each SIMD gives: beyond that the
  // waves of a SIMD take turns at their inversions
  uint32_t G = 1;
  while (G < 16 && 2 * G <= n_split && (uint64_t)R * 8 * G <= 65536) G *= 2;
  hipLaunchKernelGGL(hyrax_final_kernel, dim3(blocks_for(R, 16 / G)), dim3(64), 0, s, R, n_split, G, partials, commits);
  return hipGetLastError();
}

}  // namespace vl
