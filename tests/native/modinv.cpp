// The running inverses of modinv30 under any matrices a batch of division steps
// can have (rows of absolute sum at most 2^30), chosen to make them as large as
// they get: they stay within 3 M / 2, so that adding 2 M makes them positive and
// three subtractions of M reduce them.  Then whole inverses, multiplied back.
#include "fq.hpp"

#include <cmath>
#include <cstdio>
#include <random>

using namespace vl;

struct FrMod30 {   // that of lookup.hip, from p
  static constexpr int L = 9;
  static constexpr int kBatches = 25;
  static constexpr uint32_t inv30 = 1u;
  static uint32_t limb(int i) {
    const int bit = 30 * i, j = bit >> 5, sh = bit & 31;
    uint64_t v = p_limb(j);
    if (j < 7) v |= (uint64_t)p_limb(j + 1) << 32;
    return (uint32_t)(v >> sh) & 0x3fffffffu;
  }
};

// sign and rough size of a x + b M
template <typename Mod>
static double combine(int64_t a, const int32_t (&x)[Mod::L], int64_t b) {
  int64_t c = 0;
  double v = 0, w = 1;
  for (int i = 0; i < Mod::L; ++i) {
    c += a * x[i] + b * (int64_t)Mod::limb(i);
    v += (i < Mod::L - 1 ? (double)(c & 0x3fffffff) : (double)c) * w;
    w *= 1073741824.0;
    c >>= 30;
  }
  return v;   // the top limb's sign is the sum's (an exact zero gives 0)
}
template <typename Mod>
static bool within(const int32_t (&x)[Mod::L]) {
  return combine<Mod>(-2, x, 3) >= 0 && combine<Mod>(2, x, 3) >= 0;
}

template <typename Mod>
static int adversary(std::mt19937_64& g) {
  constexpr int L = Mod::L;
  int32_t zero[L] = {};
  const double M = combine<Mod>(0, zero, 1);
  double most = 0;
  for (int run = 0; run < 40; ++run) {
    int32_t d[L] = {}, e[L] = {};
    e[0] = 1;
    for (int batch = 0; batch < 60; ++batch) {
      int32_t bd[L] = {}, be[L] = {};
      double best = -1;
      for (int k = 0; k < 64; ++k) {
        auto row = [&](int32_t& a, int32_t& b) {
          const int64_t s = (int64_t)1 << 30;
          const int64_t x = k % 4 == 0 ? s : (int64_t)(g() % (uint64_t)(s + 1)), y = s - x;
          a = (int32_t)(g() & 1 ? -x : x);
          b = (int32_t)(g() & 1 ? -y : y);
        };
        int32_t t[4], f[L] = {}, h[L] = {}, d2[L], e2[L];
        row(t[0], t[1]);
        row(t[2], t[3]);
        for (int i = 0; i < L; ++i) d2[i] = d[i], e2[i] = e[i];
        modinv_apply<Mod>(t, f, h, d2, e2);
        if (!within<Mod>(d2) || !within<Mod>(e2)) {
          printf("beyond 3 M / 2 after %d batches: %.3f M, %.3f M\n", batch + 1, combine<Mod>(1, d2, 0) / M,
                 combine<Mod>(1, e2, 0) / M);
          return 1;
        }
        const double size = fabs(combine<Mod>(1, d2, 0)) + fabs(combine<Mod>(1, e2, 0));
        if (size > best) {
          best = size;
          for (int i = 0; i < L; ++i) bd[i] = d2[i], be[i] = e2[i];
        }
      }
      for (int i = 0; i < L; ++i) d[i] = bd[i], e[i] = be[i];
      most = std::max(most, std::max(fabs(combine<Mod>(1, d, 0)), fabs(combine<Mod>(1, e, 0))) / M);
    }
  }
  printf("largest: %.3f M\n", most);
  return 0;
}

int main() {
  std::mt19937_64 g(1);
  int bad = adversary<FqMod30>(g) + adversary<FrMod30>(g);
  // whole inverses of Fq: a a^-1 = 1
  for (int k = 0; k < 20000; ++k) {
    Fq a = fq_zero();
    for (int i = 0; i < 12; ++i) a.w[i] = k < 384 ? (i == k / 32 ? 1u << (k % 32) : 0u) : (uint32_t)g();
    a.w[11] &= k < 384 ? ~0u : 0x0fffffffu;
    if (k >= 384 && k < 500) a = fq_sub(fq_q(), fq_from12(k - 383, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0));
    if (!fq_lt_q(a)) continue;
    if (!fq_eq(fq_mul(a, fq_inv(a)), fq_one()) && bad++ < 5) printf("inverse %d wrong\n", k);
  }
  // and of Fr
  for (int k = 0; k < 20000; ++k) {
    Fr a;
    for (int i = 0; i < 8; ++i) a.w[i] = k < 255 ? (i == k / 32 ? 1u << (k % 32) : 0u) : (uint32_t)g();
    a.w[7] &= 0x7fffffffu;
    if (!fr_lt_p(a)) continue;
    int32_t x[9], d[9];
    words_to_30<8, 9>(a.w, x);
    modinv30<FrMod30>(x, d);
    add_2m30<FrMod30>(d);
    uint32_t w[9];
    limbs30_to_words<9, 9>(d, w);
    // below 4 p: w = hi 2^224 + lo, reduced by Montgomery products
    Fr lo = fr_zero(), hi = fr_zero(), s = fr_zero();
    for (int i = 0; i < 7; ++i) lo.w[i] = w[i];
    hi.w[0] = w[7], hi.w[1] = w[8], s.w[7] = 1;
    const Fr inv = fr_add(lo, fr_mul(fr_to_mont(hi), s));
    if (!fr_eq(fr_mul(fr_to_mont(a), inv), fr_one_raw()) && bad++ < 5) printf("inverse %d wrong (Fr)\n", k);
  }
  return bad != 0;
}
