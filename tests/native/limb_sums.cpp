// fr_of_limb_sums over its whole stated range, on the host: k p + r in ten limb
// sums must give r, for totals up to 2^272, also where the limbs are signed.
#include "fr.hpp"

#include <cstdio>

using namespace vl;

// k p + r as limb sums; lean > 0: limb i takes lean 2^26 from limb i + 1
static void sums(uint32_t k, const Fr& r, uint64_t lean, uint64_t (&t)[10]) {
  uint32_t w[10] = {};
  uint64_t c = 0;
  for (int i = 0; i < 8; ++i) {
    c += (uint64_t)k * p_limb(i) + r.w[i];
    w[i] = (uint32_t)c;
    c >>= 32;
  }
  w[8] = (uint32_t)c;
  for (int i = 0; i < 10; ++i) {
    const int bit = 26 * i, j = bit >> 5, sh = bit & 31;
    const uint64_t v = ((((uint64_t)w[j + 1]) << 32) | w[j]) >> sh;
    t[i] = i < 9 ? v & 0x3ffffff : v | (sh > 0 && j + 2 < 10 ? (uint64_t)w[j + 2] << (64 - sh) : 0);
  }
  for (int i = 0; i < 9; ++i) {
    t[i] += lean << 26;
    t[i + 1] -= lean;
  }
}

int main() {
  int bad = 0;
  Fr rem[5] = {fr_zero(), fr_one_raw(), fr_R(), fr_neg(fr_one_raw()), fr_half(fr_neg(fr_one_raw()))};
  // 2^272 = 144720.6 p
  for (uint32_t k = 0; k < 144720; ++k)
    for (const Fr& r : rem)
      for (uint64_t lean : {0ull, 1ull << 20}) {
        uint64_t t[10];
        sums(k, r, lean, t);
        if (!fr_eq(fr_of_limb_sums(t), r) && bad++ < 5) printf("%u p + %08x..: not reduced\n", k, r.w[7]);
      }
  printf("%d wrong\n", bad);
  return bad != 0;
}
