// The first wide sweep of a segment, whose blocks all take the transcript step:
// no more blocks than the GPU has CUs, however many groups the call has; a call
// of one group goes wide from 2^11 inner entries on.
#include <hip/hip_runtime.h>

#include "plan.hpp"

#include <cstdio>

using namespace vl;

int main() {
  int bad = 0;
  for (uint32_t segments : {1u, 2u, 4u})
    for (uint32_t n : {1u, 2u, 9u, 49u, 64u, 100u, 200u, 700u})
      for (uint32_t n1 = 8; n1 <= 20; ++n1) {
        std::vector<vl_product> prods(n);
        std::vector<vl_group> groups(n);
        for (uint32_t k = 0; k < n; ++k) {
          prods[k] = vl_product{};
          prods[k].D0 = prods[k].D2 = 8;
          prods[k].D1 = 1u << (k % 3 == 2 ? n1 - 1 : n1);   // two lengths
          prods[k].dtype_a = prods[k].dtype_b = VL_I16;
          prods[k].lda = 1u << n1;
          prods[k].ldb = 8;
          groups[k] = vl_group{};
          groups[k].group_id = k;
          groups[k].n_prods = 1;
          groups[k].prods = &prods[k];
          groups[k].dtype_c = VL_I64;
          groups[k].ldc = 8;
        }
        Tuning T;
        T.segments = segments;
        Plan P;
        plan_groups(P, T, groups.data(), 0, n, 1, nullptr, true, nullptr, nullptr, nullptr, nullptr, nullptr, nullptr);
        uint32_t wide = 0;
        for (const Segment& G : P.seg) {
          for (const RoundsJob& J : G.rounds) wide += J.wide ? 1 : 0;
          if (G.wide_blocks.size() > 1 && G.wide_blocks[1] > 256) {
            printf("%u segments, %u groups of 2^%u: %u blocks\n", segments, n, n1, G.wide_blocks[1]);
            ++bad;
          }
        }
        if (n == 1 && (wide == 1) != (n1 >= 11)) printf("one group of 2^%u: %u wide\n", n1, wide), ++bad;
        if (wide != P.n_wide) printf("%u wide groups, %u slots\n", wide, P.n_wide), ++bad;
      }
  return bad != 0;
}
