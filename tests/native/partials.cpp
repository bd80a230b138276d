// The merged launches of the provers: every block of round rd's sweep first
// reads all of round rd - 1's sums and its own table entries, and later stores
// its folded entries and its own sums, with no order between the blocks.  So no
// word that one block stores may be a word that another reads, and no two may
// store the same word.  Enumerated over the addresses that the planner and the
// *_part functions give (nothing is dereferenced).
#include "lookup.cpp"

#include <cstdio>
#include <unordered_map>

using namespace vl;

static unsigned long long g_checked = 0;

// words of 4 bytes by the block that stores them
struct Launch {
  std::unordered_map<uint64_t, uint32_t> owner;
  bool ok = true;
  explicit Launch(uint64_t words) { owner.reserve(words); }
  void store(uint32_t blk, const uint32_t* p, uint64_t words) {
    for (uint64_t i = 0; i < words; ++i) {
      auto r = owner.emplace((uint64_t)(p + i), blk);
      ok = ok && (r.second || r.first->second == blk);
    }
  }
  // read by block blk; every: by all blocks, before any is known to have stored
  void read(uint32_t blk, const uint32_t* p, uint64_t words, bool every) {
    for (uint64_t i = 0; i < words; ++i) {
      const auto f = owner.find((uint64_t)(p + i));
      ok = ok && (f == owner.end() || (!every && f->second == blk));
    }
    g_checked += words;
  }
  template <typename F>
  void planes(uint32_t* tab, uint64_t ld, uint64_t i, F f) {
    for (int w = 0; w < 8; ++w) f(tab + w * ld + i);
  }
};

// tab: SoL tables that fold (2 h entries stored, 4 h read); half: those that
// halve (h stored, 2 h read)
static bool sweep(const std::vector<uint32_t*>& tab, uint64_t ld, const std::vector<uint32_t*>& half, uint64_t h,
                  uint32_t pairs, uint32_t before, uint64_t words, const std::vector<uint32_t*>& was,
                  const std::vector<uint32_t*>& now) {
  Launch L(16 * h * tab.size() + 8 * h * half.size() + words * now.size());
  const uint32_t nb = (uint32_t)(h / pairs);
  if (nb != now.size() || before != was.size()) return false;
  for (uint32_t b = 0; b < nb; ++b) {
    for (uint64_t t = (uint64_t)b * pairs; t < (uint64_t)(b + 1) * pairs; ++t) {
      for (uint32_t* x : tab)
        for (int q = 0; q < 2; ++q) L.planes(x, ld, t + q * h, [&](uint32_t* p) { L.store(b, p, 1); });
      for (uint32_t* x : half) L.planes(x, ld, t, [&](uint32_t* p) { L.store(b, p, 1); });
    }
    L.store(b, now[b], words);
  }
  for (uint32_t* p : was) L.read(0, p, words, true);
  for (uint32_t b = 0; b < nb; ++b)
    for (uint64_t t = (uint64_t)b * pairs; t < (uint64_t)(b + 1) * pairs; ++t) {
      for (uint32_t* x : tab)
        for (int q = 0; q < 4; ++q) L.planes(x, ld, t + q * h, [&](uint32_t* p) { L.read(b, p, 1, false); });
      for (uint32_t* x : half)
        for (int q = 0; q < 2; ++q) L.planes(x, ld, t + q * h, [&](uint32_t* p) { L.read(b, p, 1, false); });
    }
  return L.ok;
}

static uint32_t* at(uint64_t word) { return reinterpret_cast<uint32_t*>(0x7f0000000000ull + 4 * word); }

static bool mat(uint32_t n1) {
  RoundsJob J{};
  const uint64_t ld = 1ull << n1;
  J.prods[0].a = at(0);
  J.prods[0].b = at(8 * ld);
  J.prods[0].n1 = n1;
  for (uint32_t rd = 1; rd < n1 && (1u << (n1 - 1 - rd)) >= kMatWidePairs; ++rd) {
    const uint32_t h = 1u << (n1 - 1 - rd);
    std::vector<uint32_t*> was, now;   // (round 0's sums lie in buffers of their own)
    for (uint32_t b = 0; rd > 1 && b < 2 * h / mat_span(2 * h); ++b) was.push_back(mat_part(J, rd - 1, b));
    for (uint32_t b = 0; b < h / mat_span(h); ++b) now.push_back(mat_part(J, rd, b));
    if (now.size() > 256) return false;   // every block takes a step: no more than the CUs
    if (!sweep({J.prods[0].a, J.prods[0].b}, ld, {}, h, mat_span(h), (uint32_t)was.size(), 24, was, now))
      return false;
  }
  return true;
}

static bool bmm(uint32_t nh, uint32_t n1) {
  BmmJob J{};
  const uint32_t nv = nh + n1;
  const uint64_t ld = 1ull << nv;
  J.nh = (uint8_t)nh;
  J.n1 = (uint8_t)n1;
  J.a = at(0);
  J.b = at(8 * ld);
  J.part = at(16 * ld);
  for (uint32_t rd = 1; rd < nv && (ld >> (rd + 1)) >= kBmmWidePairs; ++rd) {
    const uint64_t h = ld >> (rd + 1);
    if (h / kBmmSweepPairs > kBmmMergeBlocks) continue;
    std::vector<uint32_t*> was, now;
    for (uint64_t b = 0; b < 2 * h / kBmmSweepPairs; ++b) was.push_back(bmm_part(J, rd - 1, b));
    for (uint64_t b = 0; b < h / kBmmSweepPairs; ++b) now.push_back(bmm_part(J, rd, b));
    if (!sweep({J.a, J.b}, ld, {}, h, kBmmSweepPairs, (uint32_t)was.size(), 24, was, now)) return false;
  }
  return true;
}

static bool reduce(uint32_t n, uint32_t phase) {
  ReduceJob J{};
  const uint64_t ld = 1ull << n;
  J.phase = phase;
  J.n = n;
  std::vector<uint32_t*> tab, half;
  uint64_t o = 0;
  for (int k = 0; k < kMaxClaims; ++k) {
    J.b[k] = at(o), o += 8 * ld;
    J.w[k] = at(o), o += 8 * ld;
    if (phase == 1) tab.push_back(J.b[k]);
    half.push_back(J.w[k]);
  }
  J.a[0] = at(o), o += 8 * ld;
  if (phase == 2) tab.push_back(J.a[0]);
  J.part = at(o);
  for (uint32_t rd = 1; rd < n && (1u << (n - 1 - rd)) >= kRedWidePairs; ++rd) {
    const uint64_t h = 1ull << (n - 1 - rd);
    if (h / kRedSweepPairs > kRedMergeBlocks) continue;
    std::vector<uint32_t*> was, now;
    for (uint32_t b = 0; b < 2 * h / kRedSweepPairs; ++b) was.push_back(red_part(J, rd - 1, b));
    for (uint32_t b = 0; b < h / kRedSweepPairs; ++b) now.push_back(red_part(J, rd, b));
    if (!sweep(tab, ld, half, h, kRedSweepPairs, (uint32_t)was.size(), 16 * kMaxClaims, was, now)) return false;
  }
  return true;
}

// a call of lookups of (nH, nL) as planned at a made-up workspace address
static bool lookups(const std::vector<std::pair<uint32_t, uint32_t>>& sizes, uint32_t& merged) {
  Tuning T;
  Plan P;
  Builder B(P, T, 0x7f0000000000ull, 0);
  std::vector<uint64_t> end;
  for (const auto& s : sizes) {
    vl_lookup L{};
    L.D = 1ull << (s.first + s.second);
    L.N = 1u << s.second;
    plan_lookup(B, L, lookup_challenges(L, 1, false), nullptr, nullptr, nullptr, nullptr);
    end.push_back(B.base + B.off);   // the sums are the last thing a plan takes
  }
  for (size_t j = 0; j < P.lookups.size(); ++j) {
    const LookupJob& J = P.lookups[j];
    const uint32_t n = J.nH + J.nL;
    for (uint32_t k = 0; k < J.wide && k <= J.nH; ++k)
      if ((uint64_t)lk_part(J, k, lk_round_blocks(n, J.nH, k)) > end[j]) return false;
  }
  for (size_t k = 1; k < P.lk_wide[LK_LOW].size(); ++k) {
    if (!lookup_merged(P, k)) continue;
    ++merged;
    for (const LookupSweep& S : P.lk_wide[LK_LOW][k]) {
      const LookupJob& J = P.lookups[S.job];
      const uint32_t n = J.nH + J.nL, rd = (uint32_t)k, nb = lk_round_blocks(n, J.nH, rd),
                     before = lk_round_blocks(n, J.nH, rd - 1);
      const uint64_t h = 1ull << (n - 1 - rd), ldA = J.gather ? 1ull << (n - 1) : 1ull << n, ldN = 1ull << J.nL;
      const bool rows = rd > J.nH;   // the rows' tables fold from the second low round on
      Launch X(h * (rows ? 80 : 32) + nb * kLookupPartWords);
      auto entries = [&](uint32_t b, uint64_t t, bool store, int parts) {
        for (int q = 0; q < parts; ++q) {
          auto f = [&](uint32_t* p) { store ? X.store(b, p, 1) : X.read(b, p, 1, false); };
          X.planes(J.A, ldA, t + q * h, f);
          X.planes(J.S, ldA, t + q * h, f);
          if (store ? rows : (rows || q < 2)) {
            X.planes(J.M, ldN, t + q * h, f);
            for (int w = 0; w < 16; ++w) f(J.rec + 16 * (t + q * h) + w);
          }
        }
      };
      for (uint32_t b = 0; b < nb; ++b) {
        for (uint64_t t = (uint64_t)b * kLookupLowPairs; t < (uint64_t)(b + 1) * kLookupLowPairs; ++t) entries(b, t, true, 2);
        X.store(b, lk_part(J, rd, b), kLookupPartWords);
      }
      for (uint32_t b = 0; b < before; ++b) X.read(0, lk_part(J, rd - 1, b), kLookupPartWords, true);
      for (uint32_t b = 0; b < nb; ++b)
        for (uint64_t t = (uint64_t)b * kLookupLowPairs; t < (uint64_t)(b + 1) * kLookupLowPairs; ++t) entries(b, t, false, 4);
      if (!X.ok) return false;
    }
  }
  return true;
}

int main() {
  int bad = 0;
  auto say = [&](bool ok, const char* what, uint32_t x, uint32_t y) {
    if (!ok) printf("overlap: %s %u %u\n", what, x, y), ++bad;
  };
  // the smallest tables with such launches, and ones whose rounds are as wide as they get
  for (uint32_t n1 : {11, 12, 18}) say(mat(n1), "matmul", n1, 0);
  for (uint32_t nh : {0, 3})
    for (uint32_t nv : {9, 10, 18}) say(bmm(nh, nv - nh), "per-head", nh, nv - nh);
  for (uint32_t phase : {1, 2})
    for (uint32_t n : {9, 10, 17}) say(reduce(n, phase), "reduction", phase, n);
  uint32_t merged = 0;
  for (uint32_t nL = 0; nL <= 20; ++nL)
    for (uint32_t nH : {0u, 1u, 2u, 3u, 30 - nL}) say(lookups({{nH, nL}}, merged), "lookup", nH, nL);
  for (uint32_t nL = 9; nL <= 15; ++nL) say(lookups({{3, nL}, {3, nL}, {3, nL - 1}}, merged), "lookups", 3, nL);
  printf("%u merged lookup launches, %llu words read\n", merged, g_checked);
  return bad || !merged;
}
