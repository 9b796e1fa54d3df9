// Layout permutations in tile passes (sv_permute_host.h), on the host: every
// pass keeps its tile size and bits 0..3, moves values inside its tile only,
// the passes together take the layout to its target, and the wide tile's LDS
// swizzle is a bijection with at most two lanes of a wave per slot.
#include <cstdio>
#include <cstdlib>
#include <random>

#include "sv_permute_host.h"

#define CHECK(c)                                         \
  do {                                                   \
    if (!(c)) {                                          \
      std::printf("failed line %d: %s\n", __LINE__, #c); \
      return 1;                                          \
    }                                                    \
  } while (0)

int main() {
  std::mt19937 rng(7);
  for (int n = 12; n <= 35; ++n)
    for (int S = sv::kPermTileBits; S <= sv::kPermWideBits && S <= n; ++S)
      for (int trial = 0; trial < 200; ++trial) {
        int32_t L[64], T[64];
        for (int q = 0; q < n; ++q) L[q] = T[q] = q;
        for (int q = n - 1; q > 0; --q) {
          std::swap(L[q], L[rng() % unsigned(q + 1)]);
          if (trial % 4) std::swap(T[q], T[rng() % unsigned(q + 1)]);
        }
        if (trial % 7 == 0)  // a few exchanges only
          for (int q = 0; q < n; ++q) T[q] = L[q];
        for (int e = 0; e < trial % 7 && trial % 4 == 0; ++e) std::swap(T[rng() % unsigned(n)], T[rng() % unsigned(n)]);
        int cur[64];
        for (int q = 0; q < n; ++q) cur[q] = L[q];
        const std::vector<sv::PermPass> passes = sv::permutation_tiles(L, T, n, S);
        CHECK(int(passes.size()) <= (n - 4 + S - 5) / (S - 4) + 1);
        for (const sv::PermPass &p : passes) {
          CHECK(__builtin_popcountll(p.tile) == S && (p.tile & sv::kPermLowRun) == sv::kPermLowRun);
          CHECK((p.tile >> n) == 0);
          uint64_t img = 0;
          for (int b = 0; b < n; ++b) {
            CHECK(((p.tile >> b) & 1) ? ((p.tile >> p.to[b]) & 1) : p.to[b] == b);
            img |= uint64_t(1) << p.to[b];
          }
          CHECK(img == (uint64_t(1) << n) - 1);
          for (int q = 0; q < n; ++q) cur[q] = p.to[cur[q]];
          int order[16], loc[16], k = 0;  // the store side's bit map, as the launcher builds it
          for (int b = 0; b < n; ++b)
            if ((p.tile >> b) & 1) order[k++] = b;
          for (int i = 0; i < S; ++i)
            for (int j = 0; j < S; ++j)
              if (p.to[order[i]] == order[j]) loc[j] = i;
          int32_t px[8];
          sv::choose_perm_swizzle(loc, px, S - 5);
          if (trial < 4) {
            std::vector<char> hit(size_t(1) << S, 0);
            for (int l = 0; l < (1 << S); ++l) {
              const int a = sv::lin_swz_host(l, px, S - 5);
              CHECK(a >= 0 && a < (1 << S) && !hit[size_t(a)] && sv::lin_swz_host(l ^ 1, px, S - 5) == (a ^ 1));
              hit[size_t(a)] = 1;
            }
          }
          int w[32] = {0}, r[32] = {0};
          for (int lane = 0; lane < 64; ++lane) {
            int lr = 0;
            for (int b = 0; b < 6; ++b)
              if ((lane >> b) & 1) lr |= 1 << loc[b + 1];
            CHECK(++w[sv::lin_swz_host(lane << 1, px, S - 5) & 31] <= 2);
            CHECK(++r[sv::lin_swz_host(lr, px, S - 5) & 31] <= 2);
          }
        }
        for (int q = 0; q < n; ++q) CHECK(cur[q] == T[q]);
      }
  std::printf("permutation checks passed\n");
  return 0;
}
