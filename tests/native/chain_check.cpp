// Gate chains (sv_chain_host.h) replayed in FP64 with the kernel's addressing,
// against the gates one by one in their order.
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "sv_chain_host.h"

using namespace sv;
typedef std::complex<double> cd;
constexpr int kT = chain::kTileBits;

#define CHECK(x)                                    \
  if (!(x)) {                                       \
    std::printf("FAILED %s n=%d t=%d\n", #x, n, t); \
    return 1;                                       \
  }

static int slot_of(int l) { return l ^ ((l >> 5) & 31) ^ ((l >> 10) & 31); }

static void multiply(std::vector<cd> &v, const std::vector<size_t> &at, const pass::Item &it) {
  const int D = 1 << it.k;
  std::vector<cd> in(D);
  for (int r = 0; r < D; ++r) in[r] = v[at[r]];
  for (int r = 0; r < D; ++r) {
    cd s = 0;
    for (int c = 0; c < D; ++c) s += cd(it.m[2 * (r * D + c)], it.m[2 * (r * D + c) + 1]) * in[c];
    v[at[r]] = s;
  }
}

static void apply_gate(std::vector<cd> &v, const pass::Item &it) {
  const int D = 1 << it.k;
  size_t mask = 0;
  for (int j = 0; j < it.k; ++j) mask |= size_t(1) << it.A[j];
  std::vector<size_t> at(D);
  for (size_t y = 0; y < v.size(); ++y) {
    if (y & mask) continue;
    for (int r = 0; r < D; ++r) {
      at[r] = y;
      for (int j = 0; j < it.k; ++j) at[r] |= size_t(r >> j & 1) << it.A[j];
    }
    multiply(v, at, it);
  }
}

int main() {
  for (int n : {chain::kMinQubits - 1, chain::kMinQubits})
    for (int t = 0; t < 5; ++t) {
      std::mt19937 rng(unsigned(10 * n + t));
      std::uniform_real_distribution<double> u(-1, 1);
      std::vector<pass::Item> items(7);
      std::vector<std::vector<double>> mats(items.size());
      for (size_t g = 0; g < items.size(); ++g) {
        pass::Item &it = items[g];
        it.k = t == 0 ? 4 : (g == 5 ? 3 + 4 * (t & 1) : 4 + int(rng() % 3));  // a width no chain takes in between
        std::vector<int> p(static_cast<size_t>(n));
        for (int j = 0; j < n; ++j) p[size_t(j)] = j;
        std::shuffle(p.begin(), p.end(), rng);
        const int b = int(rng() % unsigned(n - it.k + 1));
        for (int j = 0; j < it.k; ++j) it.A[j] = t < 3 ? b + j : p[size_t(j)];  // neighbours, or any bits
        std::shuffle(it.A, it.A + it.k, rng);
        mats[g].resize(size_t(2) << (2 * it.k));
        for (double &z : mats[g]) z = u(rng);
        it.m = mats[g].data();
      }
      std::vector<cd> want(size_t(1) << n), got;
      for (cd &z : want) z = cd(u(rng), u(rng));
      got = want;
      for (const pass::Item &it : items) apply_gate(want, it);
      int at_item = 0, fused = 0;
      for (const chain::Step &s : chain::build(n, items)) {
        for (int i : s.items) CHECK(i == at_item++);  // none passes another one
        if (!s.fused) {
          CHECK(s.items.size() == 1);
          apply_gate(got, items[size_t(s.items[0])]);
          continue;
        }
        ++fused;
        CHECK(s.items.size() >= 2 && s.items.size() <= size_t(chain::kMaxGates) && s.sbit[0] == 0);
        for (int b = 1; b < kT; ++b) CHECK(s.sbit[b] > s.sbit[b - 1] && s.sbit[b] < n);
        for (size_t tile = 0; tile < size_t(1) << (n - kT); ++tile) {
          size_t base = tile;
          for (int b = 0; b < kT; ++b) base = ((base >> s.sbit[b]) << (s.sbit[b] + 1)) | (base & ((size_t(1) << s.sbit[b]) - 1));
          auto phys = [&](int l) {
            size_t z = base;
            for (int b = 0; b < kT; ++b) z |= size_t(l >> b & 1) << s.sbit[b];
            return z;
          };
          std::vector<cd> lds(size_t(1) << kT);
          for (int l = 0; l < 1 << kT; ++l) lds[size_t(slot_of(l))] = got[phys(l)];
          for (size_t x = 0; x < s.items.size(); ++x) {
            const chain::Gate &g = s.gate[x];
            const int K = g.K, AH = 1 << (K - 1);
            std::vector<char> hit(size_t(1) << kT, 0);
            std::vector<size_t> at(size_t(2 * AH));
            for (int unit = 0; unit < 1 << (kT - 5 - K); ++unit)
              for (int lane = 0; lane < 32; ++lane) {
                for (int r = 0; r < 2 * AH; ++r) {
                  int z = r >= AH ? g.half : 0;
                  for (int j = 0; j < 5; ++j) z ^= (lane >> j & 1) ? g.lane[j] : 0;
                  for (int j = 0; j < kT - 5 - K; ++j) z ^= (unit >> j & 1) ? g.unit[j] : 0;
                  for (int j = 0; j < K - 1; ++j) z ^= (r >> j & 1) ? g.c[j] : 0;
                  CHECK(z >= 0 && z % 8 == 0 && z / 8 < 1 << kT && !hit[size_t(z / 8)]);
                  hit[size_t(z / 8)] = 1;
                  at[size_t(r)] = size_t(z / 8);
                }
                multiply(lds, at, items[size_t(s.items[x])]);
              }
          }
          for (int l = 0; l < 1 << kT; ++l) got[phys(l)] = lds[size_t(slot_of(l))];
        }
      }
      CHECK(at_item == int(items.size()));
      CHECK((fused > 0) == (n >= chain::kMinQubits) || t >= 3);
      double err = 0, ref = 0;
      for (size_t i = 0; i < got.size(); ++i) {
        err += std::norm(got[i] - want[i]);
        ref += std::norm(want[i]);
      }
      CHECK(std::sqrt(err) <= 1e-12 * std::sqrt(ref));
    }
  std::printf("chain checks passed\n");
  return 0;
}
