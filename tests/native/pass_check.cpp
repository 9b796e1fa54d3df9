// Drives the fused-pass builder (sv_pass_host.cpp) on seeded random gate
// sequences and replays its device data in FP64 the way the kernel reads it
// (slot images, lane and unit bits, table parts, store-site tables); the
// state must equal the gates applied one by one.  Every LDS slot, table
// entry and buffer offset is range-checked on the way.
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <random>
#include <vector>

#include "sv.h"
#include "sv_pass_host.h"

using namespace sv::pass;
typedef std::complex<double> cd;

static float up(uint16_t h) {
  uint32_t u = uint32_t(h) << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

#define CHECK(c)                                                  \
  do {                                                            \
    if (!(c)) {                                                   \
      std::printf("failed line %d: %s\n", __LINE__, #c);          \
      std::exit(1);                                               \
    }                                                             \
  } while (0)

static void apply(std::vector<cd> &psi, const Item &it) {
  const size_t dim = psi.size();
  const int D = 1 << it.k;
  uint64_t mask = 0;
  for (int j = 0; j < it.k; ++j) mask |= uint64_t(1) << it.A[j];
  std::vector<cd> in(static_cast<size_t>(D));
  std::vector<size_t> off(static_cast<size_t>(D), 0);
  for (int c = 0; c < D; ++c)
    for (int j = 0; j < it.k; ++j)
      if ((c >> j) & 1) off[size_t(c)] |= size_t(1) << it.A[j];
  for (size_t b = 0; b < dim; ++b) {
    if (b & mask) continue;
    for (int c = 0; c < D; ++c) in[size_t(c)] = psi[b | off[size_t(c)]];
    for (int r = 0; r < D; ++r) {
      cd a = 0;
      for (int c = 0; c < D; ++c) a += cd(it.m[2 * (r * D + c)], it.m[2 * (r * D + c) + 1]) * in[size_t(c)];
      psi[b | off[size_t(r)]] = a;
    }
  }
}

static void replay(std::vector<cd> &psi, int n, const Fused &f) {
  const int S = f.S, pieces = 3;
  CHECK(S >= kMinS && S <= kMaxS && S <= n && f.sbit[0] == 0);
  const char *p = f.data.data();
  const size_t size = f.data.size();
  DevHead h;
  std::memcpy(&h, p, sizeof(h));
  CHECK(h.nchunks <= kMaxChunks && h.nchunks == f.nchunks && h.nops == f.nops && h.nblk * kTabBlock <= kTabEntries);
  CHECK(size_t(h.operand) + size_t(h.nchunks) * kChunkBytes <= size);
  const DevOp *ops = reinterpret_cast<const DevOp *>(p + h.ops);
  const DevTab *tabs = reinterpret_cast<const DevTab *>(p + h.tabs);
  const DevTab *stores = reinterpret_cast<const DevTab *>(p + h.stores);
  const DevBlk *blks = reinterpret_cast<const DevBlk *>(p + h.blks);
  const float *table = reinterpret_cast<const float *>(p + h.table);
  const int nwb = S - 10 < 3 ? S - 10 : 3, ntb = 6 + nwb, cb = S - 1 - ntb;
  std::vector<cd> lds(size_t(1) << S), tab(kTabEntries);
  for (uint64_t tile = 0; tile < (uint64_t(1) << (n - S)); ++tile) {
    uint64_t base = tile;
    for (int b = 0; b < S; ++b) base = ((base >> f.sbit[b]) << (f.sbit[b] + 1)) | (base & ((uint64_t(1) << f.sbit[b]) - 1));
    auto phys = [&](uint64_t l) {
      uint64_t y = base;
      for (int b = 0; b < S; ++b) y |= ((l >> b) & 1) << f.sbit[b];
      return y;
    };
    auto slot = [&](uint64_t l) {
      int32_t s = 0;
      for (int b = 0; b < S; ++b)
        if ((l >> b) & 1) s ^= slot_image(b);
      return s;
    };
    std::vector<char> hit(size_t(1) << S, 0);
    for (uint64_t l = 0; l < (uint64_t(1) << S); ++l) {
      const int32_t s = slot(l);
      CHECK(s >= 0 && s < (1 << S) && !hit[size_t(s)]);
      hit[size_t(s)] = 1;
      lds[size_t(s)] = psi[phys(l)];
    }
    for (int b = 0; b < kTabEntries / kTabBlock; ++b) {
      // a wave without a block of its own reads block 0
      const size_t at = size_t(h.blks) + size_t(b < h.nblk ? b : 0) * sizeof(DevBlk);
      CHECK(at + sizeof(DevBlk) <= size_t(h.table));
      const DevBlk &k = blks[b < h.nblk ? b : 0];
      CHECK(k.nout >= 0 && k.nout <= kTabOutMax);
      uint64_t part = 0;
      for (int q = 0; q < k.nout; ++q) {
        CHECK(k.out[q] >= 0 && k.out[q] < n);
        part |= ((base >> k.out[q]) & 1) << q;
      }
      for (int x = 0; x < kTabBlock; ++x) {
        const size_t e = size_t(k.goff) + (size_t(part) << k.nin) + size_t(x);
        CHECK(size_t(h.table) + 8 * e + 8 <= size_t(h.operand) && size_t(h.operand) <= size);
        if (b < h.nblk) tab[size_t(b * kTabBlock + x)] = cd(table[2 * e], table[2 * e + 1]);
      }
    }
    CHECK(size_t(h.ops) + size_t(h.nops) * sizeof(DevOp) <= size_t(h.tabs) && h.tabs <= h.stores &&
          size_t(h.stores) + size_t(h.nstore) * sizeof(DevTab) <= size_t(h.blks));
    for (int o = 0; o < h.nops; ++o)
      CHECK(size_t(h.tabs) + size_t((ops[o].tab & 0xFFFF) + (ops[o].tab >> 16 & 0xFF)) * sizeof(DevTab) <=
            size_t(h.stores));
    int chunk = 0;
    for (int o = 0; o < h.nops; ++o) {
      const DevOp &op = ops[o];
      const int K = (op.tab & kOpSix) ? 6 : 5, D = 1 << K, AH = D / 2, ub = S - 5 - K;
      const int tab0 = op.tab & 0xFFFF, ntab = op.tab >> 16 & 0xFF;
      CHECK(ub >= 0 && ub <= 4);
      const uint16_t *G = reinterpret_cast<const uint16_t *>(p + h.operand + size_t(chunk) * kChunkBytes);
      chunk += chunks_of(K);
      CHECK(chunk <= h.nchunks);
      // the matrix the operand blocks hold
      std::vector<cd> M(size_t(D) * D);
      const int mts = D / 32, steps = K == 6 ? 4 : 2;
      for (int mt = 0; mt < mts; ++mt)
        for (int kk = 0; kk < steps; ++kk)
          for (int l = 0; l < 64; ++l)
            for (int e = 0; e < 8; ++e) {
              const int i = l & 31, r = AH * ((i >> 2) & 1) + 16 * mt + 4 * (i >> 3) + (i & 3);
              const int c = AH * (l >> 5) + 8 * kk + e;
              double v[2] = {0, 0};
              for (int part = 0; part < 2; ++part)
                for (int w = 0; w < pieces; ++w) {
                  const int P = part * pieces + w;
                  const int block = K == 6 ? (kk * 2 * pieces + P) * 2 + mt : P * 2 + kk;
                  v[part] += up(G[(block * 64 + l) * 8 + e]);
                }
              M[size_t(r) * D + c] = cd(v[0], v[1]);
            }
      std::fill(hit.begin(), hit.end(), 0);
      for (int unit = 0; unit < (1 << ub); ++unit)
        for (int g = 0; g < 32; ++g) {
          cd x[64], y[64];
          int at[64];
          for (int half = 0; half < 2; ++half)
            for (int k = 0; k < AH; ++k) {
              int32_t a = half ? op.half : 0;
              for (int j = 0; j < 5; ++j) a ^= ((g >> j) & 1) ? op.lane[j] : 0;
              for (int j = 0; j < ub; ++j) a ^= ((unit >> j) & 1) ? op.unit[j] : 0;
              for (int j = 0; j < K - 1; ++j) a ^= ((k >> j) & 1) ? op.c[j] : 0;
              CHECK(a >= 0 && a % 8 == 0 && a / 8 < (1 << S) && !hit[size_t(a / 8)]);
              hit[size_t(a / 8)] = 1;
              at[AH * half + k] = a / 8;
              cd v = lds[size_t(a / 8)];
              for (int q = 0; q < ntab; ++q) {
                const DevTab &d = tabs[tab0 + q];
                int32_t e = d.base | (half ? d.img[5] : 0);
                for (int j = 0; j < 5; ++j) e |= ((g >> j) & 1) ? d.img[j] : 0;
                for (int j = 0; j < K - 1; ++j) e |= ((k >> j) & 1) ? d.img[6 + j] : 0;
                for (int j = 0; j < ub; ++j) e |= ((unit >> j) & 1) ? d.img[11 + j] : 0;
                CHECK(e >= 0 && e % 8 == 0 && e / 8 < h.nblk * kTabBlock);
                v *= tab[size_t(e / 8)];
              }
              x[AH * half + k] = v;
            }
          for (int r = 0; r < D; ++r) {
            y[r] = 0;
            for (int c = 0; c < D; ++c) y[r] += M[size_t(r) * D + c] * x[c];
          }
          for (int r = 0; r < D; ++r) lds[size_t(at[r])] = y[r];
        }
    }
    for (int t = 0; t < (1 << ntb); ++t)
      for (int i = 0; i < (1 << cb); ++i)
        for (int b0 = 0; b0 < 2; ++b0) {
          const uint64_t l = uint64_t(b0) | (uint64_t(t) << 1) | (uint64_t(i) << (1 + ntb));
          cd v = lds[size_t(slot(l))];
          for (int q = 0; q < h.nstore; ++q) {
            const DevTab &d = stores[q];
            int32_t e = d.base | (b0 ? d.img[13] : 0);
            for (int j = 0; j < ntb; ++j) e |= ((t >> j) & 1) ? d.img[j] : 0;
            for (int j = 0; j < cb; ++j) e |= ((i >> j) & 1) ? d.img[9 + j] : 0;
            CHECK(e >= 0 && e % 8 == 0 && e / 8 < h.nblk * kTabBlock);
            v *= tab[size_t(e / 8)];
          }
          psi[phys(l)] = v;
        }
  }
}

int main(int argc, char **argv) {
  const int rounds = argc > 1 ? std::atoi(argv[1]) : 4;
  long fused_items = 0, all_items = 0, passes = 0;
  for (int n = 1; n <= 17; ++n)
    for (int round = 0; round < rounds; ++round)
      for (int prec : {SV_PREC_FP32, SV_PREC_BF16X3}) {
        std::mt19937_64 rng(uint64_t(1000 * n + 10 * round + prec));
        auto uni = [&](int lo, int hi) { return lo + int(rng() % uint64_t(hi - lo + 1)); };
        std::normal_distribution<double> nd;
        // round 0: diagonals only; 1: narrow gates on neighbours, as fused circuits have; else anything
        const int count = 24;
        std::vector<std::vector<double>> mats;
        std::vector<Item> items;
        for (int i = 0; i < count; ++i) {
          Item it;
          const int kmax = std::min(n, round == 1 ? 5 : 8);
          it.k = uni(1, kmax);
          it.diag = round == 0 || uni(0, 2) == 0;
          const bool exact = uni(0, 1);
          if (!it.diag && it.k > 6) it.k = std::min(n, 6);
          std::vector<int> q;
          const int start = uni(0, n - it.k);
          while (int(q.size()) < it.k) {
            const int b = round == 1 ? start + int(q.size()) : uni(0, n - 1);
            bool dup = false;
            for (int y : q) dup |= y == b;
            if (!dup) q.push_back(b);
          }
          for (int j = 0; j < it.k; ++j) it.A[j] = q[size_t(j)];
          const int D = 1 << it.k;
          std::vector<double> m(2 * size_t(D) * D, 0.0);
          for (int r = 0; r < D; ++r)
            for (int c = 0; c < D; ++c) {
              if (it.diag && r != c) continue;
              const double s = it.diag ? 1.0 : 1.0 / std::sqrt(2.0 * D);
              double re = nd(rng) * s, im = nd(rng) * s;
              if (it.diag && exact) {
                re = uni(0, 1) ? 1 : -1;
                im = 0;
                if (uni(0, 3) == 0) std::swap(re, im);
              } else if (it.diag) {
                const double a = std::hypot(re, im);
                re /= a;
                im /= a;
                if (uni(0, 1)) re = 1, im = 0;
              }
              m[2 * (size_t(r) * D + c)] = re;
              m[2 * (size_t(r) * D + c) + 1] = im;
            }
          mats.push_back(m);
          it.exact = it.diag && exact;
          it.sweep = it.diag ? 0.5 : 1.0;
          items.push_back(it);
        }
        for (int i = 0; i < count; ++i) items[size_t(i)].m = mats[size_t(i)].data();
        const std::vector<Step> steps = build_steps(n, items, prec);
        std::vector<char> seen(items.size(), 0);
        std::vector<cd> ref(size_t(1) << n), got;
        for (cd &a : ref) a = cd(nd(rng), nd(rng));
        got = ref;
        for (const Item &it : items) apply(ref, it);
        for (const Step &s : steps) {
          for (int i : s.items) {
            CHECK(i >= 0 && i < count && !seen[size_t(i)]);
            seen[size_t(i)] = 1;
          }
          all_items += long(s.items.size());
          if (s.pass.S == 0) {
            CHECK(s.items.size() == 1);
            apply(got, items[size_t(s.items[0])]);
          } else {
            CHECK(n >= kMinS);
            // BF16x3 states take exact diagonals only
            for (int i : s.items) CHECK(prec == SV_PREC_FP32 || items[size_t(i)].exact);
            CHECK(prec == SV_PREC_FP32 || s.pass.nops == 0);
            replay(got, n, s.pass);
            fused_items += long(s.items.size());
            ++passes;
          }
        }
        for (char c : seen) CHECK(c);
        double num = 0, den = 0;
        for (size_t x = 0; x < ref.size(); ++x) {
          num += std::norm(ref[x] - got[x]);
          den += std::norm(ref[x]);
        }
        const double rel = std::sqrt(num / den);
        // three bf16 pieces hold 24 bits or more of each gate entry and the tables are rounded to FP32:
        // at most 2^-24 per gate
        const double tol = count * 0x1p-23;
        if (!(rel <= tol)) {
          std::printf("n %d round %d prec %d: relative error %.3g > %.3g\n", n, round, prec, rel, tol);
          return 1;
        }
      }
  std::printf("%ld of %ld gates in %ld passes\npass checks passed\n", fused_items, all_items, passes);
  return 0;
}
