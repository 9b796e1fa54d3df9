// Gate programs (sv_prog_host.h) replayed in FP64 the way the kernel reads
// them, against the gates one by one.
#include <cmath>
#include <complex>
#include <cstdio>
#include <cstdlib>
#include <random>

#include "sv_prog_host.h"

using namespace sv;
typedef std::complex<double> cd;

static void fail(const char *what, int n, int seed) {
  std::printf("FAILED %s n=%d seed=%d\n", what, n, seed);
  std::exit(1);
}
#define CHECK(x) \
  if (!(x)) fail(#x, n, seed)

static void apply(std::vector<cd> &v, int n, const pass::Item &it) {
  const int D = 1 << it.k;
  std::vector<cd> in(D);
  uint64_t mask = 0;
  for (int j = 0; j < it.k; ++j) mask |= uint64_t(1) << it.A[j];
  for (uint64_t y = 0; y < v.size(); ++y) {
    if (y & mask) continue;
    auto at = [&](int r) {
      uint64_t x = y;
      for (int j = 0; j < it.k; ++j) x |= uint64_t(r >> j & 1) << it.A[j];
      return x;
    };
    for (int r = 0; r < D; ++r) in[r] = v[at(r)];
    for (int r = 0; r < D; ++r) {
      cd s = 0;
      for (int c = 0; c < D; ++c) s += cd(it.m[2 * (r * D + c)], it.m[2 * (r * D + c) + 1]) * in[c];
      v[at(r)] = s;
    }
  }
}

// one tile at a time: each layer on the whole tile
static void replay(std::vector<cd> &v, const prog::Args &a, int n, int seed) {
  CHECK(a.n == n && a.S == std::min(n, prog::kTileBits) && a.sbit[0] == 0);
  CHECK(a.ncode >= 2 && a.ncode <= prog::kMaxCode - prog::kCodeOver);
  CHECK(a.npay >= 0 && a.npay <= prog::kMaxPay - prog::kPayOver);
  for (int b = 0; b < a.S; ++b) CHECK(a.sbit[b] < n && (b == 0 || a.sbit[b] > a.sbit[b - 1]));
  for (uint64_t tile = 0; tile < uint64_t(1) << (n - a.S); ++tile) {
    uint64_t base = tile;
    for (int b = 0; b < a.S; ++b) {
      const int p = a.sbit[b];
      base = ((base >> p) << (p + 1)) | (base & ((uint64_t(1) << p) - 1));
    }
    auto phys = [&](int x) {
      uint64_t u = base;
      for (int b = 0; b < a.S; ++b) u |= uint64_t(x >> b & 1) << a.sbit[b];
      return u;
    };
    int reg[4] = {0}, off = 0, regs = 0;
    auto source = [&](uint32_t s, int l) {
      if (s & prog::kSrcOut) return int(base >> (s & 63) & 1);
      CHECK(!(s & prog::kSrcReg) && int(s) < a.S && !(regs >> s & 1));  // a thread's index, not a register bit
      return l >> s & 1;
    };
    for (int pc = 0; pc < a.ncode;) {
      const uint32_t w = a.code[pc++];
      CHECK(w != 0 && (pc > 1 || (w >> prog::kRound & 1)));
      if (w >> prog::kRound & 1) {
        const uint32_t c = a.code[pc++];
        CHECK((c >> 16) == (pc > 2));
        regs = 0;
        for (int j = 0; j < 4; ++j) {
          reg[j] = int(c >> (4 * j) & 15);
          CHECK(reg[j] < a.S && (j == 0 || reg[j] > reg[j - 1]));
          regs |= 1 << reg[j];
        }
      }
      for (int j = 0; j < 4; ++j) {
        if (!(w >> j & 1)) continue;
        const float *p = a.pay + off;
        off += 8;
        for (int l = 0; l < 1 << a.S; ++l) {
          const int m = 1 << reg[j];
          if (l & m) continue;
          const cd x = v[phys(l)], y = v[phys(l | m)];
          v[phys(l)] = cd(p[0], p[1]) * x + cd(p[2], p[3]) * y;
          v[phys(l | m)] = cd(p[4], p[5]) * x + cd(p[6], p[7]) * y;
        }
      }
      static const int pa[6][2] = {{0, 1}, {0, 2}, {0, 3}, {1, 2}, {1, 3}, {2, 3}};
      for (int j = 0; j < 6; ++j) {
        if (!(w >> (prog::kPairs + j) & 1)) continue;
        const cd e(a.pay[off], a.pay[off + 1]);
        off += 2;
        for (int l = 0; l < 1 << a.S; ++l)
          if ((l >> reg[pa[j][0]] & 1) && (l >> reg[pa[j][1]] & 1)) v[phys(l)] *= e;
      }
      auto classes = [&](uint32_t flags, auto bit0, auto bit1) {
        const float *p = a.pay + off;
        off += flags == 8 ? 2 : 8;
        for (int l = 0; l < 1 << a.S; ++l) {
          const int cls = bit0(l) | bit1(l) << 1;
          if (!(flags >> cls & 1)) continue;
          const float *e = flags == 8 ? p : p + 2 * cls;
          v[phys(l)] *= cd(e[0], e[1]);
        }
      };
      if (w >> prog::kOnes & 15) {
        for (int j = 0; j < 4; ++j) {
          const uint32_t h = a.code[pc + j / 2] >> (16 * (j & 1)) & 0xFFFF;
          if (w >> (prog::kOnes + j) & 1)
            classes(h >> 8 & 15, [&](int l) { return l >> reg[j] & 1; }, [&](int l) { return source(h & 127, l); });
        }
        pc += 2;
      }
      for (uint32_t z = 0; z < w >> prog::kFurther; ++z) {
        const uint32_t c = a.code[pc++];
        auto any = [&](uint32_t s) {
          return [&, s](int l) {
            if ((s & (prog::kSrcOut | prog::kSrcReg)) == prog::kSrcReg) return l >> reg[s & 3] & 1;
            return source(s, l);
          };
        };
        classes(c >> 14 & 15, any(c & 127), any(c >> 7 & 127));
      }
      CHECK(pc <= a.ncode && off <= a.npay);
    }
    CHECK(off == a.npay);
  }
}

int main() {
  for (int n = prog::kMinQubits; n <= 16; ++n)
    for (int seed = 0; seed < 8; ++seed) {
      std::mt19937 rng(unsigned(100 * n + seed));
      std::uniform_real_distribution<double> u(-1, 1);
      const int count = 1 + int(rng() % (seed < 4 ? 30 : 400));
      std::vector<std::vector<double>> mats;
      std::vector<pass::Item> items;
      mats.reserve(size_t(count));
      for (int g = 0; g < count; ++g) {
        pass::Item it;
        it.diag = seed == 7 || rng() % 2;
        it.k = it.diag ? 1 + int(rng() % 2) : 1;
        it.A[0] = int(rng() % unsigned(n));
        do it.A[1] = int(rng() % unsigned(n));
        while (it.A[1] == it.A[0]);
        const int D = 1 << it.k, ones = int(rng() % 16);
        std::vector<double> m(size_t(2 * D * D), 0.0);
        auto unit = [&](double w) {  // float-exact values: the replay holds the payload's floats
          const double x = double(float(w * std::cos(3 * u(rng)))), y = double(float(w * std::sin(3 * u(rng))));
          return cd(x, y);
        };
        for (int r = 0; r < D; ++r)
          for (int c = 0; c < D; ++c) {
            if (it.diag && r != c) continue;
            cd z = unit(0.7);
            if (it.diag && (ones >> r & 1)) z = 1.0;
            m[size_t(2 * (r * D + c))] = z.real();
            m[size_t(2 * (r * D + c) + 1)] = z.imag();
          }
        mats.push_back(m);
        it.m = mats.back().data();
        items.push_back(it);
      }
      std::vector<cd> want(size_t(1) << n), got;
      for (cd &z : want) z = cd(u(rng), u(rng));
      got = want;
      for (const pass::Item &it : items) apply(want, n, it);
      std::vector<prog::Step> steps;
      prog::build(n, items, &steps);
      size_t used = 0;
      std::vector<char> seen(items.size(), 0);
      for (const prog::Step &s : steps) {
        for (int i : s.items) {
          CHECK(!seen[size_t(i)]);
          seen[size_t(i)] = 1;
          ++used;
        }
        if (s.fused)
          replay(got, s.args, n, seed);
        else
          for (int i : s.items) apply(got, n, items[size_t(i)]);
      }
      CHECK(used == items.size());
      double err = 0, ref = 0;
      for (size_t i = 0; i < got.size(); ++i) {
        err += std::norm(got[i] - want[i]);
        ref += std::norm(want[i]);
      }
      CHECK(std::sqrt(err) <= 1e-12 * count * std::sqrt(ref));
    }
  std::printf("program checks passed\n");
  return 0;
}
