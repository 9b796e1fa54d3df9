// Cutting runs of narrow gates into tile programs (host only, no HIP types).
#include "sv_prog_host.h"

#include <algorithm>
#include <cstring>

namespace sv {
namespace prog {
namespace {

inline int popc(uint64_t x) { return __builtin_popcountll(x); }

// Two qubits, and the entry of the all-ones class alone differs from 1: a controlled phase.
bool last_only(const pass::Item &it) {
  const int D = 1 << it.k;
  for (int r = 0; r + 1 < D; ++r)
    if (it.m[2 * (size_t(r) * D + r)] != 1.0 || it.m[2 * (size_t(r) * D + r) + 1] != 0.0) return false;
  return it.k == 2 && (it.m[30] != 1.0 || it.m[31] != 0.0);
}

struct Builder {
  int n, S;
  uint64_t low, all;
  const std::vector<pass::Item> &items;
  std::vector<uint64_t> bits;
  std::vector<char> done;

  Builder(int n_, const std::vector<pass::Item> &it) : n(n_), S(std::min(n_, kTileBits)), items(it), done(it.size(), 0) {
    // Runs of four amplitudes on states that stay in the caches, of a cache
    // line (16) beyond: six brickwork layers take 82 against 79 us at n=20, 100
    // against 111 at 21, 158 against 155 at 22, 616 against 535 at 24 and 10.7
    // against 10.2 ms at 28 (runs of two: 811 us at 24).
    const int lowbits = n <= kTileBits ? n : (n <= 21 ? 2 : 4);
    low = (uint64_t(1) << lowbits) - 1;
    all = (uint64_t(1) << n) - 1;
    bits.reserve(it.size());
    for (const pass::Item &x : it) {
      uint64_t b = 0;
      for (int j = 0; j < x.k; ++j) b |= uint64_t(1) << x.A[j];
      bits.push_back(b);
    }
  }

  // The gates a pass takes from item `from` on: a gate joins unless a gate
  // left behind acts on its bits (diagonals pass diagonals) or its bit no
  // longer fits the tile.
  void draft(size_t from, std::vector<int> *d, uint64_t *tile) const {
    uint64_t t = low, block_dense = 0, block_diag = 0;
    int pay = 0;
    for (size_t i = from; i < items.size() && block_dense != all; ++i) {
      if (done[i]) continue;
      const pass::Item &it = items[i];
      const uint64_t b = bits[i];
      if (pay + 8 + kPayOver > kMaxPay) break;
      if (it.diag) {
        if (b & block_dense) {
          block_diag |= b;
          continue;
        }
      } else {
        if ((b & (block_dense | block_diag)) || popc(t | b) > S) {
          block_dense |= b;
          continue;
        }
        t |= b;
      }
      d->push_back(int(i));
      pay += it.diag && last_only(it) ? 2 : 8;
    }
    for (int p = 0; p < n && popc(t) < S; ++p) t |= uint64_t(1) << p;
    *tile = t;
  }

  struct Layer {
    int dense[kRegBits] = {-1, -1, -1, -1}, pair[6] = {-1, -1, -1, -1, -1, -1}, one[kRegBits] = {-1, -1, -1, -1};
    std::vector<int> further;
  };

  // The program of a draft; items that no longer fit are left (what is
  // emitted is closed under what it depends on).
  void emit(const std::vector<int> &d, uint64_t tile, Step *st) const {
    Args &a = st->args;
    a.n = n;
    a.S = S;
    int local[64];
    int nb = 0;
    for (int p = 0; p < 16; ++p) a.sbit[p] = 0;
    for (int p = 0; p < n; ++p) {
      local[p] = -1;
      if ((tile >> p) & 1) {
        a.sbit[nb] = p;
        local[p] = nb++;
      }
    }
    static const int pair_of[4][4] = {{0, 0, 1, 2}, {0, 0, 3, 4}, {0, 0, 0, 5}, {0, 0, 0, 0}};
    int code = 0, pay = 0;
    std::vector<int> left = d, later;
    std::vector<Layer> layers;
    while (!left.empty()) {
      // a gate takes at most two words (three with the round's) if it opens a layer of its own
      const int room = (kMaxCode - kCodeOver - 2 - code) / 3;
      if (room < 1) break;
      // the register bits: first come, as the tile's in the draft
      uint64_t reg = 0, block_dense = 0, block_diag = 0;
      for (int i : left) {
        const uint64_t b = bits[size_t(i)];
        if (items[size_t(i)].diag) {
          if (b & block_dense) block_diag |= b;
        } else if (!(b & (block_dense | block_diag)) && popc(reg | b) <= kRegBits) {
          reg |= b;
        } else {
          block_dense |= b;
        }
      }
      for (size_t x = 0; x < left.size() && popc(reg) < kRegBits; ++x)  // diagonals alone are left
        for (uint64_t b = bits[size_t(left[x])] & tile; b && popc(reg) < kRegBits; b &= b - 1) reg |= b & -b;
      for (int l = S - 1; l >= 0 && popc(reg) < kRegBits; --l) reg |= uint64_t(1) << a.sbit[l];
      int rl[kRegBits], rp[64], nr = 0;
      std::fill(rp, rp + n, -1);
      for (int l = 0; l < S; ++l)
        if ((reg >> a.sbit[l]) & 1) {
          rp[a.sbit[l]] = nr;
          rl[nr++] = l;
        }
      // bits a later gate of the draft mixes: a diagonal off the registers waits for one of them
      uint64_t mixed = 0;
      for (int i : left)
        if (!items[size_t(i)].diag && !(bits[size_t(i)] & reg)) mixed |= bits[size_t(i)];
      // gates of the round, each in the earliest layer its bits allow
      layers.clear();
      int first_dense[kRegBits] = {0, 0, 0, 0};  // the layer from which a dense gate may take the bit
      int first_diag[kRegBits] = {0, 0, 0, 0};
      block_dense = block_diag = 0;
      later.clear();
      int taken = 0;
      for (int i : left) {
        const uint64_t b = bits[size_t(i)];
        const pass::Item &it = items[size_t(i)];
        bool in = taken < room;
        if (it.diag) {
          in = in && !(b & block_dense) && ((b & reg) || !(b & mixed));
          if (!in) block_diag |= b;
        } else {
          in = in && !(b & (block_dense | block_diag)) && !(b & ~reg);
          if (!in) block_dense |= b;
        }
        if (!in) {
          later.push_back(i);
          continue;
        }
        ++taken;
        st->items.push_back(i);
        const int r0 = rp[it.A[0]], r1 = it.k == 2 ? rp[it.A[1]] : -1;
        size_t at;
        auto layer = [&](size_t x) -> Layer & {
          if (layers.size() <= x) layers.resize(x + 1);
          return layers[x];
        };
        if (!it.diag) {
          at = size_t(first_dense[r0]);
          layer(at).dense[r0] = i;
          first_dense[r0] = int(at) + 1;
          first_diag[r0] = int(at);
          continue;
        }
        const bool phase = last_only(it);
        at = size_t(std::max(r0 >= 0 ? first_diag[r0] : 0, r1 >= 0 ? first_diag[r1] : 0));
        for (;; ++at) {
          Layer &y = layer(at);
          if (r0 >= 0 && r1 >= 0 && phase) {
            int &slot = y.pair[pair_of[std::min(r0, r1)][std::max(r0, r1)]];
            if (slot >= 0) continue;
            slot = i;
          } else if ((r0 >= 0) != (r1 >= 0)) {
            int &slot = y.one[r0 >= 0 ? r0 : r1];
            if (slot >= 0) continue;
            slot = i;
          } else {
            if (y.further.size() == kMaxFurther) continue;
            y.further.push_back(i);
          }
          break;
        }
        for (int r : {r0, r1})
          if (r >= 0) first_dense[r] = std::max(first_dense[r], int(at) + 1);
      }
      auto source = [&](int p) {
        return rp[p] >= 0 ? (uint32_t(rp[p]) | kSrcReg) : local[p] >= 0 ? uint32_t(local[p]) : (uint32_t(p) | kSrcOut);
      };
      // entries by class: bit 0 <-> target x, bit 1 <-> the other
      auto entries = [&](const pass::Item &it, int x, uint32_t *flags) {
        const int D = 1 << it.k;
        float e[8] = {0};
        *flags = 0;
        for (int r = 0; r < D; ++r) {
          const double *z = it.m + 2 * (size_t(r) * D + size_t(r));
          const int cls = x ? ((r & 1) << 1 | (r >> 1)) : r;
          e[2 * cls] = float(z[0]);
          e[2 * cls + 1] = float(z[1]);
          if (z[0] != 1.0 || z[1] != 0.0) *flags |= 1u << cls;
        }
        if (*flags == 8) {
          a.pay[pay++] = e[6];
          a.pay[pay++] = e[7];
        } else {
          std::memcpy(a.pay + pay, e, sizeof(e));
          pay += 8;
        }
      };
      for (size_t x = 0; x < layers.size(); ++x) {
        const Layer &y = layers[x];
        uint32_t &w = a.code[code++];
        w = 0;
        if (x == 0) {
          w |= 1u << kRound;
          uint32_t c = code > 1 ? 1u << 16 : 0;  // registers of a round before to be stored
          for (int j = 0; j < kRegBits; ++j) c |= uint32_t(rl[j]) << (4 * j);
          a.code[code++] = c;
        }
        for (int j = 0; j < kRegBits; ++j)
          if (y.dense[j] >= 0) {
            w |= 1u << j;
            for (int z = 0; z < 8; ++z) a.pay[pay++] = float(items[size_t(y.dense[j])].m[z]);
          }
        for (int j = 0; j < 6; ++j)
          if (y.pair[j] >= 0) {
            w |= 1u << (kPairs + j);
            const double *m = items[size_t(y.pair[j])].m;
            a.pay[pay++] = float(m[30]);
            a.pay[pay++] = float(m[31]);
          }
        uint32_t half[kRegBits] = {0, 0, 0, 0}, flags = 0;
        for (int j = 0; j < kRegBits; ++j)
          if (y.one[j] >= 0) {
            w |= 1u << (kOnes + j);
            const pass::Item &it = items[size_t(y.one[j])];
            const int x1 = it.k == 2 && rp[it.A[1]] >= 0;
            entries(it, x1, &flags);
            half[j] = (it.k == 2 ? source(it.A[1 - x1]) : kSrcZero) | flags << 8;
          }
        if (w >> kOnes & 15) {
          a.code[code++] = half[0] | half[1] << 16;
          a.code[code++] = half[2] | half[3] << 16;
        }
        w |= uint32_t(y.further.size()) << kFurther;
        for (int i : y.further) {
          const pass::Item &it = items[size_t(i)];
          entries(it, 0, &flags);
          a.code[code++] = source(it.A[0]) | (it.k == 2 ? source(it.A[1]) : kSrcZero) << 7 | flags << 14;
        }
      }
      left.swap(later);
    }
    a.ncode = code;
    a.npay = pay;
  }
};

}  // namespace

void build(int n, const std::vector<pass::Item> &items, std::vector<Step> *out) {
  Builder B(n, items);
  std::vector<int> d;
  for (size_t from = 0; from < items.size();) {
    if (B.done[from]) {
      ++from;
      continue;
    }
    d.clear();
    uint64_t tile = 0;
    B.draft(from, &d, &tile);
    double alone = 0.0;
    for (int i : d) alone += items[size_t(i)].sweep;
    out->emplace_back();
    Step &s = out->back();
    // A pass costs little more than a sweep (n=28: 0.78 ms for two to eight
    // dense gates, 0.66 for a sweep of one; n=20: 8 against 4 us), so two
    // gates are enough.  Large states' controlled phases visit a quarter each:
    // two of them are cheaper alone (0.49 ms), four are not (0.97).
    if (d.size() == 1 || (n > 24 && alone < 0.8)) {
      s.items = d;
    } else {
      s.fused = true;
      B.emit(d, tile, &s);
    }
    for (int i : s.items) B.done[size_t(i)] = 1;
  }
}

}  // namespace prog
}  // namespace sv
