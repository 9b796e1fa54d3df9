// Gate chains, host side: a sequence of dense gates on four to six bits is cut
// into passes that read and write the state once and apply up to four of the
// gates in LDS, each with the arithmetic of its own FP32 sweep, bit for bit
// (density handles, whose FP64 outputs show every rounding).  Plain C++, no
// HIP; the kernel is in sv_chain.hip.
#pragma once

#include <algorithm>
#include <cstdint>
#include <vector>

#include "sv_pass_host.h"

namespace sv {
namespace chain {

constexpr int kTileBits = 13;  // 64 KiB of LDS, two workgroups per CU
// From here on chains win, also with tiles for a fraction of the CUs: four
// noisy layers in blocks of four qubits take 217 us in single sweeps and 190
// in chains at 18, 331 and 263 at 20 (at 14: 169 and 189).
constexpr int kMinQubits = 18;
constexpr int kMaxGates = 4;
// The lowest bits that every tile holds.  Whole cache lines (16 amplitudes) on
// states beyond the caches: blocks of four at 28 qubits 23.3 ms against 24.9
// with eight, 1.49 against 1.62 at 24; below, more gates per tile do more
// (blocks of six at 22: 591 us with eight, 626 with sixteen).
inline int low_bits(int n) { return n >= 24 ? 4 : 3; }

// Byte images in LDS (slot_image of sv_pass_host.h) of the bits that number a
// gate's groups and its inputs: lane 0..31 -> lane[], lane / 32 -> half (the
// top target), the other targets -> c[], units of 32 groups -> unit[].
struct Gate {
  int32_t K;
  int32_t lane[5], half, c[5], unit[5];
  int32_t op;  // byte offset of its operand
};

struct Step {
  std::vector<int> items;  // in the order they are applied
  bool fused = false;
  int32_t sbit[kTileBits];
  Gate gate[kMaxGates];
};

inline bool takes(const pass::Item &it) { return !it.diag && it.k >= 4 && it.k <= 6; }

inline std::vector<Step> build(int n, const std::vector<pass::Item> &items) {
  std::vector<Step> steps;
  std::vector<uint64_t> bits(items.size(), 0);
  for (size_t i = 0; i < items.size(); ++i)
    for (int j = 0; j < items[i].k; ++j) bits[i] |= uint64_t(1) << items[i].A[j];
  const uint64_t low = (uint64_t(1) << low_bits(n)) - 1;
  for (size_t from = 0; from < items.size(); ++from) {
    steps.emplace_back();
    Step &s = steps.back();
    s.items.push_back(int(from));
    if (n < kMinQubits || !takes(items[from])) continue;
    // the gates that follow, as long as they fit the tile: none passes another
    // one, not even on other bits, which would round in another order
    uint64_t tile = bits[from] | low;
    for (; from + 1 < items.size() && int(s.items.size()) < kMaxGates; ++from) {
      const size_t i = from + 1;
      if (!takes(items[i]) || __builtin_popcountll(tile | bits[i]) > kTileBits) break;
      tile |= bits[i];
      s.items.push_back(int(i));
    }
    if (s.items.size() < 2) continue;
    s.fused = true;
    for (int p = 0; __builtin_popcountll(tile) < kTileBits; ++p) tile |= uint64_t(1) << p;
    int local[64], nb = 0;
    for (int p = 0; p < n; ++p) {
      local[p] = -1;
      if ((tile >> p) & 1) {
        s.sbit[nb] = p;
        local[p] = nb++;
      }
    }
    for (size_t x = 0; x < s.items.size(); ++x) {
      const pass::Item &it = items[size_t(s.items[x])];
      Gate &g = s.gate[x];
      g = Gate{};
      g.K = it.k;
      uint32_t used = 0, res = 0;
      for (int j = 0; j < it.k; ++j) used |= 1u << local[it.A[j]];
      for (int j = 0; j + 1 < it.k; ++j) g.c[j] = 8 * pass::slot_image(local[it.A[j]]);
      g.half = 8 * pass::slot_image(local[it.A[it.k - 1]]);
      // lane bits: five others, of different residues mod 5 (different banks) where they exist
      int ng = 0;
      for (int round = 0; round < 2; ++round)
        for (int b = 0; b < kTileBits && ng < 5; ++b) {
          if ((used >> b) & 1 || (round == 0 && ((res >> (b % 5)) & 1))) continue;
          g.lane[ng++] = 8 * pass::slot_image(b);
          used |= 1u << b;
          res |= 1u << (b % 5);
        }
      int nu = 0;
      for (int b = 0; b < kTileBits; ++b)
        if (!((used >> b) & 1)) g.unit[nu++] = 8 * pass::slot_image(b);
    }
  }
  return steps;
}

}  // namespace chain
}  // namespace sv
