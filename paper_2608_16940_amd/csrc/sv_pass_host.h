// Fused tile passes, host side: a sequence of gates on physical bits is cut
// into passes, each of which reads and writes the state once and applies
// several gates to it while it sits in LDS.  Plain C++, no HIP; the kernel
// that runs a pass is in sv_pass.hip and reads the structures below.
#pragma once

#include <cstddef>
#include <cstdint>
#include <vector>

#include "sv.h"

namespace sv {
namespace pass {

// A pass owns tiles of 2^S amplitudes: the S tile bits sbit[0..S) in
// ascending physical order (local bit b <-> physical bit sbit[b]).  LDS holds
// the tile in local order, element l at slot(l) = l ^ (l >> 5 & 31) ^
// (l >> 10 & 31): linear over GF(2), so a slot is the XOR of the images of
// l's bits, and five tile bits whose numbers differ mod 5 reach 32 slots
// that lie on different banks.
constexpr int kMinS = 10;  // one 32-group unit of a five-bit gate
constexpr int kMaxS = 14;  // 128 KiB of the 160 KiB LDS
constexpr int kGateBits = 6;         // widest dense gate of a pass; narrower than five act as G (x) 1
constexpr int kMaxChunks = 16;       // operand chunks of a pass
constexpr int kTabEntries = 1024;    // diagonal table entries a pass holds in LDS (8 KiB)
constexpr int kTabBlock = 64;        // tables are loaded in blocks of one wave
constexpr int kTabInBits = 8;        // tile bits of one table
constexpr int kTabBits = 9;          // tile and tile-index bits of one table
constexpr int kTabOutMax = 11;

constexpr int32_t slot_image(int b) { return int32_t((1 << b) ^ (b >= 10 ? 1 << (b - 10) : (b >= 5 ? 1 << (b - 5) : 0))); }

// Device structures, 64 bytes each; images are byte offsets in LDS.
// A dense gate on five or six tile bits.  Lane l of a unit (32 groups of 32
// or 64 amplitudes) holds group l mod 32 and the half of its inputs with the
// top target bit equal to l / 32.
struct DevOp {
  int32_t lane[5], half, c[5], unit[4];  // slot images of the group's lane bits, the top target, the others, unit bits
  int32_t tab;                           // diagonal tables on its inputs: first | count << 16; bit 30: six bits
};
constexpr int32_t kOpSix = int32_t(1) << 30;
struct DevTab {  // one diagonal table at one place: index images of the bits that vary there
  int32_t base;  // byte offset of the table in the LDS table area
  int32_t img[15];
  // at a dense gate: lane[5], half, c[5], unit[4]; at the store: thread[9], chunk[4], bit 0
};
struct DevBlk {  // 64 table entries to load for a tile
  int32_t goff;  // first entry in the pass's table area, tile-index bits all zero
  int32_t nin;   // log2 of the table's entries per tile
  int32_t nout;  // tile-index bits selecting the part
  int32_t out[kTabOutMax];
  int32_t pad[2];
};
struct DevHead {
  int32_t nops, nblk, nstore, nchunks;
  int32_t ops, tabs, stores, blks;  // byte offsets from the head
  int32_t table, operand;           // likewise: the tables (float2), the gate operands
  int32_t pad[6];
  int32_t sbit[kMaxS], pad2[2];  // the tile bits
};
static_assert(sizeof(DevOp) == 64 && sizeof(DevTab) == 64 && sizeof(DevBlk) == 64 && sizeof(DevHead) == 128,
              "read with scalar loads of whole lines");

// A gate on physical bits.  m: 2^k x 2^k complex128 row-major, interleaved.
struct Item {
  int k = 0;
  int32_t A[8];
  const double *m = nullptr;
  bool diag = false;
  bool exact = false;  // diagonal with entries 1, -1, i, -i only
  double sweep = 1.0;  // share of a full sweep (plus launches) it costs on its own
  int launches = 1;    // on its own
};

struct Fused {
  int S = 0;
  int nops = 0;
  int nchunks = 0;
  int wide = 0;  // bits of the widest gate as the kernel runs it: 0, 5 or 6
  int sbit[kMaxS];
  std::vector<char> data;  // DevHead and what it points to
};

// One step of a sequence: the items it applies, in order; fused when pass.S > 0,
// else each item by its own sweep.
struct Step {
  std::vector<int> items;
  Fused pass;
};

// Cuts items into steps whose order is equivalent to the given one (gates
// move only past gates on other bits, and diagonals past diagonals), one step
// at a time: a caller launches a step while the next one is drafted and packed,
// and holds no more of them than it wants.  prec: SV_PREC_FP32 or
// SV_PREC_BF16X3; items outlive the cutter.
class Cutter {
 public:
  Cutter(int n, const std::vector<Item> &items, int prec);
  ~Cutter();
  Cutter(const Cutter &) = delete;
  Cutter &operator=(const Cutter &) = delete;
  bool next(Step *s);  // false when no step is left

 private:
  struct Draws;
  Draws *const d_;
};

// All steps of a sequence.
std::vector<Step> build_steps(int n, const std::vector<Item> &items, int prec);

// Operands come in chunks of this size: a five-bit gate is one chunk (two
// reduction steps of 16), a six-bit gate four (one step each, two row tiles).
constexpr size_t kChunkBytes = 6 * 2048;
inline int chunks_of(int k) { return k == 6 ? 4 : 1; }

// Bytes of device data a gate on k of n qubits adds to the passes of a
// sequence, at most: what it brings itself, and a pass that it is alone in (the
// head, a block that is always there, and the gaps to multiples of 256 bytes).
inline size_t share_bytes(int n, int k, bool diag, int prec) {
  if (n < kMinS || (!diag && (k > kGateBits || prec != SV_PREC_FP32))) return 0;
  const size_t pass = sizeof(DevHead) + sizeof(DevBlk) + 8 * kTabBlock + 3 * 256;
  if (!diag) return pass + sizeof(DevOp) + kChunkBytes * size_t(chunks_of(k));
  return pass + sizeof(DevTab) + sizeof(DevBlk) * (size_t(1) << kTabInBits) / kTabBlock +
         8 * ((size_t(1) << kTabBits) + kTabBlock);
}

}  // namespace pass
}  // namespace sv
