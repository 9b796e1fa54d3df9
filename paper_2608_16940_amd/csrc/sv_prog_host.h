// Gate programs, host side: runs of narrow gates (dense on one qubit, diagonal
// on one or two) are cut into passes.  A pass reads and writes the state once;
// a workgroup keeps a tile of it in LDS and runs the pass's program on it,
// sixteen amplitudes per thread in registers at a time.  Plain C++, no HIP;
// the kernel is in sv_prog.hip.
#pragma once

#include <cstdint>
#include <vector>

#include "sv_pass_host.h"

namespace sv {
namespace prog {

constexpr int kTileBits = 12;  // 32 KiB of LDS, 256 threads
constexpr int kRegBits = 4;    // tile bits a thread holds in registers during a round
constexpr int kMaxCode = 192;
constexpr int kMaxPay = 776;  // floats
constexpr int kPayOver = 8;   // floats that may be read past a layer's payload
constexpr int kCodeOver = 4;  // words that may be read past the program

// A program is a list of layers: dense gates on the four register bits, then
// diagonals.  A layer is one word, of bits
//   0..3   a dense 2x2 on register bit j (payload the matrix)
//   4..9   a phase on the all-ones class of register bits 01 02 03 12 13 23
//          (payload one entry)
//   10..13 a diagonal on register bit j and a source (a word's half each)
//   14     a round opens (one word: the register bits' tile bits, four bits
//          each, ascending; bit 16 from the second round on)
//   16..19 further diagonals (a word each)
// followed by the words of the round, the sources (two, if there is any) and
// the further diagonals; its payload has the same order.
// A source: bit number | kSrcOut where it is a physical bit of the tile's base
// and not a tile bit.  Its half word: source | flags << 8; the class of an
// amplitude is (register bit) | (source) << 1, and the flagged classes are
// multiplied by their entry.  Payload: four entries, or the entry of class 3
// alone where only that is flagged.
// A further diagonal: source | source << 7 | flags << 14, kSrcReg | position
// naming a register bit.
constexpr int kPairs = 4, kOnes = 10, kRound = 14, kFurther = 16;
constexpr int kMaxFurther = 15;
constexpr uint32_t kSrcOut = 64;
constexpr uint32_t kSrcReg = 32;
constexpr uint32_t kSrcZero = kSrcOut | 63;  // a bit no state has

// Travels as the kernel's arguments: nothing to copy or keep, also under capture.
struct Args {
  int32_t n, S, ncode, npay;
  int32_t sbit[16];  // tile bit -> physical bit, ascending
  uint32_t code[kMaxCode];
  float pay[kMaxPay];
};
static_assert(sizeof(Args) <= 4032, "kernel arguments");

constexpr int kMinQubits = kRegBits;

inline bool takes(const pass::Item &it) { return it.diag ? it.k <= 2 : it.k == 1; }

struct Step {
  std::vector<int> items;  // in the order they are applied
  bool fused = false;      // one pass running args; else each item by its own sweep
  Args args;
};

// Cuts items (all of them takes()) on n >= kMinQubits qubits into steps, in an
// order equivalent to the given one.
void build(int n, const std::vector<pass::Item> &items, std::vector<Step> *out);

}  // namespace prog
}  // namespace sv
