// Gate programs for gfx950: a run of one-qubit gates and one- and two-qubit
// diagonals in one pass over the state (sv_prog_host.h cuts the passes).
//
// A workgroup owns a tile of 2^S amplitudes in LDS.  A round puts four tile
// bits into registers (16 amplitudes per thread, 2^(S-4) threads), applies the
// round's layers there and writes back in place, so a round costs one LDS read,
// one write and one barrier however many gates it holds.  The arithmetic is
// FP32, as in a gate's own sweep.
//
// Bound by the vector units once a pass holds a few gates: a dense gate is 16
// multiply-adds per pair of amplitudes, 0.21 us on a CU that holds a 2^12 tile
// (one wave per SIMD), and takes 0.29 in a full layer.  The 2^12 tile fills 256
// CUs from n=20 on; wider ones would hold more gates per pass but leave CUs idle
// there.  590 gates of a 20-qubit circuit: 3.86 ms one launch each, 0.26 ms in 7
// passes; 140 gates on 12 qubits: 0.94 ms and 51 us.
#include <algorithm>

#include "sv_internal.h"
#include "sv_prog.h"

#define LIKELY(x) __builtin_expect(!!(x), 1)

namespace sv {
namespace prog {
namespace {

constexpr int kR = 1 << kRegBits;
constexpr int kThreadsMax = 1 << (kTileBits - kRegBits);

__device__ __forceinline__ int slot_of(int l) { return l ^ ((l >> 5) & 31) ^ (l >> 10); }

__device__ __forceinline__ float2 mul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}
// a b + c into a register of its own: as a two-operand form it would land on
// c's, and every amplitude would be copied back after each gate
__device__ __forceinline__ float fma3(float a, float b, float c) {
  float d;
  asm("v_fma_f32 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}
__device__ __forceinline__ float fms3(float a, float b, float c) {  // c - a b
  float d;
  asm("v_fma_f32 %0, -%1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
  return d;
}

template <int J>
__device__ __forceinline__ void dense(float2 (&x)[kR], const float2 (&m)[4]) {
#pragma unroll
  for (int i = 0; i < kR; ++i)
    if (!(i >> J & 1)) {
      // inputs one after the other over all four outputs, so that the last
      // step can write where the first inputs were
      const float2 a = x[i], b = x[i | 1 << J];
      float2 o0 = make_float2(m[0].x * a.x, m[0].y * a.x), o1 = make_float2(m[2].x * a.x, m[2].y * a.x);
      o0 = make_float2(o0.x - m[0].y * a.y, o0.y + m[0].x * a.y);
      o1 = make_float2(o1.x - m[2].y * a.y, o1.y + m[2].x * a.y);
      o0 = make_float2(o0.x + m[1].x * b.x, o0.y + m[1].y * b.x);
      o1 = make_float2(o1.x + m[3].x * b.x, o1.y + m[3].y * b.x);
      x[i].x = fms3(m[1].y, b.y, o0.x);
      x[i].y = fma3(m[1].x, b.y, o0.y);
      x[i | 1 << J].x = fms3(m[3].y, b.y, o1.x);
      x[i | 1 << J].y = fma3(m[3].x, b.y, o1.y);
    }
}

// amplitudes whose register bits under MASK read VAL
template <int MASK, int VAL>
__device__ __forceinline__ void scale(float2 (&x)[kR], float2 f) {
#pragma unroll
  for (int i = 0; i < kR; ++i)
    if ((i & MASK) == VAL) x[i] = mul(f, x[i]);
}
// the same in the lanes where `on`
template <int MASK, int VAL>
__device__ __forceinline__ void scale(float2 (&x)[kR], float2 f, bool on) {
#pragma unroll
  for (int i = 0; i < kR; ++i)
    if ((i & MASK) == VAL) {
      const float2 y = mul(f, x[i]);
      x[i] = make_float2(on ? y.x : x[i].x, on ? y.y : x[i].y);
    }
}

// a diagonal on register bit J and a source of value `hi`; h: flags << 8
template <int J>
__device__ __forceinline__ void one(float2 (&x)[kR], uint32_t h, bool hi, const float2 **pay) {
  const uint32_t flags = h >> 8 & 15, f = hi ? flags >> 2 : flags;
  const float2 *p = *pay;
  const float2 e0 = p[0], e1 = p[1], e2 = p[2], e3 = flags == 8 ? e0 : p[3];
  *pay += flags == 8 ? 1 : 4;
  if (flags & 5) scale<1 << J, 0>(x, hi ? e2 : e0, f & 1);
  if (flags & 10) scale<1 << J, 1 << J>(x, hi ? e3 : e1, f & 2);
}

typedef const Args __attribute__((address_space(4))) *ArgsPtr;

__global__ __launch_bounds__(kThreadsMax) void k_prog(const Args by_value, float4 *__restrict__ psi4) {
  __shared__ float2 tile[1 << kTileBits];
  __shared__ __attribute__((aligned(16))) uint32_t words[sizeof(Args) / 4];
  ArgsPtr a = (ArgsPtr)__builtin_amdgcn_kernarg_segment_ptr();
  for (int i = threadIdx.x; i < int(sizeof(Args) / 4); i += blockDim.x)
    words[i] = ((const uint32_t __attribute__((address_space(4))) *)a)[i];
  const Args *prog = reinterpret_cast<const Args *>(words);
  // Below ten tile bits there are fewer threads' worth than a wave has lanes:
  // the others repeat them, in step with them, so that no branch diverges.
  const int S = a->S, T = 1 << (S - kRegBits), tid = threadIdx.x & (T - 1);
  uint64_t base = blockIdx.x;   // the tile's physical index, tile bits zero
  for (int b = 0; b < S; ++b) {
    const int p = a->sbit[b];
    base = ((base >> p) << (p + 1)) | (base & ((uint64_t(1) << p) - 1));
  }
  // load: 16-byte chunks, the thread number in the low chunk bits
  uint64_t tphys = base;
  for (int b = 0; b < S - kRegBits; ++b) tphys |= uint64_t(tid >> b & 1) << a->sbit[b + 1];
  const int tslot = slot_of(2 * tid);
  auto chunk_phys = [&](int c) {
    uint64_t u = tphys;
    for (int b = 0; b < kRegBits - 1; ++b) u |= uint64_t(c >> b & 1) << a->sbit[S - kRegBits + 1 + b];
    return u >> 1;
  };
  float4 v[kR / 2];
#pragma unroll
  for (int c = 0; c < kR / 2; ++c) v[c] = psi4[chunk_phys(c)];
#pragma unroll
  for (int c = 0; c < kR / 2; ++c) {
    const int s = tslot ^ slot_of(c << (S - kRegBits + 1));
    tile[s] = make_float2(v[c].x, v[c].y);
    tile[s ^ 1] = make_float2(v[c].z, v[c].w);
  }
  __syncthreads();

  float2 x[kR];
#pragma unroll
  for (int i = 0; i < kR; ++i) x[i] = make_float2(0.f, 0.f);
  int lbase = 0, sbase = 0;  // the thread's local index and slot, register bits zero
  int im[kRegBits] = {0, 0, 0, 0};
  auto slot = [&](int i) {
    int s = sbase;
#pragma unroll
    for (int j = 0; j < kRegBits; ++j)
      if (i >> j & 1) s ^= im[j];
    return s;
  };
  auto store = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kR; ++i) tile[slot(i)] = x[i];
    __syncthreads();
  };
  // value of a source that is no register bit
  auto source = [&](uint32_t src) {
    return (src & kSrcOut) ? int(base >> (src & 63) & 1) : (lbase >> (src & 31) & 1);
  };
  const float2 *pay = reinterpret_cast<const float2 *>(prog->pay);
  const int ncode = a->ncode;
  uint32_t nw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) nw[i] = prog->code[i];
  for (int pc = 0; pc < ncode;) {
    uint32_t w = uint32_t(__builtin_amdgcn_readfirstlane(int(nw[0])));
    const uint32_t w1 = uint32_t(__builtin_amdgcn_readfirstlane(int(nw[1])));
    const uint32_t w2 = uint32_t(__builtin_amdgcn_readfirstlane(int(nw[2])));
    const uint32_t w3 = uint32_t(__builtin_amdgcn_readfirstlane(int(nw[3])));
    const int opens = int(w >> kRound & 1);
    int further = int(w >> kFurther);
    pc += 1 + opens + ((w >> kOnes & 15) ? 2 : 0) + further;
#pragma unroll
    for (int i = 0; i < 4; ++i) nw[i] = prog->code[pc + i];
    // the layer's matrices and phases; absent ones read what comes next
    float2 m[kRegBits][4], ph[6];
#pragma unroll
    for (int j = 0; j < kRegBits; ++j) {
#pragma unroll
      for (int i = 0; i < 4; ++i) m[j][i] = pay[i];
      pay += (w >> j & 1) * 4;
    }
#pragma unroll
    for (int j = 0; j < 6; ++j) {
      ph[j] = pay[0];
      pay += w >> (kPairs + j) & 1;
    }
    if (opens) {
      if (w1 >> 16) store();
      lbase = tid;
#pragma unroll
      for (int j = 0; j < kRegBits; ++j) {
        const int b = int(w1 >> (4 * j) & 15);
        lbase = (lbase >> b << (b + 1)) | (lbase & ((1 << b) - 1));
        im[j] = slot_of(1 << b);
      }
      sbase = slot_of(lbase);
#pragma unroll
      for (int i = 0; i < kR; ++i) x[i] = tile[slot(i)];
    }
    // the tests as independent ones, bodies in line: a switch over cases (or
    // tests that the compiler sees to exclude each other) became two-sided
    // branches that copy all amplitudes at every join, and a lone wave pays
    // about 70 cycles for every branch it takes
    asm("" : "+s"(w));
    if (LIKELY(w & 1)) dense<0>(x, m[0]);
    if (LIKELY(w & 2)) dense<1>(x, m[1]);
    if (LIKELY(w & 4)) dense<2>(x, m[2]);
    if (LIKELY(w & 8)) dense<3>(x, m[3]);
    if (LIKELY(w & 63u << kPairs)) {
      if (LIKELY(w & 1u << kPairs)) scale<3, 3>(x, ph[0]);
      if (LIKELY(w & 8u << kPairs)) scale<6, 6>(x, ph[3]);
      if (LIKELY(w & 32u << kPairs)) scale<12, 12>(x, ph[5]);
      if (w & 22u << kPairs) {
        if (w & 2u << kPairs) scale<5, 5>(x, ph[1]);
        if (w & 4u << kPairs) scale<9, 9>(x, ph[2]);
        if (w & 16u << kPairs) scale<10, 10>(x, ph[4]);
      }
    }
    if (LIKELY(w & 15u << kOnes)) {
      const uint32_t h01 = opens ? w2 : w1, h23 = opens ? w3 : w2;
      if (w & 1u << kOnes) one<0>(x, h01, source(h01 & 127), &pay);
      if (w & 2u << kOnes) one<1>(x, h01 >> 16, source(h01 >> 16 & 127), &pay);
      if (w & 4u << kOnes) one<2>(x, h23, source(h23 & 127), &pay);
      if (w & 8u << kOnes) one<3>(x, h23 >> 16, source(h23 >> 16 & 127), &pay);
    }
    for (int z = 0; z < further; ++z) {
      const uint32_t c = uint32_t(__builtin_amdgcn_readfirstlane(int(prog->code[pc - further + z])));
      const uint32_t s0 = c & 127, s1 = c >> 7 & 127, flags = c >> 14 & 15;
      // register bits by amplitude number, other sources for all at once
      constexpr uint32_t kBit[4] = {0xAAAA, 0xCCCC, 0xF0F0, 0xFF00};
      auto isreg = [](uint32_t s) { return (s & (kSrcOut | kSrcReg)) == kSrcReg; };
      auto pattern = [&](uint32_t s) {
        const uint32_t j = s & 3;
        return j & 2 ? (j & 1 ? kBit[3] : kBit[2]) : (j & 1 ? kBit[1] : kBit[0]);
      };
      const uint32_t v0 = isreg(s0) ? pattern(s0) : (source(s0) ? 0xFFFFu : 0u);
      const uint32_t v1 = isreg(s1) ? pattern(s1) : (source(s1) ? 0xFFFFu : 0u);
      const float2 e0 = pay[0], e1 = pay[1], e2 = pay[2], e3 = flags == 8 ? e0 : pay[3];
      pay += flags == 8 ? 1 : 4;
#pragma unroll
      for (int i = 0; i < kR; ++i) {
        const bool b0 = v0 >> i & 1, b1 = v1 >> i & 1;
        const float2 f = b1 ? (b0 ? e3 : e2) : (b0 ? e1 : e0);
        const float2 y = mul(f, x[i]);
        const bool on = flags >> (int(b0) | int(b1) << 1) & 1;
        x[i] = make_float2(on ? y.x : x[i].x, on ? y.y : x[i].y);
      }
    }
  }
  store();
#pragma unroll
  for (int c = 0; c < kR / 2; ++c) {
    const int s = tslot ^ slot_of(c << (S - kRegBits + 1));
    const float2 u = tile[s], w = tile[s ^ 1];
    psi4[chunk_phys(c)] = make_float4(u.x, u.y, w.x, w.y);
  }
}

}  // namespace

hipError_t launch(const Args &a, float2 *psi, hipStream_t st) {
  if (a.S < kRegBits || a.S > kTileBits || a.S > a.n || a.n - a.S > 23 || a.ncode < 2 ||
      a.ncode > kMaxCode - kCodeOver || a.npay > kMaxPay - kPayOver || a.sbit[0] != 0)
    return hipErrorInvalidValue;
  const int threads = std::max(64, 1 << (a.S - kRegBits));
  hipLaunchKernelGGL(k_prog, dim3(1u << (a.n - a.S)), dim3(threads), 0, st, a, reinterpret_cast<float4 *>(psi));
  return hipGetLastError();
}

}  // namespace prog
}  // namespace sv
