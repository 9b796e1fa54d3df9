// Fused tile passes for gfx950: several gates applied to a tile of the state
// while it sits in LDS, with one read and one write of the state.
//
// A workgroup owns tiles of 2^S amplitudes (the tile bits are chosen by
// sv_pass_host.cpp so that every dense gate of the pass acts inside the
// tile).  Per tile: the amplitudes land in LDS; each dense gate (five tile
// bits; narrower ones act as G (x) 1) multiplies the tile's groups of 32
// amplitudes on the matrix cores, in place; diagonal factors are table
// lookups applied to a gate's inputs or to the amplitudes on their way out,
// whatever bits they act on -- the bits outside the tile select the part of
// the table that the tile loads.
//
// Arithmetic of a dense gate: Re y = Gr Xr - Gi Xi, Im y = Gi Xr + Gr Xi on
// v_mfma_f32_32x32x16_bf16 with FP32 accumulation, both operands in three
// bf16 pieces (hi + mid + lo holds all 24 bits of the significand) and the six
// products down to 2^-16 of the leading one; the three dropped ones lie below
// 2^-25.  Against 64 bits a plan run this way is nearer than with the FP32
// matrix instructions' three-product form (N=23, 12 brickwork layers: 7e-7
// against 1.1e-6), which also take twice the time.
#include <algorithm>
#include <type_traits>

#include "sv_internal.h"
#include "sv_pass.h"

// Lambdas of the kernel that are used more than once must not become calls.
#define SV_INLINE __attribute__((always_inline))

namespace sv {
namespace pass {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ floatx16 mfma(uint4 a, uint4 b, floatx16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0,
                                                  0, 0);
}

__device__ __forceinline__ int64_t insert_zero_bit(int64_t x, int p) {
  const int64_t low = x & ((int64_t(1) << p) - 1);
  return ((x >> p) << (p + 1)) | low;
}

// bf16 pair (round to nearest even), a in the low half
__device__ __forceinline__ uint32_t pk(float a, float b) {
  const floatx2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float pk_lo(uint32_t p) { return __uint_as_float(p << 16); }
__device__ __forceinline__ float pk_hi(uint32_t p) { return __uint_as_float(p & 0xFFFF0000u); }

constexpr int PIECES = 3;  // x = hi + mid + lo, each difference exact in FP32

__device__ __forceinline__ float flip_by(float x, uint32_t m) { return __uint_as_float(__float_as_uint(x) ^ m); }

__device__ __forceinline__ float2 cmul(float2 d, float2 x) {
  return make_float2(d.x * x.x - d.y * x.y, d.x * x.y + d.y * x.x);
}

// Memory that no kernel writes while this one runs, for wave-uniform reads.
template <class T>
using Const = const __attribute__((address_space(4))) T;
template <class T>
__device__ __forceinline__ Const<T> *constant(const char *p) {
  return (Const<T> *)(reinterpret_cast<uintptr_t>(p));
}

// Slot image of input k of a lane's sixteen or 32.
__device__ __forceinline__ int32_t op_slot(Const<DevOp> &op, int k) {
  int32_t a = 0;
#pragma unroll
  for (int j = 0; j < 5; ++j)
    if ((k >> j) & 1) a ^= op.c[j];
  return a;
}

template <int S>
struct Cfg {
  static constexpr int NW = 1 << (S - 10 < 3 ? S - 10 : 3);  // waves
  static constexpr int NT = 64 * NW;
  static constexpr int NTB = 6 + (S - 10 < 3 ? S - 10 : 3);  // thread bits
  static constexpr int CHUNKS = (1 << (S - 1)) / NT;          // 16-byte chunks per thread
  static constexpr int UNITS = (1 << (S - 10)) / NW;          // 32-group units per wave
  static constexpr int BLKS = kTabEntries / kTabBlock / NW;   // table blocks per wave
};

// WIDE: the widest gate, 0 for a pass of diagonal factors alone (a pass
// without six-bit gates gets by without spills).
template <int S, int WIDE>
__global__ __launch_bounds__(Cfg<S>::NT, 2) void k_pass(float2 *__restrict__ psi, const char *__restrict__ data,
                                                        int64_t ntiles) {
  using C = Cfg<S>;
  constexpr bool GATES = WIDE > 0;
  constexpr int OPB = kChunkBytes;
  __shared__ __attribute__((aligned(16))) char lds[8 << S];
  __shared__ __attribute__((aligned(16))) char opl[GATES ? 2 * OPB : 16];
  __shared__ __attribute__((aligned(16))) char tabl[8 * kTabEntries];

  // the descriptors are constant for the launch and read wave-uniformly: scalar loads
  const auto *head = constant<DevHead>(data);
  const auto *ops = constant<DevOp>(data + head->ops);
  const auto *tabs = constant<DevTab>(data + head->tabs);
  const auto *stores = constant<DevTab>(data + head->stores);
  const auto *blks = constant<DevBlk>(data + head->blks);
  const float2 *__restrict__ table = reinterpret_cast<const float2 *>(data + head->table);
  const char *__restrict__ operand = data + head->operand;
  const int nops = head->nops, nblk = head->nblk, nstore = head->nstore, nchunks = head->nchunks;

  const int t = threadIdx.x;
  const int lane = t & 63;
  const int wave = __builtin_amdgcn_readfirstlane(t >> 6);

  // of the two waves a SIMD holds, one leads: its vector work then runs under
  // the other's matrix work instead of beside it (4-gate passes 4% faster)
  if (wave < C::NW / 2) __builtin_amdgcn_s_setprio(2);

  // this thread's share of a tile: chunk i covers local bits 1.. of
  // (t | i << NTB), bit 0 inside the chunk
  int64_t goff_t = 0;
  int32_t slot_t = 0;
#pragma unroll
  for (int b = 0; b < C::NTB; ++b) {
    const int on = (t >> b) & 1;
    goff_t |= int64_t(on) << head->sbit[1 + b];
    slot_t ^= on * (8 * slot_image(1 + b));
  }
  float2 *const psi_t = psi + goff_t;
  // The tile bits are read again at each use: kept in scalar registers across
  // the gates they crowd out the rest (100 of them spilled).
  auto fresh = [&]() SV_INLINE {
    const auto *h = head;
    asm volatile("" : "+s"(h));
    return h;
  };
  auto goff = [](const auto *h, int i) SV_INLINE {
    int64_t o = 0;
#pragma unroll
    for (int b = 0; (1 << b) < C::CHUNKS; ++b)
      if ((i >> b) & 1) o |= int64_t(1) << h->sbit[1 + C::NTB + b];
    return o;
  };
  auto slot = [&](int i) SV_INLINE {
    int32_t s = 0;
#pragma unroll
    for (int b = 0; (1 << b) < C::CHUNKS; ++b)
      if ((i >> b) & 1) s ^= 8 * slot_image(1 + C::NTB + b);
    return slot_t ^ s;
  };
  auto tile_base = [&](int64_t tl) SV_INLINE {
    const auto *h = fresh();
    int64_t b0 = tl;
#pragma unroll
    for (int b = 0; b < S; ++b) b0 = insert_zero_bit(b0, h->sbit[b]);
    return b0;
  };

  // operand chunk o: global -> registers, then -> LDS buffer `buf`
  constexpr int OPC = OPB / 8 / C::NT;
  static_assert(OPC * C::NT * 8 == OPB, "whole steps");
  floatx2 ov[OPC];
  auto load_operand = [&](int o) SV_INLINE {
    const floatx2 *src = reinterpret_cast<const floatx2 *>(operand + int64_t(o) * OPB);
#pragma unroll
    for (int i = 0; i < OPC; ++i) ov[i] = src[i * C::NT + t];
  };
  auto put_operand = [&](int buf) SV_INLINE {
    floatx2 *dst = reinterpret_cast<floatx2 *>(opl + buf * OPB);
#pragma unroll
    for (int i = 0; i < OPC; ++i) dst[i * C::NT + t] = ov[i];
  };

  // table blocks of a tile, likewise (a wave without a block re-reads block 0)
  float2 tv[C::BLKS];
  auto load_tables = [&](int64_t base) SV_INLINE {
#pragma unroll
    for (int j = 0; j < C::BLKS; ++j) {
      const int b = j * C::NW + wave;
      Const<DevBlk> &k = blks[b < nblk ? b : 0];
      int64_t part = 0;
      for (int q = 0; q < k.nout; ++q) part |= ((base >> k.out[q]) & 1) << q;
      tv[j] = table[k.goff + (part << k.nin) + lane];
    }
  };
  auto put_tables = [&]() SV_INLINE {
#pragma unroll
    for (int j = 0; j < C::BLKS; ++j)
      if (j * C::NW + wave < nblk)
        *reinterpret_cast<float2 *>(tabl + 8 * ((j * C::NW + wave) * kTabBlock + lane)) = tv[j];
  };

  floatx4 v[C::CHUNKS];  // the thread's chunks of the next tile on their way in
  auto load_chunks = [&](int64_t base) SV_INLINE {
    const auto *h = fresh();
#pragma unroll
    for (int i = 0; i < C::CHUNKS; ++i)
      v[i] = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(psi_t + (base + goff(h, i))));
  };
  auto put_chunks = [&]() SV_INLINE {
#pragma unroll
    for (int i = 0; i < C::CHUNKS; ++i) {
      *reinterpret_cast<float2 *>(lds + slot(i)) = make_float2(v[i].x, v[i].y);
      *reinterpret_cast<float2 *>(lds + (slot(i) ^ 8)) = make_float2(v[i].z, v[i].w);
    }
  };

  // Sign of a group.  The matrix cores round an accumulation slightly
  // downwards (measured: a mean error of -5e-10 of the amplitudes' rms per
  // gate, against 2e-7 of noise), the same way for every group, and a later
  // QFT or Hadamard layer gathers such a constant into one amplitude (the
  // zero frequency of a 30-qubit QFT was off by 7e-4 of the rms).  Half of
  // the groups therefore go through negated, in the pattern of the
  // Rudin-Shapiro sequence over the group and tile index, whose spectrum is
  // flat, so that no transform can gather it.
  auto rs = [](uint32_t z) SV_INLINE -> uint32_t { return uint32_t(__popc(z & (z >> 1)) & 1) << 31; };

  // ---- gates.  A unit is 32 groups; lane l holds group l mod 32 and half of
  // its inputs.  Vector and matrix instructions of one wave overlap when they
  // are neighbours in its instruction stream, so the splitting of the next
  // eight inputs is laid between the matrix instructions of the current ones
  // (an N=28 pass spends 0.26 ms per five-bit gate, 0.29 with the two apart;
  // the matrix instructions alone need 0.19).
  struct Half {  // eight inputs of a lane in pieces
    uint32_t r[4][PIECES], i[4][PIECES];
  };
  constexpr int NS = 8 * PIECES;                 // steps of splitting eight inputs
  constexpr int NP = 2 * PIECES * (PIECES + 1);  // matrix instructions of a reduction step and row tile
  float ra, rb;  // the pair of reals being split: one pair in PIECES steps
  auto split_step = [&](Half &h, const float2 *x, uint32_t flip, int i, int held = 8) SV_INLINE {  // x: `held` inputs at a time
    const int pair = i / PIECES, piece = i % PIECES, q = pair >> 1, at = (2 * q) & (held - 1);
    if (piece == 0) {
      ra = flip_by((pair & 1) ? x[at].y : x[at].x, flip);
      rb = flip_by((pair & 1) ? x[at + 1].y : x[at + 1].x, flip);
    }
    const uint32_t w = pk(ra, rb);
    ((pair & 1) ? h.i[q] : h.r[q])[piece] = w;
    if (piece + 1 < PIECES) {
      ra -= pk_lo(w);
      rb -= pk_hi(w);
    }
  };
  auto read8 = [&](Const<DevOp> &op, float2 *x, int32_t s0, int s) SV_INLINE {
#pragma unroll
    for (int k = 0; k < 8; ++k) x[k] = *reinterpret_cast<const float2 *>(lds + (s0 ^ op_slot(op, 8 * s + k)));
  };
  auto read4 = [&](Const<DevOp> &op, float2 *x, int32_t s0, int s) SV_INLINE {
#pragma unroll
    for (int k = 0; k < 4; ++k) x[k] = *reinterpret_cast<const float2 *>(lds + (s0 ^ op_slot(op, 4 * s + k)));
  };
  // One reduction step of one row tile, small products first; block(P) is the
  // 1 KiB operand block of plane P, under(i) the vector work that goes beside
  // matrix instruction i (the scheduling barriers keep it there).
  auto products = [&](floatx16 &re, floatx16 &im, const Half &h, auto block, auto under) SV_INLINE {
    int i = 0;
#pragma unroll
    for (int w = PIECES - 1; w >= 0; --w)
#pragma unroll
      for (int ga = 0; ga <= w; ++ga) {
        const int xa = w - ga;
        const uint4 gr = *reinterpret_cast<const uint4 *>(block(ga) + lane * 16);
        const uint4 gi = *reinterpret_cast<const uint4 *>(block(PIECES + ga) + lane * 16);
        const uint4 br = make_uint4(h.r[0][xa], h.r[1][xa], h.r[2][xa], h.r[3][xa]);
        const uint4 bi = make_uint4(h.i[0][xa], h.i[1][xa], h.i[2][xa], h.i[3][xa]);
        re = mfma(gr, br, re);
        under(i++);
        __builtin_amdgcn_sched_barrier(0);
        im = mfma(gi, br, im);
        under(i++);
        const uint4 nbi = make_uint4(bi.x ^ 0x80008000u, bi.y ^ 0x80008000u, bi.z ^ 0x80008000u, bi.w ^ 0x80008000u);
        __builtin_amdgcn_sched_barrier(0);
        re = mfma(gi, nbi, re);
        under(i++);
        __builtin_amdgcn_sched_barrier(0);
        im = mfma(gr, bi, im);
        under(i++);
        __builtin_amdgcn_sched_barrier(0);
      }
  };
  auto clear = [](floatx16 &a) SV_INLINE {
#pragma unroll
    for (int r = 0; r < 16; ++r) a[r] = 0.f;
  };
  // Slot and sign of this lane's group in `unit` (UB unit bits).
  auto unit_slot = [&](Const<DevOp> &op, int unit, int UB) SV_INLINE {
    int32_t s0 = op.half & -(lane >> 5);
#pragma unroll
    for (int j = 0; j < 5; ++j) s0 ^= op.lane[j] & -((lane >> j) & 1);
#pragma unroll
    for (int j = 0; j < 4; ++j)
      if (j < UB) s0 ^= op.unit[j] & -((unit >> j) & 1);
    return s0;
  };
  auto unit_flip = [&](int unit, int UB, uint32_t tile_no) SV_INLINE {
    const uint32_t z = uint32_t(unit) | (tile_no << UB);
    int l = lane;
    asm volatile("" : "+v"(l));  // formed at each use, not kept
    return rs(uint32_t(l & 31)) ^ rs(z) ^ (uint32_t(lane & 16) << 27 & (z << 31));
  };
  // Diagonal tables on sixteen of a lane's inputs, in place (every lane its own slots).
  auto apply_tables = [&](Const<DevOp> &op, int32_t s0, int unit, int UB, int part) SV_INLINE {
    const int ntab = op.tab >> 16 & 0xFF, tab0 = op.tab & 0xFFFF;
    if (ntab == 0) return;
    float2 x[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) x[k] = *reinterpret_cast<const float2 *>(lds + (s0 ^ op_slot(op, 16 * part + k)));
#pragma unroll 1
    for (int q = 0; q < ntab; ++q) {
      Const<DevTab> &d = tabs[tab0 + q];
      int32_t b = d.base | (d.img[5] & -(lane >> 5)) | (part ? d.img[10] : 0);
#pragma unroll
      for (int j = 0; j < 5; ++j) b |= d.img[j] & -((lane >> j) & 1);
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (j < UB) b |= d.img[11 + j] & -((unit >> j) & 1);
#pragma unroll
      for (int k = 0; k < 16; ++k) {
        int32_t e = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          if ((k >> j) & 1) e |= d.img[6 + j];
        x[k] = cmul(*reinterpret_cast<const float2 *>(tabl + (b | e)), x[k]);
      }
    }
#pragma unroll
    for (int k = 0; k < 16; ++k) *reinterpret_cast<float2 *>(lds + (s0 ^ op_slot(op, 16 * part + k))) = x[k];
  };
  auto write16 = [&](Const<DevOp> &op, const floatx16 &re, const floatx16 &im, int32_t s0, uint32_t flip, int part) SV_INLINE {
    asm volatile("" : "+v"(s0));  // the slots are formed again: keeping them would cost 16 registers
#pragma unroll
    for (int k = 0; k < 16; ++k)
      *reinterpret_cast<float2 *>(lds + (s0 ^ op_slot(op, 16 * part + k))) =
          make_float2(flip_by(re[k], flip), flip_by(im[k], flip));
  };

  // A five-bit gate on this wave's units; operand chunk at opb.
  auto gate5 = [&](Const<DevOp> &op, const char *opb, uint32_t tile_no) SV_INLINE {
    constexpr int UB = S - 10, LU = C::UNITS - 1;
    int32_t su[C::UNITS];
    uint32_t flip[C::UNITS];
#pragma unroll
    for (int u = 0; u < C::UNITS; ++u) {
      const int unit = wave * C::UNITS + u;
      su[u] = unit_slot(op, unit, UB);
      flip[u] = unit_flip(unit, UB, tile_no);
      apply_tables(op, su[u], unit, UB, 0);
    }
    float2 x0[8], x1[8];
    Half h0, h1;
    floatx16 re, im;
    clear(re);
    clear(im);
    auto block0 = [&](int P) SV_INLINE { return opb + P * 2048; };
    auto block1 = [&](int P) SV_INLINE { return opb + P * 2048 + 1024; };
    auto split_under = [&](Half &h, const float2 *x, int u) SV_INLINE {
      return [&h, x, u, &split_step, &flip](int i) SV_INLINE {
#pragma unroll
        for (int j = i * NS / NP; j < (i + 1) * NS / NP; ++j) split_step(h, x, flip[u], j);
      };
    };
    read8(op, x0, su[0], 0);
    read8(op, x1, su[0], 1);
#pragma unroll
    for (int i = 0; i < NS; ++i) split_step(h0, x0, flip[0], i);
    if (LU > 0) read8(op, x0, su[LU], 0);
    __builtin_amdgcn_sched_barrier(0);
    products(re, im, h0, block0, split_under(h1, x1, 0));
    if (LU > 0) {
      read8(op, x1, su[LU], 1);
      __builtin_amdgcn_sched_barrier(0);
      products(re, im, h1, block1, split_under(h0, x0, LU));
      write16(op, re, im, su[0], flip[0], 0);
      clear(re);
      clear(im);
      __builtin_amdgcn_sched_barrier(0);
      products(re, im, h0, block0, split_under(h1, x1, LU));
    }
    products(re, im, h1, block1, [](int) {});
    write16(op, re, im, su[LU], flip[LU], 0);
  };

  int64_t tile = blockIdx.x;
  int64_t base = tile_base(tile);
  if (GATES) {
    load_operand(0);
    put_operand(0);
    if (nchunks > 1) {
      load_operand(1);
      put_operand(1);
    }
  }
  load_chunks(base);
  load_tables(base);
  put_chunks();
  put_tables();

  const bool resident = nchunks <= 2;  // the operands stay in LDS for all tiles
  int seq = 0;    // chunks used so far by this workgroup: chunk seq sits in buffer seq & 1
  int chunk = 0;  // the next chunk's number in the pass
  for (;;) {
    __syncthreads();
    const uint32_t tile_no = uint32_t(tile) & 0xFFFFFu;
    const int64_t here = base;
    tile += gridDim.x;
    const bool more = tile < ntiles;
    base = more ? tile_base(tile) : base;  // the last tile reads itself again, unused
    if (GATES) {
      auto buffer = [&]() SV_INLINE { return opl + ((resident ? chunk : seq) & 1) * OPB; };
      // The next tile's loads go out under the tile's first gate, after the
      // operand's: the wait for the operand then leaves them in flight (the
      // first gate has its own copy of the code for that).
      auto begin = [&](bool first) SV_INLINE {
        if (!resident) load_operand(chunk + 2 < nchunks ? chunk + 2 : chunk + 2 - nchunks);
        if (first) load_chunks(base);
      };
      auto finish = [&]() SV_INLINE {
        __syncthreads();
        // the chunk's buffer is free: the chunk after next goes there; it is
        // read after at least one more barrier
        if (!resident) put_operand(seq & 1);
        ++seq;
        chunk = chunk + 1 < nchunks ? chunk + 1 : 0;
      };
      auto run = [&](int o, auto is_first) SV_INLINE {
        constexpr bool first = decltype(is_first)::value;
        Const<DevOp> &op = ops[o];
        if (WIDE < 6 || !(op.tab & kOpSix)) {
          begin(first);
          gate5(op, buffer(), tile_no);
          finish();
          return;
        }
        if constexpr (WIDE >= 6) {
          // A six-bit gate: four operand chunks, one reduction step for both
          // row tiles each.  S = 14: a wave takes a unit; smaller tiles have
          // half as many units as waves, so a wave takes one row tile of a unit.
          constexpr int UB = S - 11, MTW = (1 << UB) >= C::NW ? 2 : 1;
          const int unit = MTW == 2 ? wave : wave >> 1, mt0 = MTW == 2 ? 0 : wave & 1;
          const int32_t s0 = unit_slot(op, unit, UB);
          const uint32_t flip = unit_flip(unit, UB, tile_no);
          if (MTW == 2) {
            apply_tables(op, s0, unit, UB, 0);
            apply_tables(op, s0, unit, UB, 1);
          } else if (op.tab >> 16 & 0xFF) {
            apply_tables(op, s0, unit, UB, mt0);
            __syncthreads();
          }
          float2 x[4];
          Half h0, h1;
          floatx16 re[MTW], im[MTW];
#pragma unroll
          for (int m = 0; m < MTW; ++m) {
            clear(re[m]);
            clear(im[m]);
          }
#pragma unroll
          for (int hf = 0; hf < 2; ++hf) {
            read4(op, x, s0, hf);
#pragma unroll
            for (int i = hf * NS / 2; i < (hf + 1) * NS / 2; ++i) split_step(h0, x, flip, i, 4);
          }
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            begin(first && s == 0);
            const char *opb = buffer();
            Half &now = (s & 1) ? h1 : h0, &then = (s & 1) ? h0 : h1;
            // the next eight inputs, four at a time: under the first and the second half of the products
            constexpr int TOTAL = MTW * NP;
#pragma unroll
            for (int m = 0; m < MTW; ++m) {
              if (s < 3 && (MTW == 1 || m == 0)) read4(op, x, s0, 2 * (s + 1));
              if (s < 3 && MTW == 2 && m == 1) read4(op, x, s0, 2 * (s + 1) + 1);
              __builtin_amdgcn_sched_barrier(0);
              products(re[m], im[m], now, [&](int P) SV_INLINE { return opb + P * 2048 + (mt0 + m) * 1024; }, [&](int i) SV_INLINE {
                if (s < 3) {
                  if (MTW == 1 && i == NP / 2) read4(op, x, s0, 2 * (s + 1) + 1);
#pragma unroll
                  for (int j = (m * NP + i) * NS / TOTAL; j < (m * NP + i + 1) * NS / TOTAL; ++j)
                    split_step(then, x, flip, j, 4);
                }
              });
            }
            // every wave has read its inputs before the last step's barrier
            if (s == 3) {
#pragma unroll
              for (int m = 0; m < MTW; ++m) write16(op, re[m], im[m], s0, flip, mt0 + m);
            }
            finish();
          }
        }
      };
      run(0, std::true_type());
#pragma unroll 1
      for (int o = 1; o < nops; ++o) run(o, std::false_type());
    } else {
      load_chunks(base);
    }

    load_tables(base);  // the next tile's, under the stores below

    // ---- LDS -> global, store-site tables on the way, a few chunks at a time
    constexpr int G = 4;
    const auto *hs = fresh();
#pragma unroll
    for (int i0 = 0; i0 < C::CHUNKS; i0 += G) {
      float2 a0[G], a1[G];
#pragma unroll
      for (int i = 0; i < G; ++i) {
        a0[i] = *reinterpret_cast<const float2 *>(lds + slot(i0 + i));
        a1[i] = *reinterpret_cast<const float2 *>(lds + (slot(i0 + i) ^ 8));
      }
#pragma unroll 1
      for (int q = 0; q < nstore; ++q) {
        Const<DevTab> &d = stores[q];
        int32_t b = d.base;
#pragma unroll
        for (int j = 0; j < C::NTB; ++j) b |= d.img[j] & -((t >> j) & 1);
        const int32_t b1 = d.img[13];
#pragma unroll
        for (int i = 0; i < G; ++i) {
          int32_t e = 0;
#pragma unroll
          for (int j = 0; (1 << j) < C::CHUNKS; ++j)
            if (((i0 + i) >> j) & 1) e |= d.img[9 + j];
          a0[i] = cmul(*reinterpret_cast<const float2 *>(tabl + (b | e)), a0[i]);
          a1[i] = cmul(*reinterpret_cast<const float2 *>(tabl + (b | (e | b1))), a1[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < G; ++i) {
        const floatx4 o = {a0[i].x, a0[i].y, a1[i].x, a1[i].y};
        __builtin_nontemporal_store(o, reinterpret_cast<floatx4 *>(psi_t + (here + goff(hs, i0 + i))));
      }
    }
    if (!more) break;
    // every thread owns the same slots on both sides: only the tables need a
    // barrier.  After the stores in program order, so that the wait for the
    // loads leaves the stores in flight.
    put_chunks();
    if (nstore > 0) __syncthreads();
    put_tables();
  }
}

template <int S>
hipError_t launch_s(int64_t ntiles, int wide, float2 *psi, const char *data, hipStream_t st) {
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  const int64_t per_cu = S >= 14 ? 1 : 2;
  const unsigned grid = unsigned(std::min<int64_t>(ntiles, per_cu * cus));
  const dim3 g(grid), b(Cfg<S>::NT);
  if (wide == 0)
    hipLaunchKernelGGL((k_pass<S, 0>), g, b, 0, st, psi, data, ntiles);
  else if (wide == 5)
    hipLaunchKernelGGL((k_pass<S, 5>), g, b, 0, st, psi, data, ntiles);
  else if constexpr (S >= 11)  // a unit of a six-bit gate is 2^11 amplitudes
    hipLaunchKernelGGL((k_pass<S, 6>), g, b, 0, st, psi, data, ntiles);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace

hipError_t launch(int n, const Fused &f, float2 *psi, const char *data_dev, hipStream_t st) {
  if (f.S < kMinS || f.S > kMaxS || f.S > n || f.sbit[0] != 0)  // 16-byte chunks pair amplitudes of physical bit 0
    return hipErrorInvalidValue;
  for (int b = 0; b < f.S; ++b)
    if (f.sbit[b] < 0 || f.sbit[b] >= n || (b > 0 && f.sbit[b] <= f.sbit[b - 1])) return hipErrorInvalidValue;
  const int64_t ntiles = int64_t(1) << (n - f.S);
  switch (f.S) {
    case 10: return launch_s<10>(ntiles, f.wide, psi, data_dev, st);
    case 11: return launch_s<11>(ntiles, f.wide, psi, data_dev, st);
    case 12: return launch_s<12>(ntiles, f.wide, psi, data_dev, st);
    case 13: return launch_s<13>(ntiles, f.wide, psi, data_dev, st);
    case 14: return launch_s<14>(ntiles, f.wide, psi, data_dev, st);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace pass
}  // namespace sv
