// Gate chains for gfx950: two to four dense gates of four to six bits on a tile
// of 2^13 amplitudes in LDS, with one read and one write of the state.
//
// Each gate is the FP32 matrix-core arithmetic of its own sweep (k_tile_mfma:
// the embedding at four bits, the three-multiplication product above), with
// the same operand, the same instruction and the same order of reduction, so
// every amplitude is the same bit for bit; only where the groups sit differs.
//
// Bound by the matrix cores where a six-bit gate is in the chain, by memory
// otherwise: at 2^26 amplitudes two four-bit gates take 222 us (one 171 alone;
// 181 us of memory, 110 of products), a six- and a four-bit one 352 (262 +
// 171), two six-bit ones 473 to 550 (the products alone 343).  Two workgroups of
// four waves per CU, one tile each, cover each other's loads and stores; a
// persistent grid that held the next tile in registers was 5% slower (the wait
// for an operand is one for all loads before it), a 2^14 tile on one workgroup
// per CU 10%.
#include <algorithm>

#include "sv_chain.h"
#include "sv_internal.h"

namespace sv {
namespace chain {
namespace {

typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kThreadBits = 8, kThreads = 1 << kThreadBits;
constexpr int kChunks = (1 << kTileBits) / 2 / kThreads;  // of 16 bytes per thread

struct Args {
  float2 *psi;
  const char *ops;
  int32_t ngates, cus;
  int32_t sbit[kTileBits];
  Gate gate[kMaxGates];
};

__device__ __forceinline__ int slot_of(int l) { return l ^ ((l >> 5) & 31) ^ ((l >> 10) & 31); }
__device__ __forceinline__ float2 &at(char *lds, int byte) { return *reinterpret_cast<float2 *>(lds + byte); }

// byte image of input (or output) amplitude e of a lane's half
template <int K>
__device__ __forceinline__ int input(const Gate &g, int e) {
  int s = 0;
#pragma unroll
  for (int j = 0; j < K - 1; ++j)
    if (e >> j & 1) s ^= g.c[j];
  return s;
}

template <int K>
__device__ __forceinline__ int unit_base(const Gate &g, int lane, int unit) {
  int s = (lane >> 5) ? g.half : 0;
#pragma unroll
  for (int j = 0; j < 5; ++j) s ^= (lane >> j & 1) ? g.lane[j] : 0;
#pragma unroll
  for (int j = 0; j < kTileBits - 5 - K; ++j) s ^= (unit >> j & 1) ? g.unit[j] : 0;
  return s;
}

__device__ __forceinline__ floatx16 zero16() {
  floatx16 z;
#pragma unroll
  for (int r = 0; r < 16; ++r) z[r] = 0.f;
  return z;
}

// Operands stream through two LDS buffers of 8 KiB in chunks, one per step of
// a gate: eight reduction steps of the real or imaginary rows (four planes of
// 2 KiB at six bits, two at five, one at four).  Every gate has an even number
// of steps, so that a step's parity, which names its buffer, is known where it
// is compiled.
constexpr int kChunkBytes = 8192;
constexpr int kPieces = kChunkBytes / 16 / kThreads;  // of 16 bytes per thread
__host__ __device__ constexpr int steps_of(int K) { return K == 6 ? 4 : 2; }
__device__ __forceinline__ int chunk_source(int K, int q, int p) {  // of the chunk's p-th 16 bytes
  const int plane = (p >> 7) & ((1 << (K - 4)) - 1);
  return plane * (K == 6 ? 8192 : 4096) + q * 2048 + (p & 127) * 16;
}

// K = 5, 6: T1 = Gr Xr, T2 = Gi Xi, T3 = (Gr + Gi)(Xr + Xi) on U units.  At six
// bits two waves share their units, one for each 32 rows of the outputs.
template <int K, typename Begin, typename End>
__device__ __forceinline__ void gauss(const Gate &g, char *lds, int lane, int wave, Begin begin, End end) {
  constexpr int AH = 1 << (K - 1), STEPS = steps_of(K), KS = AH / STEPS;
  const int mt = K == 6 ? wave & 1 : 0;
  const int first = K == 6 ? (wave >> 1) * 2 : wave * 2;
  int s[2];
  floatx16 t1[2], t2[2], t3[2];
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    s[u] = unit_base<K>(g, lane, first + u);
    t1[u] = t2[u] = t3[u] = zero16();
  }
#pragma unroll
  for (int q = 0; q < STEPS; ++q) {
    const float *op = begin(q & 1) + lane;
    const float *pr = op + (K == 6 ? mt * 512 : 0), *pi = op + (K == 6 ? (2 + mt) * 512 : 512);
    // the next reduction step's reads go out before this one's products
    float gr = pr[0], gi = pi[0];
    float2 x[2];
#pragma unroll
    for (int u = 0; u < 2; ++u) x[u] = at(lds, s[u] ^ input<K>(g, q * KS));
#pragma unroll
    for (int k = 0; k < KS; ++k) {
      float nr = 0.f, ni = 0.f;
      float2 nx[2];
      if (k + 1 < KS) {
        nr = pr[(k + 1) * 64];
        ni = pi[(k + 1) * 64];
#pragma unroll
        for (int u = 0; u < 2; ++u) nx[u] = at(lds, s[u] ^ input<K>(g, q * KS + k + 1));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        t1[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(gr, x[u].x, t1[u], 0, 0, 0);
        t2[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(gi, x[u].y, t2[u], 0, 0, 0);
        t3[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(gr + gi, x[u].x + x[u].y, t3[u], 0, 0, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
      gr = nr;
      gi = ni;
#pragma unroll
      for (int u = 0; u < 2; ++u) x[u] = nx[u];
    }
    if (K == 6 || q + 1 < STEPS) end();  // after the last one the other wave has read these groups
  }
  const int em = mt ? g.c[4] : 0;  // outputs 16 mt + r of the half
#pragma unroll
  for (int u = 0; u < 2; ++u)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const float a = t1[u][r], b = t2[u][r], c = t3[u][r];
      at(lds, s[u] ^ em ^ input<5>(g, r)) = make_float2(a - b, c - a - b);
    }
  end();
}

// K = 4: [Re y; Im y] = [[Re G, -Im G], [Im G, Re G]] [Re x; Im x], four units per wave
template <typename Begin, typename End>
__device__ __forceinline__ void embed(const Gate &g, char *lds, int lane, int wave, Begin begin, End end) {
  int s[4];
  floatx16 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) {
    s[u] = unit_base<4>(g, lane, wave * 4 + u);
    acc[u] = zero16();
  }
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const float *op = begin(q) + lane;
    float a0 = op[0], a1 = op[64];
    float2 x[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) x[u] = at(lds, s[u] ^ input<4>(g, 4 * q));
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float n0 = 0.f, n1 = 0.f;
      float2 nx[4];
      if (e < 3) {
        n0 = op[(2 * e + 2) * 64];
        n1 = op[(2 * e + 3) * 64];
#pragma unroll
        for (int u = 0; u < 4; ++u) nx[u] = at(lds, s[u] ^ input<4>(g, 4 * q + e + 1));
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a0, x[u].x, acc[u], 0, 0, 0);
#pragma unroll
      for (int u = 0; u < 4; ++u) acc[u] = __builtin_amdgcn_mfma_f32_32x32x2f32(a1, x[u].y, acc[u], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
      a0 = n0;
      a1 = n1;
#pragma unroll
      for (int u = 0; u < 4; ++u) x[u] = nx[u];
    }
    if (q == 0) end();
  }
#pragma unroll
  for (int u = 0; u < 4; ++u)
#pragma unroll
    for (int e = 0; e < 8; ++e) at(lds, s[u] ^ input<4>(g, e)) = make_float2(acc[u][2 * e], acc[u][2 * e + 1]);
  end();
}

// launch_bounds: two waves per SIMD
__global__ __launch_bounds__(kThreads, 2) void k_chain(Args a) {
  __shared__ float2 tile[1 << kTileBits];
  __shared__ __attribute__((aligned(16))) char ring[2 * kChunkBytes];
  char *const lds = reinterpret_cast<char *>(tile);
  const int t = threadIdx.x, lane = t & 63, wave = __builtin_amdgcn_readfirstlane(t >> 6);
  int64_t goff = 0;
#pragma unroll
  for (int b = 0; b < kThreadBits; ++b) goff |= int64_t(t >> b & 1) << a.sbit[1 + b];
  auto chunk = [&](int i) {  // global offset of chunk i, thread bits apart
    int64_t o = 0;
#pragma unroll
    for (int b = 0; b < kTileBits - 1 - kThreadBits; ++b)
      if (i >> b & 1) o |= int64_t(1) << a.sbit[1 + kThreadBits + b];
    return o;
  };
  auto slot = [&](int i) { return 8 * (slot_of(2 * t) ^ slot_of(i << (1 + kThreadBits))); };
  auto tile_base = [&](int64_t x) {
#pragma unroll
    for (int b = 0; b < kTileBits; ++b) {
      const int p = a.sbit[b];
      x = ((x >> p) << (p + 1)) | (x & ((int64_t(1) << p) - 1));
    }
    return x;
  };
  // operand chunks in the order of the gates (after the last the first again, unused).  Step c reads
  // chunk c from buffer c mod 2, puts c + 1, which its registers hold, into the
  // other one (whose readers met at the last barrier) and fetches c + 3.
  int fg = 0, fq = 0;  // the chunk to fetch next
  floatx4 even[kPieces], odd[kPieces];
  auto fetch = [&](floatx4(&to)[kPieces]) __attribute__((always_inline)) {
    const int K = a.gate[fg].K;
    const char *src = a.ops + a.gate[fg].op;
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
      to[i] = *reinterpret_cast<const floatx4 *>(src + chunk_source(K, fq, t + i * kThreads));
    if (++fq == steps_of(K)) {
      fq = 0;
      fg = fg + 1 == a.ngates ? 0 : fg + 1;
    }
  };
  auto put = [&](int buf, const floatx4(&from)[kPieces]) __attribute__((always_inline)) {
#pragma unroll
    for (int i = 0; i < kPieces; ++i)
      *reinterpret_cast<floatx4 *>(ring + buf * kChunkBytes + (t + i * kThreads) * 16) = from[i];
  };
  fetch(even);
  put(0, even);
  fetch(odd);
  fetch(even);
  auto begin = [&](int parity) __attribute__((always_inline)) {
    if (parity) {
      put(0, even);
      fetch(even);
    } else {
      put(1, odd);
      fetch(odd);
    }
    return reinterpret_cast<const float *>(ring + parity * kChunkBytes);
  };
  auto end = [&]() __attribute__((always_inline)) { __syncthreads(); };

  // The second workgroup of each CU starts a few microseconds late, so that one
  // loads or stores while the other multiplies: in step, both wait for memory
  // at once (two four-bit gates 236 -> 222 us, a six- and a four-bit one 370 ->
  // 352 at 2^26 amplitudes; two six-bit ones unchanged).  cus: 0 for small states.
  if (int(blockIdx.x) >= a.cus && int(blockIdx.x) < 2 * a.cus) __builtin_amdgcn_s_sleep(127);
  const int64_t base = tile_base(blockIdx.x) + goff;
  {
    floatx4 v[kChunks];
#pragma unroll
    for (int i = 0; i < kChunks; ++i)
      v[i] = __builtin_nontemporal_load(reinterpret_cast<const floatx4 *>(a.psi + base + chunk(i)));
#pragma unroll
    for (int i = 0; i < kChunks; ++i) {
      at(lds, slot(i)) = make_float2(v[i][0], v[i][1]);
      at(lds, slot(i) ^ 8) = make_float2(v[i][2], v[i][3]);
    }
  }
  __syncthreads();
#pragma unroll 1
  for (int o = 0; o < a.ngates; ++o) {
    const Gate &g = a.gate[o];
    uint32_t k = 1u << g.K;  // independent tests, no joins
    asm("" : "+s"(k));
    if (k & 16) embed(g, lds, lane, wave, begin, end);
    if (k & 32) gauss<5>(g, lds, lane, wave, begin, end);
    if (k & 64) gauss<6>(g, lds, lane, wave, begin, end);
  }
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    const float2 p = at(lds, slot(i)), q = at(lds, slot(i) ^ 8);
    const floatx4 w = {p.x, p.y, q.x, q.y};
    __builtin_nontemporal_store(w, reinterpret_cast<floatx4 *>(a.psi + base + chunk(i)));
  }
}

}  // namespace

hipError_t launch(int n, const Step &s, float2 *psi, const char *ops, hipStream_t st) {
  Args a;
  a.psi = psi;
  a.ops = ops;
  a.ngates = int32_t(s.items.size());
  if (n < kTileBits || a.ngates < 1 || a.ngates > kMaxGates || s.sbit[0] != 0) return hipErrorInvalidValue;
  for (int b = 0; b < kTileBits; ++b) a.sbit[b] = s.sbit[b];
  for (int i = 0; i < kMaxGates; ++i) {
    a.gate[i] = i < a.ngates ? s.gate[i] : Gate{};
    if (i < a.ngates && (a.gate[i].K < 4 || a.gate[i].K > 6)) return hipErrorInvalidValue;
  }
  int dev = 0, cus = 256;
  if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
  a.cus = (1 << (n - kTileBits)) >= 8 * cus ? cus : 0;  // with few tiles per CU the start costs more than it gives
  hipLaunchKernelGGL(k_chain, dim3(1u << (n - kTileBits)), dim3(kThreads), 0, st, a);
  return hipGetLastError();
}

}  // namespace chain
}  // namespace sv
