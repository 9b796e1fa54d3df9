// Cutting a gate sequence into fused tile passes (host only, no HIP types).
#include "sv_pass_host.h"

#include <algorithm>
#include <cstring>

#include "sv.h"

namespace sv {

namespace pass {
namespace {

inline int popc(uint64_t x) { return __builtin_popcountll(x); }

// Tile bits of a pass on n qubits, and the lowest bits every tile holds.
// Wider tiles take more gates per pass, narrower ones spread a small state over
// more CUs; runs of 8 amplitudes do while the state stays in the caches, of a
// cache line (16) beyond.  Twelve brickwork layers in blocks of five / six
// qubits, us, by tile bits:
//   n=14  12: 140/211  13: 180/261  14: 249/366
//   n=16  12: 146/256  13: 185/301  14: 307/446
//   n=20  12: 273/335  13: 261/389  14: 403/544
//   n=21  12: 400/463  13: 352/398  14: 462/554
//   n=22  12: 768/995  13: 712/1015 14: 632/859
//   n=24  12: 2571/3447 13: 2487/3336 14: 2333/2940
// and one workgroup for all of n=12 (99/166) against 2^11 tiles (134/188).
struct Shape {
  int S, low;
};
Shape shape_for(int n) {
  if (n <= 12) return {n, n};
  if (n <= 20) return {12, 3};
  if (n == 21) return {13, 3};
  return {14, 4};
}

uint16_t bf16_rne(float x) {
  uint32_t u;
  std::memcpy(&u, &x, 4);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return uint16_t(u >> 16);
}
float bf16_to_f(uint16_t h) {
  const uint32_t u = uint32_t(h) << 16;
  float f;
  std::memcpy(&f, &u, 4);
  return f;
}

// The three bf16 pieces of a component, each what the ones before leave.
inline void split3(double v, uint16_t *p) {
  p[0] = bf16_rne(float(v));
  const double v1 = v - double(bf16_to_f(p[0]));
  p[1] = bf16_rne(float(v1));
  p[2] = bf16_rne(float(v1 - double(bf16_to_f(p[1]))));
}

// Operand of a K-bit gate (K = 5, 6): each component of G in three bf16
// pieces (hi + mid + lo keeps 24 bits), planes (Gr, Gi) x (hi, mid, lo).  A
// block of 1 KiB holds one plane of one 32-row tile mt and one reduction step
// kk: lane l has the eight values G[row][2^(K-1) (l / 32) + 8 kk + e], the rows
// ordered so that accumulator register r of lane half h is row
// 2^(K-1) h + 16 mt + r.  Blocks: five bits (plane, step), six bits
// (step, plane, row tile).
void pack_gate(int K, const double *G, char *out) {
  const int D = 1 << K, AH = D / 2, mts = D / 32, steps = AH / 8;
  for (int mt = 0; mt < mts; ++mt)
    for (int i = 0; i < 32; ++i) {
      const double *row = G + 2 * size_t(AH * ((i >> 2) & 1) + 16 * mt + 4 * (i >> 3) + (i & 3)) * D;
      for (int half = 0; half < 2; ++half)
        for (int kk = 0; kk < steps; ++kk) {
          const double *src = row + 2 * (AH * half + 8 * kk);
          uint16_t piece[2][3][8];
          for (int part = 0; part < 2; ++part)
            for (int e = 0; e < 8; ++e) {
              uint16_t p[3];
              split3(src[2 * e + part], p);
              for (int w = 0; w < 3; ++w) piece[part][w][e] = p[w];
            }
          for (int part = 0; part < 2; ++part)
            for (int w = 0; w < 3; ++w) {
              const int P = part * 3 + w, block = K == 6 ? (kk * 6 + P) * 2 + mt : P * 2 + kk;
              std::memcpy(out + 1024 * size_t(block) + 16 * size_t(32 * half + i), piece[part][w], 16);
            }
        }
    }
}

// Operand of a gate on k < 5 bits, G (x) 1 on five, into zeroed memory: only
// the 4^k entries are split, and only the places they go to are written (45
// two-bit gates and 15 diagonals on 20 qubits: cut and packed in 0.11 ms, 0.30
// with every gate as a full matrix).
void pack_narrow(int k, const double *G, char *out) {
  const int D = 1 << k;
  uint16_t piece[16 * 16][2][3];
  for (int z = 0; z < D * D; ++z)
    for (int part = 0; part < 2; ++part) split3(G[2 * z + part], piece[z][part]);
  for (int i = 0; i < 32; ++i) {
    const int R = 16 * ((i >> 2) & 1) + 4 * (i >> 3) + (i & 3);
    for (int c = 0; c < D; ++c) {
      const int C = (R & ~(D - 1)) | c, z = (R & (D - 1)) * D + c;
      char *at = out + 1024 * ((C >> 3) & 1) + 16 * (32 * (C >> 4) + i) + 2 * (C & 7);
      for (int P = 0; P < 6; ++P) std::memcpy(at + 2048 * P, &piece[z][P / 3][P % 3], 2);
    }
  }
}

// A diagonal factor collected at one site of a pass.
struct Table {
  int site = 0;              // applied before dense gate `site` (or at the store)
  uint64_t in = 0, out = 0;  // physical bits inside and outside the tile
  std::vector<int> items;
};

struct Draft {
  uint64_t tile = 0;       // bits the dense gates need
  std::vector<int> items;  // in order
  std::vector<int> dense;
  int chunks = 0;
  std::vector<Table> tabs;
};

uint64_t bits_of(const Item &it) {
  uint64_t b = 0;
  for (int j = 0; j < it.k; ++j) b |= uint64_t(1) << it.A[j];
  return b;
}

int padded_entries(const Table &t, uint64_t tile) { return std::max(kTabBlock, 1 << popc((t.in | t.out) & tile)); }

// The tables must fit LDS for the final tile, so they are checked against
// the largest tile the pass may still take: every bit of a table counts as
// a tile bit until the tile is closed.
struct Builder {
  int n;
  const std::vector<Item> &items;
  bool f32;
  Shape sh;
  uint64_t low;

  Builder(int n_, const std::vector<Item> &it, int p) : n(n_), items(it), f32(p == SV_PREC_FP32), sh(shape_for(n_)) {
    low = sh.low >= 64 ? ~uint64_t(0) : (uint64_t(1) << sh.low) - 1;
  }

  // Gates a pass can take.  Dense ones in FP32 (a unit of a six-bit gate is
  // 2^11 amplitudes); in BF16x3 every sweep's rounding is the caller's choice
  // and any other order of it shows at the 4e-5 of that arithmetic, so there
  // a pass takes only diagonals that are exact (entries 1, -1, i, -i).
  bool takes(const Item &it) const {
    if (it.diag) return f32 || it.exact;
    return f32 && it.k <= (sh.S >= 11 ? 6 : 5);
  }

  bool tile_fits(uint64_t tile) const {
    return popc(tile | low) <= sh.S;
  }

  // Entries a set of tables takes when the tile is `tile` (chosen bits only).
  int entries(const std::vector<Table> &tabs, uint64_t tile) const {
    int e = 0;
    for (const Table &t : tabs) e += padded_entries(t, tile | low);
    return e;
  }

  bool table_ok(uint64_t bits, uint64_t tile) const {
    return popc(bits) <= kTabBits && popc(bits & (tile | low)) <= kTabInBits;
  }

  // Adds diagonal item i to the draft: into a table whose site commutes with
  // everything between, or a new one at the current site.
  bool add_diag(Draft &d, int i) const {
    const uint64_t b = bits_of(items[size_t(i)]);
    int earliest = 0;
    for (size_t j = 0; j < d.dense.size(); ++j)
      if (bits_of(items[size_t(d.dense[j])]) & b) earliest = int(j) + 1;
    Table *best = nullptr;
    int best_new = 99;
    for (Table &t : d.tabs) {
      if (t.site < earliest) continue;
      // an item may move to any site from its earliest on that no later dense gate on its bits precedes:
      // it is the newest item, so every site from `earliest` to the end qualifies
      const uint64_t u = t.in | b;
      if (!table_ok(u, d.tile)) continue;
      const int extra = popc(u) - popc(t.in);
      if (extra < best_new) {
        best_new = extra;
        best = &t;
      }
    }
    if (best) {
      const uint64_t keep = best->in;
      best->in |= b;
      if (entries(d.tabs, d.tile) <= kTabEntries) {
        best->items.push_back(i);
        d.items.push_back(i);
        return true;
      }
      best->in = keep;
    }
    if (!table_ok(b, d.tile)) return false;
    Table t;
    t.site = std::max(earliest, int(d.dense.size()));
    t.in = b;
    t.items.push_back(i);
    d.tabs.push_back(t);
    if (entries(d.tabs, d.tile) > kTabEntries) {
      d.tabs.pop_back();
      return false;
    }
    d.items.push_back(i);
    return true;
  }

  bool add_dense(Draft &d, int i) const {
    const int chunks = d.chunks + chunks_of(items[size_t(i)].k);
    if (chunks > kMaxChunks) return false;
    const uint64_t t = d.tile | bits_of(items[size_t(i)]);
    if (!tile_fits(t)) return false;
    for (const Table &tb : d.tabs)  // tables keep fitting when more of their bits join the tile
      if (!table_ok(tb.in, t)) return false;
    if (entries(d.tabs, t) > kTabEntries) return false;
    d.tile = t;
    d.chunks = chunks;
    d.dense.push_back(i);
    d.items.push_back(i);
    return true;
  }

  Draft draft(std::vector<char> &done, size_t from) const {
    Draft d;
    uint64_t block_dense = 0, block_diag = 0;  // bits of skipped dense and diagonal items
    const uint64_t all = n >= 64 ? ~uint64_t(0) : (uint64_t(1) << n) - 1;
    for (size_t i = from; i < items.size() && (block_dense & all) != all; ++i) {
      if (done[i]) continue;
      const Item &it = items[i];
      const uint64_t b = bits_of(it);
      if (it.diag) {
        if (takes(it) && !(b & block_dense) && add_diag(d, int(i))) continue;
        block_diag |= b;
      } else {
        if (takes(it) && !(b & (block_dense | block_diag)) && add_dense(d, int(i))) continue;
        block_dense |= b;
      }
    }
    for (int i : d.items) done[size_t(i)] = 1;
    return d;
  }

  // Tile of a draft: the dense gates' bits, the low bits, then the lowest
  // others -- leaving the three lowest free bits from bit 7 up to the tile
  // index, whose low bits name the XCD (as the single-gate tiles do) -- as
  // long as the tables, which widen with every bit of theirs that joins the
  // tile, keep fitting LDS.
  uint64_t close_tile(const Draft &d) const {
    uint64_t t = d.tile | low;
    if (sh.S >= n) return (uint64_t(1) << n) - 1;
    uint64_t reserve = 0;
    for (int p = 7, r = 0; p < n && r < 3; ++p)
      if (!((t >> p) & 1)) {
        reserve |= uint64_t(1) << p;
        ++r;
      }
    for (int round = 0; round < 3; ++round)
      for (int p = 0; p < n && popc(t) < sh.S; ++p) {
        const uint64_t u = t | (uint64_t(1) << p);
        if (u == t || (round == 0 && ((reserve >> p) & 1))) continue;
        if (round < 2 && entries(d.tabs, u) > kTabEntries) continue;
        t = u;
      }
    return t;
  }

  // Takes back store-site tables, the last first, until the rest fit the
  // closed tile's LDS area (nothing in the draft follows them).
  void trim(Draft &d, std::vector<char> &done) const {
    while (entries(d.tabs, close_tile(d)) > kTabEntries) {
      int last = -1;
      for (size_t t = 0; t < d.tabs.size(); ++t)
        if (d.tabs[t].site == int(d.dense.size())) last = int(t);
      if (last < 0) return;
      for (int i : d.tabs[size_t(last)].items) {
        done[size_t(i)] = 0;
        d.items.erase(std::find(d.items.begin(), d.items.end(), i));
      }
      d.tabs.erase(d.tabs.begin() + last);
    }
  }

  // Device data of a draft; false when its tables do not fit (its items then
  // run one by one).
  bool emit(Draft &d, Fused *f) const {
    const uint64_t tile = close_tile(d);
    // the widest first: a table's base is then a multiple of its size, and indices combine by OR
    std::stable_sort(d.tabs.begin(), d.tabs.end(),
                     [&](const Table &a, const Table &b) { return padded_entries(a, tile) > padded_entries(b, tile); });
    if (popc(tile) != sh.S) return false;
    int local[64];
    int b = 0;
    for (int p = 0; p < n; ++p) {
      local[p] = -1;
      if ((tile >> p) & 1) {
        f->sbit[b] = p;
        local[p] = b++;
      }
    }
    const int S = sh.S;
    const int nw_bits = std::min(3, S - 10);      // waves per workgroup
    const int nt_bits = 6 + nw_bits;              // threads
    const int chunk_bits = S - 1 - nt_bits;       // 16-byte chunks per thread
    int tab_entries = 0;
    size_t global_entries = 0;
    struct TabPlace {
      int base = 0;
      size_t goff = 0;
      std::vector<int> inb, outb;  // physical bits, low index bits first
    };
    std::vector<TabPlace> place(d.tabs.size());
    for (size_t t = 0; t < d.tabs.size(); ++t) {
      TabPlace &q = place[t];
      for (int p = 0; p < n; ++p)
        if ((d.tabs[t].in >> p) & 1) ((tile >> p) & 1 ? q.inb : q.outb).push_back(p);
      const int e = std::max(kTabBlock, 1 << q.inb.size());
      if (int(q.inb.size()) + int(q.outb.size()) > kTabBits) return false;
      q.base = tab_entries;
      q.goff = global_entries;
      tab_entries += e;
      global_entries += (size_t(1) << (q.inb.size() + q.outb.size())) + kTabBlock;  // whole blocks may be read past the end
    }
    if (tab_entries > kTabEntries) return false;

    std::vector<DevOp> ops(d.dense.size());
    std::vector<DevTab> tabs;
    std::vector<DevTab> stores;
    int nchunks = 0;
    auto index_img = [&](size_t t, int lb) -> int32_t {  // byte image of local bit lb in table t's index
      for (size_t j = 0; j < place[t].inb.size(); ++j)
        if (local[place[t].inb[j]] == lb) return int32_t(8 << j);
      return 0;
    };
    for (size_t o = 0; o < d.dense.size(); ++o) {
      const Item &it = items[size_t(d.dense[o])];
      DevOp &op = ops[o];
      std::memset(&op, 0, sizeof(op));
      const int K = std::max(it.k, 5), unit_bits = S - 5 - K;
      int tb[kGateBits];
      uint32_t used = 0;
      for (int j = 0; j < it.k; ++j) {
        tb[j] = local[it.A[j]];
        used |= 1u << tb[j];
      }
      for (int j = it.k, lb = S - 1; j < K; --lb)  // narrower gates act as G (x) 1 on spare tile bits
        if (!((used >> lb) & 1)) {
          tb[j++] = lb;
          used |= 1u << lb;
        }
      // lane bits: five of the other tile bits, of different residues mod 5 where they exist
      int gl[5], ng = 0;
      uint32_t lane_used = 0, res = 0;
      for (int round = 0; round < 2; ++round)
        for (int lb = 0; lb < S && ng < 5; ++lb) {
          if (((used | lane_used) >> lb) & 1) continue;
          if (round == 0 && ((res >> (lb % 5)) & 1)) continue;
          gl[ng++] = lb;
          lane_used |= 1u << lb;
          res |= 1u << (lb % 5);
        }
      int un[4] = {-1, -1, -1, -1}, nu = 0;
      for (int lb = 0; lb < S && nu < 4; ++lb)
        if (!(((used | lane_used) >> lb) & 1)) un[nu++] = lb;
      if (ng != 5 || nu != unit_bits) return false;
      for (int j = 0; j < 5; ++j) op.lane[j] = 8 * slot_image(gl[j]);
      op.half = 8 * slot_image(tb[K - 1]);
      for (int j = 0; j + 1 < K; ++j) op.c[j] = 8 * slot_image(tb[j]);
      for (int j = 0; j < nu; ++j) op.unit[j] = 8 * slot_image(un[j]);
      const int tab0 = int(tabs.size());
      for (size_t t = 0; t < d.tabs.size(); ++t) {
        if (d.tabs[t].site != int(o)) continue;
        DevTab dt;
        std::memset(&dt, 0, sizeof(dt));
        dt.base = 8 * place[t].base;
        for (int j = 0; j < 5; ++j) dt.img[j] = index_img(t, gl[j]);
        dt.img[5] = index_img(t, tb[K - 1]);
        for (int j = 0; j + 1 < K; ++j) dt.img[6 + j] = index_img(t, tb[j]);
        for (int j = 0; j < nu; ++j) dt.img[11 + j] = index_img(t, un[j]);
        tabs.push_back(dt);
      }
      op.tab = tab0 | int32_t(tabs.size() - size_t(tab0)) << 16 | (K == 6 ? kOpSix : 0);
      nchunks += chunks_of(K);
      f->wide = std::max(f->wide, K);
    }
    for (size_t t = 0; t < d.tabs.size(); ++t) {
      if (d.tabs[t].site != int(d.dense.size())) continue;
      DevTab dt;
      std::memset(&dt, 0, sizeof(dt));
      dt.base = 8 * place[t].base;
      for (int j = 0; j < nt_bits; ++j) dt.img[j] = index_img(t, 1 + j);
      for (int j = 0; j < chunk_bits; ++j) dt.img[9 + j] = index_img(t, 1 + nt_bits + j);
      dt.img[13] = index_img(t, 0);
      stores.push_back(dt);
    }
    std::vector<DevBlk> blks;
    for (size_t t = 0; t < d.tabs.size(); ++t) {
      const TabPlace &q = place[t];
      const int e = std::max(kTabBlock, 1 << q.inb.size());
      for (int x = 0; x < e / kTabBlock; ++x) {
        DevBlk bk;
        std::memset(&bk, 0, sizeof(bk));
        bk.goff = int32_t(q.goff) + x * kTabBlock;
        bk.nin = int32_t(q.inb.size());
        bk.nout = int32_t(q.outb.size());
        for (size_t j = 0; j < q.outb.size(); ++j) bk.out[j] = q.outb[j];
        blks.push_back(bk);
      }
    }
    // lay everything out
    auto align = [](size_t x) { return (x + 255) & ~size_t(255); };
    DevHead h;
    std::memset(&h, 0, sizeof(h));
    h.nops = int32_t(ops.size());
    h.nblk = int32_t(blks.size());
    if (blks.empty()) {  // waves without a block of their own read block 0: one that is always readable
      DevBlk none;
      std::memset(&none, 0, sizeof(none));
      blks.push_back(none);
      global_entries = std::max(global_entries, size_t(kTabBlock));
    }
    h.nstore = int32_t(stores.size());
    h.nchunks = nchunks;
    for (int j = 0; j < S; ++j) h.sbit[j] = f->sbit[j];
    size_t off = sizeof(DevHead);
    h.ops = int32_t(off);
    off += ops.size() * sizeof(DevOp);
    h.tabs = int32_t(off);
    off += tabs.size() * sizeof(DevTab);
    h.stores = int32_t(off);
    off += stores.size() * sizeof(DevTab);
    h.blks = int32_t(off);
    off += blks.size() * sizeof(DevBlk);
    off = align(off);
    h.table = int32_t(off);
    off = align(off + global_entries * 8);
    h.operand = int32_t(off);
    const size_t cb = kChunkBytes;
    off += size_t(nchunks) * cb;
    f->data.assign(off, 0);
    char *p = f->data.data();
    std::memcpy(p, &h, sizeof(h));
    if (!ops.empty()) std::memcpy(p + h.ops, ops.data(), ops.size() * sizeof(DevOp));
    if (!tabs.empty()) std::memcpy(p + h.tabs, tabs.data(), tabs.size() * sizeof(DevTab));
    if (!stores.empty()) std::memcpy(p + h.stores, stores.data(), stores.size() * sizeof(DevTab));
    if (!blks.empty()) std::memcpy(p + h.blks, blks.data(), blks.size() * sizeof(DevBlk));
    std::vector<double> prod;
    for (size_t t = 0; t < d.tabs.size(); ++t) {
      const TabPlace &q = place[t];
      const int nin = int(q.inb.size()), nout = int(q.outb.size());
      const size_t len = size_t(1) << (nin + nout);
      prod.assign(2 * len, 0.0);
      for (size_t x = 0; x < len; ++x) prod[2 * x] = 1.0;
      for (int i : d.tabs[t].items) {
        const Item &it = items[size_t(i)];
        const int D = 1 << it.k;
        // entry of the item's diagonal at table index x: lo[x & 31] | hi[x >> 5]
        uint8_t lo[32] = {0}, hi[1 << (kTabBits - 5)] = {0};
        for (int j = 0; j < it.k; ++j)
          for (int z = 0; z < nin + nout; ++z) {
            if ((z < nin ? q.inb[size_t(z)] : q.outb[size_t(z - nin)]) != it.A[j]) continue;
            if (z < 5)
              for (int v = 0; v < 32; ++v) lo[v] = uint8_t(lo[v] | ((v >> z) & 1) << j);
            else
              for (int v = 0; v < (1 << (kTabBits - 5)); ++v) hi[v] = uint8_t(hi[v] | ((v >> (z - 5)) & 1) << j);
          }
        for (size_t x = 0; x < len; ++x) {
          const size_t r = size_t(lo[x & 31] | hi[x >> 5]);
          const double vr = it.m[2 * (r * D + r)], vi = it.m[2 * (r * D + r) + 1];
          const double ar = prod[2 * x], ai = prod[2 * x + 1];
          prod[2 * x] = ar * vr - ai * vi;
          prod[2 * x + 1] = ar * vi + ai * vr;
        }
      }
      float *g = reinterpret_cast<float *>(p + h.table);
      for (size_t x = 0; x < 2 * len; ++x) g[2 * q.goff + x] = float(prod[x]);
    }
    char *dst = p + h.operand;
    for (size_t o = 0; o < ops.size(); ++o) {
      const Item &it = items[size_t(d.dense[o])];
      if (it.k < 5)
        pack_narrow(it.k, it.m, dst);
      else
        pack_gate(it.k, it.m, dst);
      dst += size_t(chunks_of(it.k)) * cb;
    }
    f->S = S;
    f->nops = int(ops.size());
    f->nchunks = nchunks;
    return true;
  }
};

}  // namespace

struct Cutter::Draws {
  const std::vector<Item> &items;
  const Builder B;
  std::vector<char> done;
  size_t from = 0;
  // Dense gates of four bits or fewer with nothing else keep their own
  // sweeps: the layout swaps of sv_plan_swaps are priced by those, and a
  // sequence that gained the same from passes would make them a loss (20 + 20
  // alternating four-bit gates at N=30: 52 ms in passes with or without the
  // swap's 3 ms permutation; 117 and 98 ms in single sweeps).  The price is
  // paid by sequences that no swap helps: 40 four-bit gates, replayed, take 126
  // us in sweeps and 86 in passes at n=12, 269 and 123 at 20, 1023 and 502 at
  // 23.  Of narrow gates on small states and of few gates sweeps are the better
  // choice (launched, 40 two-bit gates at n=14: 103 and 124 us; four four-bit
  // ones: 26 and 31).
  bool plain = true;
  std::vector<int> alone;  // drafted items that run by their own sweeps, the next one last

  Draws(int n, const std::vector<Item> &it, int prec) : items(it), B(n, it, prec), done(it.size(), 0) {
    for (const Item &x : it) plain = plain && !x.diag && x.k <= 4;
  }

  void single(int i, Step *s) {
    s->items.assign(1, i);
    s->pass = Fused();
    done[size_t(i)] = 1;
  }

  bool next(Step *s) {
    if (!alone.empty()) {
      single(alone.back(), s);
      alone.pop_back();
      return true;
    }
    while (from < items.size() && done[from]) ++from;
    if (from == items.size()) return false;
    if (B.n < kMinS || plain || !B.takes(items[from])) {
      single(int(from), s);
      return true;
    }
    Draft d = B.draft(done, from);
    B.trim(d, done);
    if (d.items.empty()) {  // tables that cannot fit on their own
      single(int(from), s);
      return true;
    }
    // one gate, or diagonals alone whose partial sweeps cost less than a pass
    // (on small states, where a launch of 3 us is all they cost, three of them
    // against the 9 us of a pass).  A lone six-bit gate runs as a pass: its sweep
    // and its pass take, in us, launched / replayed as a graph, 26.3/17.6 and
    // 27.7/14.4 at n=16, 41.4/27.5 and 40.3/24.4 at 22, 95/82 and 88/74 at 24,
    // 895/884 and 901/900 at 28, and the pass rounds less (three bf16 pieces
    // against the FP32 sweep's three-product form).
    double cost = 0.0;
    int launches = 0;
    for (int i : d.items) {
      cost += items[size_t(i)].sweep;
      launches += items[size_t(i)].launches;
    }
    s->pass = Fused();
    const bool lone = d.items.size() == 1 && items[size_t(d.items[0])].k != 6;
    if (lone || (d.dense.empty() && (cost <= 1.1 || (B.n <= 18 && launches <= 3))) || !B.emit(d, &s->pass)) {
      alone.assign(d.items.rbegin(), d.items.rend());
      return next(s);
    }
    s->items = std::move(d.items);
    return true;
  }
};

Cutter::Cutter(int n, const std::vector<Item> &items, int prec) : d_(new Draws(n, items, prec)) {}
Cutter::~Cutter() { delete d_; }
bool Cutter::next(Step *s) { return d_->next(s); }

std::vector<Step> build_steps(int n, const std::vector<Item> &items, int prec) {
  std::vector<Step> steps;
  Cutter cut(n, items, prec);
  for (Step s; cut.next(&s);) steps.push_back(std::move(s));
  return steps;
}

}  // namespace pass
}  // namespace sv
