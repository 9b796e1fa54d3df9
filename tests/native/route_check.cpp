// What the library's entry points ask of the GPU, checked on the host (see
// host_runtime.h): which kernels a call launches and when, what it packs and
// copies for them, and what a failed launch leaves.  The argument names a check.
#include "host_runtime.h"

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <functional>
#include <random>

#include "sv.h"
#include "sv_batch.h"
#include "sv_density.h"
#include "sv_plan.h"

namespace {

int failures = 0;

#define CHECK(cond, ...)                                    \
  do {                                                      \
    if (!(cond)) {                                          \
      std::printf("%s:%d: %s: ", __FILE__, __LINE__, #cond); \
      std::printf(__VA_ARGS__);                             \
      std::printf("\n");                                    \
      ++failures;                                           \
    }                                                       \
  } while (0)

struct Gate {
  std::vector<int32_t> t;
  std::vector<double> m;
};

std::mt19937 rng(7);

double uniform() { return std::uniform_real_distribution<double>(-1.0, 1.0)(rng); }

// A dense matrix: what it holds does not matter to the host.
Gate dense(const std::vector<int32_t> &t) {
  Gate g{t, std::vector<double>(size_t(2) << (2 * t.size()))};
  for (double &x : g.m) x = uniform();
  return g;
}

Gate diagonal(const std::vector<int32_t> &t) {
  const size_t D = size_t(1) << t.size();
  Gate g{t, std::vector<double>(2 * D * D, 0.0)};
  for (size_t r = 0; r < D; ++r) {
    const double a = uniform() * 3.0;
    g.m[2 * (r * D + r)] = std::cos(a);
    g.m[2 * (r * D + r) + 1] = std::sin(a);
  }
  return g;
}

Gate swap(int32_t a, int32_t b) {
  Gate g{{a, b}, std::vector<double>(32, 0.0)};
  const int one[4] = {0, 2, 1, 3};
  for (int c = 0; c < 4; ++c) g.m[size_t(2 * (one[c] * 4 + c))] = 1.0;
  return g;
}

std::vector<int32_t> targets(int n, int k) {
  std::vector<int32_t> all(static_cast<size_t>(n));
  for (int i = 0; i < n; ++i) all[size_t(i)] = i;
  std::shuffle(all.begin(), all.end(), rng);
  all.resize(size_t(k));
  return all;
}

std::vector<int32_t> window(int n, int k) {
  std::vector<int32_t> t(static_cast<size_t>(k));
  const int s = std::uniform_int_distribution<int>(0, n - k)(rng);
  for (int i = 0; i < k; ++i) t[size_t(i)] = s + i;
  return t;
}

// A plan whose blocks are the given gates, one each but for one-qubit gates that meet (the cap is one).
sv_plan *plan_of(int n, const std::vector<Gate> &gates) {
  std::vector<int32_t> ks, ts;
  std::vector<double> ms;
  std::vector<int8_t> dg(gates.size(), 0);
  for (const Gate &g : gates) {
    ks.push_back(int32_t(g.t.size()));
    ts.insert(ts.end(), g.t.begin(), g.t.end());
    ms.insert(ms.end(), g.m.begin(), g.m.end());
  }
  sv_plan *p = nullptr;
  const int rc = sv_plan_greedy(n, int(gates.size()), ks.data(), ts.data(), ms.data(), dg.data(), 1, &p);
  int nb = 0;
  sv_plan_num_blocks(p, &nb);
  CHECK(rc == SV_OK && nb <= int(gates.size()) && 2 * nb > int(gates.size()), "rc %d, %d blocks of %zu gates", rc, nb, gates.size());
  return p;
}

void *const kAmps = reinterpret_cast<void *>(uintptr_t(1) << 40);
void *const kWork = reinterpret_cast<void *>(uintptr_t(1) << 44);
void *const kOps = reinterpret_cast<void *>(uintptr_t(1) << 45);

sv_state *state(int n) {
  sv_state *s = nullptr;
  const int rc = sv_alloc(&s, n, kAmps, size_t(8) << n, kWork, sv_workspace_bytes(n), nullptr);
  CHECK(rc == SV_OK, "sv_alloc %d: %s", rc, sv_last_error());
  return s;
}

int apply_list(sv_state *s, const std::vector<Gate> &gates) {
  std::vector<int32_t> ks, ts;
  std::vector<double> ms;
  for (const Gate &g : gates) {
    ks.push_back(int32_t(g.t.size()));
    ts.insert(ts.end(), g.t.begin(), g.t.end());
    ms.insert(ms.end(), g.m.begin(), g.m.end());
  }
  return sv_apply_gates(s, int64_t(gates.size()), ks.data(), ts.data(), ms.data());
}

std::vector<int32_t> layout(sv_state *s, int n) {
  std::vector<int32_t> L(static_cast<size_t>(n));
  sv_get_layout(s, L.data());
  return L;
}

size_t count(const std::string &kernel) {
  size_t c = 0;
  for (const std::string &k : rt::launched()) c += k == kernel;
  return c;
}

// ---------------------------------------------------------------- checks
// An operand is packed once, also where a staging slot is full before it.
void packed_once() {
  const int n = 24;
  for (int k : {6, 7}) {
    std::vector<Gate> gates;
    for (int i = 0; i < 40; ++i) gates.push_back(dense(targets(n, k)));
    for (int prec : {SV_PREC_FP32, SV_PREC_BF16X3}) {
      if (k == 6 && prec == SV_PREC_FP32) continue;  // those run in passes
      sv_state *s = state(n);
      sv_set_option(s, SV_OPT_PRECISION, prec);
      sv_plan *p = plan_of(n, gates);
      rt::start();
      CHECK(sv_run_plan(s, p) == SV_OK, "%s", sv_last_error());
      rt::stop();
      size_t copied = 0;
      for (const rt::Event &e : rt::events()) copied += e.bytes;
      CHECK(rt::launched().size() == gates.size(), "%zu launches", rt::launched().size());
      // the split of a BF16x3 operand works in a few planes of the matrix besides; 8 KiB a gate for its descriptors
      const double want = (prec == SV_PREC_BF16X3 ? 2.2 : 1.1) * double(copied) + 8192.0 * double(gates.size());
      CHECK(double(rt::allocated) < want, "k=%d prec=%d: %zu allocated for %zu of operands", k, prec, rt::allocated, copied);
      sv_plan_free(p);
      sv_free(s);
    }
  }
}

// The device has work after two seven-qubit operands, whatever follows.
void first_copy_early() {
  for (int n : {8, 14, 24}) {
    std::vector<Gate> gates;
    for (int i = 0; i < 12; ++i) gates.push_back(dense(targets(n, 7)));
    sv_state *s = state(n);
    sv_plan *p = plan_of(n, gates);
    rt::start();
    CHECK(sv_run_plan(s, p) == SV_OK, "%s", sv_last_error());
    rt::stop();
    size_t copied = 0;
    for (const rt::Event &e : rt::events()) {
      if (!e.kernel.empty()) break;
      copied += e.bytes;
    }
    CHECK(copied > 0 && copied <= size_t(2) << 17, "n=%d: %zu bytes before the first launch", n, copied);
    sv_plan_free(p);
    sv_free(s);
  }
  // nor for more than four five-bit splits
  std::vector<Gate> gates;
  for (int i = 0; i < 40; ++i) gates.push_back(dense(targets(22, 5)));
  sv_state *s = state(22);
  sv_set_option(s, SV_OPT_PRECISION, SV_PREC_BF16X3);
  sv_plan *p = plan_of(22, gates);
  rt::start();
  CHECK(sv_run_plan(s, p) == SV_OK, "%s", sv_last_error());
  rt::stop();
  for (const rt::Event &e : rt::events()) CHECK(e.bytes <= size_t(4) << 13, "%zu bytes in one copy", e.bytes);
  sv_plan_free(p);
  sv_free(s);
}

// A long plan is launched while it is cut: what is held of it stays bounded, and
// the device does not wait for the whole plan.
void long_plan_bounded() {
  const int n = 30;
  std::vector<Gate> gates;
  for (int i = 0; i < 400; ++i) {
    gates.push_back(dense(window(n, 6)));
    gates.push_back(diagonal(targets(n, 2)));
  }
  sv_state *s = state(n);
  sv_plan *p = plan_of(n, gates);
  rt::start();
  CHECK(sv_run_plan(s, p) == SV_OK, "%s", sv_last_error());
  rt::stop();
  size_t first = 0;
  for (const rt::Event &e : rt::events())
    if (!e.kernel.empty() && !first) first = e.allocated;
  CHECK(count("k_pass") > 50, "%zu passes", count("k_pass"));
  // a slot's worth of passes, the one being packed, 256 bytes a gate for the list
  CHECK(rt::peak < (size_t(2) << 20) + 256 * gates.size(), "%zu bytes held", rt::peak);
  CHECK(first < rt::allocated / 4, "first launch after %zu of %zu bytes", first, rt::allocated);
  sv_plan_free(p);
  sv_free(s);
}

std::vector<Gate> mixed(int n, int most, int gates) {
  std::vector<Gate> out;
  for (int i = 0; i < gates; ++i) {
    const int k = std::uniform_int_distribution<int>(1, most)(rng), kind = std::uniform_int_distribution<int>(0, 9)(rng);
    const std::vector<int32_t> t = kind < 7 ? window(n, k) : targets(n, k), pair = targets(n, 2);
    out.push_back(kind == 0 ? swap(pair[0], pair[1]) : kind < 4 ? diagonal(t) : dense(t));
  }
  return out;
}

// sv_bound_bytes packs nothing, and its answer serves every layout the plan is
// bound from.
void bound_bytes_cheap_and_enough() {
  for (int n : {4, 9, 10, 14, 18, 23})
    for (int most : {1, 2, 6, 8})
      for (int prec : {SV_PREC_FP32, SV_PREC_BF16X3}) {
        if (most > n) continue;
        sv_state *s = state(n);
        sv_set_option(s, SV_OPT_PRECISION, prec);
        sv_plan *p = plan_of(n, mixed(n, most, 60));
        size_t need = 0;
        rt::start();
        CHECK(sv_bound_bytes(s, p, &need) == SV_OK, "%s", sv_last_error());
        rt::stop();
        CHECK(rt::allocated <= 16384, "n=%d k<=%d prec=%d: %zu bytes allocated for an answer of %zu", n, most, prec,
              rt::allocated, need);
        for (int round = 0; round < 12; ++round) {
          sv_bound *b = nullptr;
          const int rc = sv_plan_bind(s, p, kOps, need, &b);
          CHECK(rc == SV_OK, "n=%d k<=%d prec=%d round %d: %s", n, most, prec, round, sv_last_error());
          if (rc == SV_OK) sv_bound_free(b);
          const std::vector<int32_t> L = targets(n, n);
          CHECK(sv_permute_layout(s, L.data()) == SV_OK, "%s", sv_last_error());
        }
        sv_plan_free(p);
        sv_free(s);
      }
}

// A bound plan launches the kernels that the plan launches (on a density handle
// each block's own), counts the same and leaves the same layout, also after the
// plan is gone.
void bound_runs_what_the_plan_runs() {
  struct Handle {
    int n, most, prec;
    bool density;
  };
  const std::vector<Handle> handles = {
      {3, 1, SV_PREC_FP32, false},  {4, 1, SV_PREC_FP32, false},   {12, 1, SV_PREC_FP32, false}, {23, 1, SV_PREC_FP32, false},
      {26, 1, SV_PREC_FP32, false}, {12, 1, SV_PREC_BF16X3, false}, {9, 6, SV_PREC_FP32, false},  {10, 4, SV_PREC_FP32, false},
      {16, 6, SV_PREC_FP32, false}, {24, 8, SV_PREC_FP32, false},  {16, 6, SV_PREC_BF16X3, false}, {6, 6, SV_PREC_FP32, true},
      {9, 6, SV_PREC_FP32, true},   {12, 6, SV_PREC_FP32, true},   {10, 6, SV_PREC_BF16X3, true}};
  for (const Handle &h : handles) {
    const int n = h.density ? 2 * h.n : h.n;
    std::vector<Gate> gates;
    if (h.most == 1) {  // narrow ones: the sequence runs as programs
      for (int i = 0; i < 120; ++i)
        gates.push_back(i % 3 ? dense(targets(n, 1)) : diagonal(targets(n, 2)));
    } else {
      gates = mixed(n, h.most, 80);
    }
    sv_plan *p = plan_of(n, gates);
    auto open = [&]() {
      sv_state *s = nullptr;
      const int rc = h.density ? sv_dm_alloc(&s, h.n, kAmps, sv_dm_state_bytes(h.n), kWork, sv_dm_workspace_bytes(h.n), nullptr)
                               : sv_alloc(&s, n, kAmps, size_t(8) << n, kWork, sv_workspace_bytes(n), nullptr);
      CHECK(rc == SV_OK, "%s", sv_last_error());
      sv_set_option(s, SV_OPT_PRECISION, h.prec);
      return s;
    };
    sv_state *a = open(), *b = open();
    rt::start();
    CHECK(sv_run_plan(a, p) == SV_OK, "%s", sv_last_error());
    rt::stop();
    const std::vector<std::string> want = rt::launched();
    size_t need = 0;
    sv_bound *bound = nullptr;
    CHECK(sv_bound_bytes(b, p, &need) == SV_OK, "%s", sv_last_error());
    CHECK(sv_plan_bind(b, p, kOps, need, &bound) == SV_OK, "%s", sv_last_error());
    sv_plan_free(p);
    rt::start();
    CHECK(sv_bound_run(bound) == SV_OK, "%s", sv_last_error());
    rt::stop();
    const std::vector<std::string> ran = rt::launched();
    CHECK(h.density ? count("k_chain") == 0 && ran.size() >= want.size() : ran == want,
          "n=%d k<=%d prec=%d density=%d: %zu launches bound, %zu as a plan", n, h.most, h.prec, int(h.density), ran.size(),
          want.size());
    CHECK(layout(a, n) == layout(b, n), "n=%d: layouts differ", n);
    sv_stats x, y;
    sv_get_stats(a, &x);
    sv_get_stats(b, &y);
    if (h.density) y.launches = x.launches;
    CHECK(std::memcmp(&x, &y, sizeof(x)) == 0, "n=%d k<=%d density=%d: statistics differ", n, h.most, int(h.density));
    // the graph's kernels are the same ones
    sv_reset(b);
    rt::start();
    CHECK(sv_bound_graph_run(bound) == SV_OK, "%s", sv_last_error());
    rt::stop();
    CHECK(rt::launched() == ran, "n=%d k<=%d: %zu launches captured", n, h.most, rt::launched().size());
    sv_bound_free(bound);
    sv_free(a);
    sv_free(b);
  }
}

// Narrow gates in passes are packed from their own entries, not from a padded matrix.
void narrow_gates_packed_lean() {
  const int n = 20;
  for (int k : {1, 2, 3}) {
    std::vector<Gate> gates;
    for (int i = 0; i < 60; ++i) gates.push_back(dense(window(n, k)));
    for (int i = 0; i < 20; ++i) gates.push_back(diagonal(window(n, 5)));
    sv_state *s = state(n);
    sv_plan *p = plan_of(n, gates);
    size_t need = 0;
    CHECK(sv_bound_bytes(s, p, &need) == SV_OK, "%s", sv_last_error());
    sv_bound *b = nullptr;
    rt::start();
    CHECK(sv_plan_bind(s, p, kOps, need, &b) == SV_OK, "%s", sv_last_error());
    rt::stop();
    size_t copied = 0;
    for (const rt::Event &e : rt::events()) copied += e.bytes;
    // the steps' operands and the copy that is uploaded, and 6 KiB a gate for descriptors and drafts
    CHECK(rt::allocated < 2 * copied + 6144 * gates.size(), "k=%d: %zu allocated for %zu", k, rt::allocated, copied);
    sv_bound_free(b);
    sv_plan_free(p);
    sv_free(s);
  }
}

// A launch that fails leaves the layout and statistics of the gates before it.
void failed_launch_in_a_list() {
  const int n = 12;
  const Gate h2 = dense({2}), h3 = dense({3}), h5 = dense({5}), wide = dense({1, 4, 6, 8, 9});
  // launches: gates 1 and 2 as a program, gate 4 by itself, gates 5 and 7 as a program
  const std::vector<Gate> gates = {swap(0, 1), h2, h3, swap(2, 7), wide, h5, swap(3, 10), h2, swap(4, 5)};
  const size_t ran[] = {1, 4, 5};  // gates known to have run when launch i fails
  for (long fail = 0; fail < 3; ++fail) {
    sv_state *a = state(n), *b = state(n);
    rt::fail_at = fail;
    CHECK(apply_list(a, gates) == SV_ERR_DEVICE, "launch %ld did not fail", fail);
    rt::fail_at = -1;
    CHECK(apply_list(b, std::vector<Gate>(gates.begin(), gates.begin() + long(ran[fail]))) == SV_OK, "%s", sv_last_error());
    CHECK(layout(a, n) == layout(b, n), "launch %ld: the layout is not that of %zu gates", fail, ran[fail]);
    sv_stats x, y;
    sv_get_stats(a, &x);
    sv_get_stats(b, &y);
    CHECK(std::memcmp(&x, &y, sizeof(x)) == 0, "launch %ld: the statistics are not those of %zu gates", fail, ran[fail]);
    sv_free(a);
    sv_free(b);
  }
}

// A staging slot whose copy was issued is released also when a launch fails:
// its next user waits for the copy.
void failed_launch_releases_its_slot() {
  const int n = 20;
  std::vector<Gate> gates;
  for (int i = 0; i < 30; ++i) gates.push_back(dense(targets(n, 6)));
  sv_plan *p = plan_of(n, gates);
  sv_state *s = state(n);
  for (long fail : {0, 1, 3}) {
    for (int one = 0; one < 2; ++one) {
      rt::start();
      rt::fail_at = one ? 0 : fail;
      const int rc = one ? sv_apply_fused(s, gates[0].m.data(), gates[0].t.data(), 6) : sv_run_plan(s, p);
      CHECK(rc == SV_ERR_DEVICE, "launch %ld did not fail", fail);
      rt::fail_at = -1;
      rt::stop();
      size_t copies = 0;
      for (const rt::Event &e : rt::events()) copies += e.kernel.empty();
      CHECK(copies > 0 && copies == rt::recorded, "launch %ld: %zu copies, %zu slots released", fail, copies, rt::recorded);
    }
  }
  sv_free(s);
  sv_plan_free(p);
}

// Of a plan's run that fails nothing is recorded.
void failed_launch_in_a_plan() {
  for (int n : {8, 20}) {
    std::vector<Gate> gates = mixed(n, 6, 60);
    gates.push_back(swap(1, n - 1));
    sv_plan *p = plan_of(n, gates);
    sv_state *s = state(n);
    sv_stats x, y;
    sv_get_stats(s, &x);
    const std::vector<int32_t> L = layout(s, n);
    for (long fail : {0, 2, 5}) {
      rt::fail_at = fail;
      CHECK(sv_run_plan(s, p) == SV_ERR_DEVICE, "launch %ld did not fail", fail);
      rt::fail_at = -1;
      sv_get_stats(s, &y);
      CHECK(std::memcmp(&x, &y, sizeof(x)) == 0, "n=%d launch %ld: statistics moved", n, fail);
      CHECK(layout(s, n) == L, "n=%d launch %ld: layout moved", n, fail);
    }
    sv_free(s);
    sv_plan_free(p);
  }
}

// The records of a small batch go to the device by one copy, circuits in passes included.
void small_batch_one_copy() {
  for (int n : {6, 15, 18}) {
    std::vector<int32_t> kinds, qubits;
    std::vector<double> mats;
    for (int q = 0; q < n; ++q) {
      kinds.push_back(SV_BATCH_GATE_1Q);
      qubits.insert(qubits.end(), {q, -1});
      for (int e = 0; e < 8; ++e) mats.push_back(uniform());
    }
    sv_batch_circuit c{};
    c.n_qubits = n;
    c.n_gates = int(kinds.size());
    c.kinds = kinds.data();
    c.qubits = qubits.data();
    c.mats = mats.data();
    const int64_t off = 0;
    sv_batch_prepared *p = nullptr;
    rt::start();
    CHECK(sv_batch_prepare(1, &c, size_t(8) << n, &off, nullptr, kWork, sv_batch_workspace_bytes(1, &c), nullptr, &p) == SV_OK,
          "%s", sv_last_error());
    rt::stop();
    CHECK(rt::events().size() == 1, "n=%d: %zu copies", n, rt::events().size());
    sv_batch_prepared_free(p);
  }
}

const std::map<std::string, std::function<void()>> kChecks = {
    {"packed_once", packed_once},
    {"bound_bytes_cheap_and_enough", bound_bytes_cheap_and_enough},
    {"bound_runs_what_the_plan_runs", bound_runs_what_the_plan_runs},
    {"narrow_gates_packed_lean", narrow_gates_packed_lean},
    {"failed_launch_in_a_list", failed_launch_in_a_list},
    {"failed_launch_in_a_plan", failed_launch_in_a_plan},
    {"small_batch_one_copy", small_batch_one_copy},
    {"failed_launch_releases_its_slot", failed_launch_releases_its_slot},
    {"long_plan_bounded", long_plan_bounded},
    {"first_copy_early", first_copy_early},
};

}  // namespace

int main(int argc, char **argv) {
  for (int i = 1; i < argc; ++i) {
    const auto it = kChecks.find(argv[i]);
    if (it == kChecks.end()) {
      std::printf("no check %s\n", argv[i]);
      return 2;
    }
    it->second();
  }
  if (failures == 0) std::printf("route checks passed\n");
  return failures != 0;
}
