// Which kernel the host code gives a launch to, and what it assumes about device memory between calls, without a GPU:
// dadam_host.cpp linked against a modelled HIP runtime (memory is the host's) and modelled launchers that note what they
// were asked to do.  Launches on a stream that is "being captured" are recorded and run when the graph is replayed; a
// launch can be made to fail.  Prints one line per question; tests/test_host_abi.py holds the answers.
#include "dadam.h"
#include "dadam_internal.h"
#include <hip/hip_runtime_api.h>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <functional>
#include <string>
#include <vector>

// ---- modelled runtime ----
static bool capturing = false;
static std::vector<std::function<void()>> recorded;
static const char* fail_launch = nullptr;  // name of the launcher whose next call fails
static std::string route, how;  // how: the shape of the tile's workgroup, the order of a row launch
static uint32_t shares = 0;  // workgroups that share the rows of a loop's tile
static bool streams = false; // accesses carry the non-temporal hint
static bool wide_search = false;  // all lanes search the segments
static std::string walk;     // by the map or by how many segments
static void note_walk(const dadam::StepArgs& a) { walk = a.map ? a.n_seg == 1 ? "map" : "map and segments" : std::to_string(a.n_seg) + " segments"; }
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeNumberOfXccs ? 8 : 160 * 1024;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = malloc(n); memset(*p, 0xA5, n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "modelled"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) {
  *s = capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
}
static int enqueue(const char* name, std::function<void()> work) {
  if (fail_launch && !strcmp(fail_launch, name)) { fail_launch = nullptr; return (int)hipErrorLaunchFailure; }
  if (capturing) recorded.push_back(work); else work();
  return 0;
}
namespace dadam {
static double static_scratch[kConsensusPartials];
int launch_tile(int, int, Phase phase, TileShape shape, const StepArgs& a, uint32_t, uint32_t, void*) {
  how = std::to_string(shape.waves) + "x" + std::to_string(shape.ut) + (shape.nontemporal ? " streaming" : "") + " block " +
        std::to_string(a.xcd_block) + (a.d == 0 ? " cut by elements" : "");
  route = a.n_loops > 0 ? "loop" + std::to_string(shape.waves) : "tile";
  shares = a.n_loops > 0 ? a.loop_shares : 0;
  streams = shape.nontemporal;
  wide_search = a.wide_search != 0;
  note_walk(a);
  if (shares > 1 && shape.nontemporal && phase == kMixOnly) return (int)hipErrorInvalidDeviceFunction;  // there is no such kernel
  double* p = a.partials;
  return enqueue("tile", [=] { if (phase == kMixConsensus) p[7] += 3.0; });  // the modelled error of any pass is 3
}
int launch_direct(int, int, Phase, bool nontemporal, bool, bool whole_items, const StepArgs& a, uint32_t, void*) {
  streams = nontemporal;
  note_walk(a);
  how = std::string(a.order == kOrderDieBlocks ? "blocks, runs of " + std::to_string(a.die_run) : a.order == kOrderDieGroups ? "groups" : "linear") +
        (whole_items ? ", whole items" : "") + (a.d == 0 ? " cut by elements" : "");
  route = a.order == kOrderDieBlocks ? "direct-blocks" : a.order == kOrderDieGroups ? "direct-groups" : "direct";
  if (whole_items) route += " whole";
  return enqueue("direct", [] {});
}
int launch_accumulate(int, Phase, bool nontemporal, bool whole_items, const StepArgs& a, uint32_t, void*, int) {
  streams = nontemporal;
  note_walk(a);
  how = (a.order == kOrderDieBlocks ? "blocks, runs of " + std::to_string(a.die_run) : std::string("linear")) + (whole_items ? ", whole items" : "");
  route = whole_items ? "whole" : "pieces";
  return enqueue("accumulate", [] {});
}
int launch_consensus_zero(double* p, void*) {
  return enqueue("zero", [=] { for (uint32_t i = 0; i < kConsensusPartials; ++i) p[i] = 0.0; });
}
int launch_consensus_sum(double* p, double* out, void*) {
  return enqueue("sum", [=] {
    double s = 0.0;
    for (uint32_t i = 0; i < kConsensusPartials; ++i) { s += p[i]; p[i] = 0.0; }
    *out = s;
  });
}
int static_partials(double** out, uint32_t* capacity) { *out = static_scratch; *capacity = kConsensusPartials; return 0; }
int vec_elems(int xdt) { return xdt == DADAM_BF16 ? 8 : 4; }
bool tile_shape_supported(TileShape s) {
  if (s.ut == 2 && (s.waves == 8 || s.waves == 16)) return s.nontemporal;
  if (s.ut == 1 && s.waves == 16) return true;
  return (s.waves == 4 && s.ut == 2) || ((s.waves == 4 || s.waves == 8) && s.ut == 1);
}
}  // namespace dadam

// ---- a handle and its buffers (addresses only: nothing reads or writes through them) ----
struct Rows { std::vector<int32_t> ptr{0}, col; std::vector<float> w; };
static void add_row(Rows& r, const std::vector<int32_t>& cols, float tilt = 0.f) {  // tilt: unequal weights
  const float each = 1.0f / (float)cols.size();
  for (size_t k = 0; k < cols.size(); ++k) {
    r.col.push_back(cols[k]);
    r.w.push_back(each + (cols.size() < 2 ? 0.f : k == 0 ? tilt : k == 1 ? -tilt : 0.f));
  }
  r.ptr.push_back((int32_t)r.col.size());
}
struct Sim {
  dadam_handle* h = nullptr;
  uint32_t R, C;
  size_t pitch;
  std::vector<const void*> xs, g;
  std::vector<void*> xd;
  std::vector<float*> m, v, b;
  Sim(uint32_t rows, uint32_t cols, const std::vector<dadam_tensor_desc>& ts, const Rows& lists, uint32_t dtype = DADAM_F32)
      : R(rows), C(cols) {
    dadam_config cfg{};
    cfg.abi_version = DADAM_ABI_VERSION; cfg.n_rows = R; cfg.n_cols = C;
    cfg.d = ts.back().offset_elems + ts.back().numel; cfg.n_tensors = (uint32_t)ts.size(); cfg.tensors = ts.data();
    cfg.param_dtype = cfg.grad_dtype = dtype; cfg.lr = 1e-3f; cfg.beta1 = 0.9f; cfg.beta2 = 0.999f; cfg.eps = 1e-8f;
    cfg.accum_s = 2; cfg.beta_vhat = -1.f; cfg.device = 0;
    if (dadam_init(&cfg, &h) != DADAM_OK) { printf("init failed: %s\n", dadam_last_error(nullptr)); exit(1); }
    if (dadam_set_topology(h, 0, lists.ptr.data(), lists.col.data(), lists.w.data(), nullptr) != DADAM_OK) {
      printf("topology refused: %s\n", dadam_last_error(h)); exit(1);
    }
    pitch = (cfg.d * 4 + 4095) / 4096 * 4096;
    size_t k = 0;
    auto address = [&] { return (char*)(1ull << 30) + pitch * k++; };
    for (uint32_t c = 0; c < C; ++c) xs.push_back(address());
    for (uint32_t i = 0; i < R; ++i) { xd.push_back(address()); m.push_back((float*)address()); v.push_back((float*)address()); }
    for (uint32_t i = 0; i < R; ++i) { b.push_back((float*)address()); g.push_back(address()); }
  }
  ~Sim() { dadam_destroy(h); }
  void bind() {
    dadam_buffers bufs{xs.data(), xd.data(), m.data(), v.data(), b.data()};
    if (dadam_bind(h, &bufs) != DADAM_OK) { printf("bind refused: %s\n", dadam_last_error(h)); exit(1); }
  }
  std::string step(uint32_t flags, uint32_t begin = 0, uint32_t end = ~0u) {
    route = "nothing";
    const int rc = end == ~0u ? dadam_gossip_step(h, 0, g.data(), 1, flags, nullptr)
                              : dadam_gossip_step_range(h, 0, g.data(), 1, flags, begin, end, nullptr);
    return rc == DADAM_OK ? route : "error " + std::to_string(rc);
  }
  std::string mix(uint32_t flags) {
    route = "nothing";
    const int rc = dadam_mix(h, 0, flags, nullptr);
    return rc == DADAM_OK ? route : "error " + std::to_string(rc);
  }
};
static void say(const char* what, const std::string& answer) { printf("%s: %s\n", what, answer.c_str()); }

// Row 0 is updated in place in source 1, which only row 0 lists; row 1's decay reads source 1 all the same.
static void foreign_in_place() {
  Rows shared, alone;
  for (int i = 0; i < 16; ++i) {
    add_row(shared, i == 0 ? std::vector<int32_t>{0, 1, 2} : i == 1 ? std::vector<int32_t>{2, 3, 4} : std::vector<int32_t>{i, i == 15 ? 2 : i + 1, 0});
    add_row(alone, {i == 0 ? 1 : i == 1 ? 0 : i});
  }
  const std::vector<dadam_tensor_desc> ts = {{0, 700, 0.1f, 0}, {700, 900, 0.f, 0}};
  Sim s(16, 16, ts, shared), a(16, 16, ts, alone);
  for (Sim* x : {&s, &a}) { x->xd[0] = const_cast<void*>(x->xs[1]); x->bind(); }
  const uint32_t F = DADAM_FUSE_ACCUM, D = DADAM_FORCE_DIRECT;
  say("shared, step", s.step(F));
  say("shared, update only", s.step(0));
  say("shared, range with decay", s.step(F, 0, 1));
  say("shared, range without decay", s.step(F, 1, 2));
  say("shared, mixing", s.mix(0));
  say("shared, step forced direct", s.step(F | D));
  say("shared, range without decay forced direct", s.step(F | D, 1, 2));
  say("shared, mixing forced direct", s.mix(D));
  say("shared, step forced tile", s.step(F | DADAM_FORCE_TILE));
  say("alone, step", a.step(F));
  say("alone, range without decay", a.step(F, 1, 2));
  say("alone, step forced direct", a.step(F | D));
  say("alone, mixing", a.mix(0));
  Sim own(16, 16, ts, shared);  // every row in place in its own buffer, which others read: the tile as ever
  for (int i = 0; i < 16; ++i) own.xd[i] = const_cast<void*>(own.xs[i]);
  own.bind();
  say("all in place, step", own.step(F));
  Sim solo(1, 3, {{0, 700, 0.1f, 0}}, [] { Rows r; add_row(r, {0, 1, 2}); return r; }());  // one node's share
  solo.xd[0] = const_cast<void*>(solo.xs[0]);
  solo.bind();
  say("one row in place with decay", solo.step(F));
  say("one row in place with decay forced direct", solo.step(F | D));
}

// Consensus passes over partial sums that live in (modelled) device memory: every pass must report 3.
static void consensus() {
  Rows ring;
  for (int i = 0; i < 4; ++i) add_row(ring, {i, (i + 1) % 4, (i + 3) % 4});
  const std::vector<dadam_tensor_desc> ts = {{0, 700, 0.f, 0}};
  auto pass = [](Sim& s, double* out, const char* failing = nullptr) {
    *out = -1.0;
    fail_launch = failing;
    const int rc = dadam_mix_consensus(s.h, 0, 0, out, nullptr);
    fail_launch = nullptr;
    return rc;
  };
  auto run = [](std::vector<std::function<void()>>& graph) { for (auto& launch : graph) launch(); };
  auto record = [&](Sim& s, double* out) {
    capturing = true;
    recorded.clear();
    (void)pass(s, out);
    capturing = false;
    return recorded;
  };
  double out[8];
  {
    Sim s(4, 4, ts, ring);
    s.bind();
    pass(s, &out[0]);
    pass(s, &out[1]);
    say("one after the other", std::to_string(out[0]) + " " + std::to_string(out[1]));
    auto graph = record(s, &out[2]);
    run(graph);
    const double first = out[2];
    run(graph);
    pass(s, &out[3]);
    say("two replays, then a pass", std::to_string(first) + " " + std::to_string(out[2]) + " " + std::to_string(out[3]));
  }
  for (const char* failing : {"zero", "tile", "sum"}) {
    Sim s(4, 4, ts, ring);
    s.bind();
    auto graph = record(s, &out[0]);
    const int rc = pass(s, &out[1], failing);
    run(graph);
    say((std::string("replay after a pass that failed in ") + failing).c_str(), (rc == DADAM_OK ? "accepted " : "refused ") + std::to_string(out[0]));
  }
  {
    Sim s(4, 4, ts, ring);
    s.bind();
    pass(s, &out[0], "sum");
    auto graph = record(s, &out[1]);  // recorded, not yet run
    pass(s, &out[2]);
    run(graph);
    pass(s, &out[3]);
    say("pass behind a recorded one after a failed one", std::to_string(out[2]) + " " + std::to_string(out[1]) + " " + std::to_string(out[3]));
  }
  {
    Sim s(4, 4, ts, ring);
    s.bind();
    (void)dadam_mix_consensus_static(s.h, 0, 0, &out[0], nullptr);
    pass(s, &out[1]);
    (void)dadam_mix_consensus_static(s.h, 0, 0, &out[2], nullptr);
    say("static array in between", std::to_string(out[0]) + " " + std::to_string(out[1]) + " " + std::to_string(out[2]));
  }
}

static Rows complete(int n) {
  Rows r;
  std::vector<int32_t> all;
  for (int c = 0; c < n; ++c) all.push_back(c);
  for (int i = 0; i < n; ++i) add_row(r, all);
  return r;
}
static Rows halves(int n) {  // loops of n/2, n/4, n/4 rows
  Rows r;
  const int from[] = {0, n / 2, n / 2 + n / 4, n};
  for (int l = 0; l < 3; ++l) {
    std::vector<int32_t> own;
    for (int c = from[l]; c < from[l + 1]; ++c) own.push_back(c);
    for (size_t i = 0; i < own.size(); ++i) add_row(r, own);
  }
  return r;
}

// Which launches of an All-Reduce loop, or of several, share one sum.
static void loops() {
  struct { const char* kind; int rows; uint64_t tiles; } cases[] = {
      {"complete", 15, 256}, {"complete", 16, 256}, {"complete", 16, 257}, {"complete", 16, 512}, {"complete", 16, 513},
      {"complete", 28, 257}, {"complete", 28, 512}, {"complete", 28, 513}, {"complete", 32, 1024}, {"complete", 32, 1025}, {"complete", 55, 1761},
      {"complete", 56, 4000}, {"complete", 68, 4000}, {"halves", 32, 256}, {"halves", 32, 257}, {"halves", 64, 170},
      {"halves", 64, 171}, {"halves", 64, 682}, {"halves", 64, 683}, {"halves", 72, 4000}, {"halves", 24, 100}};
  for (const auto& c : cases)
    for (uint32_t dtype : {DADAM_F32, DADAM_BF16}) {
      const uint64_t d = c.tiles * (dtype == DADAM_BF16 ? 512 : 256);
      const Rows rows = !strcmp(c.kind, "complete") ? complete(c.rows) : halves(c.rows);
      Sim plain(c.rows, c.rows, {{0, d - 300, 0.f, 0}, {d - 300, 300, 0.f, 0}}, rows, dtype);
      Sim decay(c.rows, c.rows, {{0, d - 300, 0.1f, 0}, {d - 300, 300, 0.1f, 0}}, rows, dtype);
      plain.bind();
      decay.bind();
      const uint32_t F = DADAM_FUSE_ACCUM;
      std::string ranges = decay.step(F, 0, 1);  // the sum's order does not depend on the range
      const bool shared = decay.step(F).substr(0, 4) == "loop";
      auto differs = [&](const std::string& r) { return (r.substr(0, 4) == "loop") != shared; };
      ranges = differs(ranges) || differs(decay.step(F, 1, 2)) || differs(decay.step(0)) ? " but ranges differ" : "";
      say((std::string(c.kind) + std::to_string(c.rows) + " " + std::to_string(c.tiles) + (dtype == DADAM_BF16 ? " bf16" : " f32")).c_str(),
          plain.step(F) + " " + plain.mix(0) + " decay " + decay.step(F) + " " + decay.mix(0) + ranges);
    }
}

// Handles whose size says that they stream and whose tensors cover few tiles: one tensor of 20000 elements in 2.3e7 of all rows.
static void sparse_loops() {
  for (int n : {32, 64, 96})
    for (uint32_t dtype : {DADAM_F32, DADAM_BF16}) {
      const uint64_t d = 23000000 / n / 8 * 8 + 8;
      Sim s(n, n, {{d / 2 / 8 * 8, 20000, 0.f, 0}, {d, 0, 0.f, 0}}, complete(n), dtype);
      s.bind();
      auto told = [](const std::string& r) { return r + " shared by " + std::to_string(shares) + (how.find("streaming") != std::string::npos ? " streaming" : ""); };
      const std::string step = told(s.step(DADAM_FUSE_ACCUM)), update = told(s.step(0)), mix = told(s.mix(0));
      say((std::to_string(n) + (dtype == DADAM_BF16 ? " bf16" : " f32")).c_str(), step + ", update " + update + ", mix " + mix);
    }
}

// How many workgroups take the rows of a loop's tile: fused step, update of the first tensor alone, mixing, and a step and mixing of rows updated in place.
static void loop_shares() {
  struct { const char* kind; int rows; uint64_t tiles; uint32_t dtype; bool cut; } cases[] = {
      {"complete", 16, 128, DADAM_F32, true}, {"complete", 17, 128, DADAM_F32, true}, {"complete", 17, 129, DADAM_F32, true}, {"complete", 32, 24, DADAM_F32, true},
      {"complete", 31, 24, DADAM_F32, true}, {"complete", 33, 85, DADAM_F32, true}, {"complete", 33, 86, DADAM_F32, true}, {"complete", 64, 64, DADAM_BF16, true},
      {"complete", 64, 129, DADAM_F32, true}, {"complete", 96, 42, DADAM_F32, true}, {"complete", 96, 40, DADAM_BF16, true}, {"complete", 100, 36, DADAM_BF16, true},
      {"halves", 96, 42, DADAM_F32, true}, {"halves", 96, 16, DADAM_F32, true}, {"halves", 96, 43, DADAM_F32, true},
      {"complete", 32, 2900, DADAM_F32, true}, {"complete", 95, 1100, DADAM_F32, true}, {"halves", 128, 900, DADAM_F32, true},
      {"complete", 128, 768, DADAM_F32, true}, {"complete", 128, 769, DADAM_F32, false}, {"complete", 128, 960, DADAM_F32, false}, {"complete", 128, 961, DADAM_F32, false},
      {"complete", 128, 961, DADAM_F32, true}, {"complete", 128, 1152, DADAM_F32, true}, {"complete", 128, 1153, DADAM_F32, true}, {"complete", 96, 1536, DADAM_F32, true},
      {"complete", 96, 1537, DADAM_F32, true}, {"complete", 96, 1728, DADAM_F32, true}, {"complete", 96, 1729, DADAM_F32, true}, {"complete", 96, 2305, DADAM_F32, true},
      {"complete", 97, 512, DADAM_BF16, true}, {"complete", 97, 513, DADAM_BF16, false}, {"complete", 97, 640, DADAM_BF16, false}, {"complete", 97, 641, DADAM_BF16, false},
      {"complete", 97, 768, DADAM_BF16, true}, {"complete", 97, 769, DADAM_BF16, true}, {"complete", 97, 1024, DADAM_BF16, true}, {"complete", 97, 1152, DADAM_BF16, true},
      {"complete", 97, 1153, DADAM_BF16, true}, {"complete", 97, 1664, DADAM_BF16, false}, {"complete", 97, 2049, DADAM_BF16, false}};
  for (const auto& c : cases) {
    const uint64_t T = c.dtype == DADAM_BF16 ? 512 : 256, d = c.tiles * T - (c.cut ? 6 : 0), half = d / 2 / T * T;
    const std::vector<dadam_tensor_desc> ts = {{0, half, 0.f, 0}, {half, d - half, 0.f, 0}};
    std::string answers;
    for (bool in_place : {false, true}) {
      Sim s(c.rows, c.rows, ts, !strcmp(c.kind, "complete") ? complete(c.rows) : halves(c.rows), c.dtype);
      if (in_place) s.xd[c.rows - 1] = const_cast<void*>(s.xs[c.rows - 1]);
      s.bind();
      if (in_place) answers += " |";
      auto told = [&answers](const std::string& r) { answers += " " + (r.substr(0, 4) == "loop" ? std::to_string(shares) : r); };
      told(s.step(DADAM_FUSE_ACCUM));
      if (!in_place) told(s.step(0, 0, 1));
      told(s.mix(0));
    }
    say((std::string(c.kind) + std::to_string(c.rows) + " " + std::to_string(c.tiles) + (c.dtype == DADAM_BF16 ? " bf16" : " f32") + (c.cut ? "" : " whole")).c_str(), answers.substr(1));
  }
  for (uint64_t tiles : {1030, 1300}) {  // of two segments: 8 wavefronts to a workgroup, two and one of them to a tile
    const uint64_t half = tiles * 256;
    Sim s(97, 97, {{0, half - 8, 0.f, 0}, {half, half - 8, 0.f, 0}}, complete(97), DADAM_BF16);
    s.bind();
    s.step(DADAM_FUSE_ACCUM);
    say(("wide search, " + std::to_string(tiles)).c_str(), std::to_string(shares) + (wide_search ? " yes" : " no"));
  }
}

// Layouts of tensors with gaps of a few elements between them: what goes by the map, what by the segments, and which of it by whole items.
static void maps() {
  struct { const char* kind; int rows, degree; uint32_t dtype; uint64_t each, total, gap; } cases[] = {
      {"share", 1, 3, DADAM_F32, 1100, 30000, 4}, {"share", 1, 3, DADAM_BF16, 1100, 30000, 4}, {"ring", 8, 3, DADAM_BF16, 1100, 2400000, 4},
      {"ring", 8, 3, DADAM_F32, 1100, 2400000, 8}, {"ring", 8, 3, DADAM_F32, 70000, 2400000, 4},
      {"ring", 40, 2, DADAM_F32, 1100, 120000000, 4}, {"ring", 40, 2, DADAM_F32, 1100, 120000000, 12}, {"ring", 48, 2, DADAM_BF16, 1100, 120000000, 4}, {"ring", 100, 2, DADAM_F32, 1100, 120000000, 4},
      {"complete", 32, 32, DADAM_F32, 16380, 205000000, 4}, {"complete", 32, 32, DADAM_F32, 16388, 205000000, 4}, {"complete", 32, 32, DADAM_F32, 16388, 190000000, 4},
      {"complete", 32, 32, DADAM_F32, 20484, 81000000, 4}, {"complete", 32, 32, DADAM_F32, 20476, 81000000, 4}, {"complete", 32, 32, DADAM_F32, 20484, 79000000, 4},
      {"complete", 64, 64, DADAM_BF16, 20484, 81000000, 4}, {"halves", 64, 0, DADAM_F32, 2564, 205000000, 4}, {"halves", 64, 0, DADAM_F32, 2556, 205000000, 4},
      {"complete", 96, 96, DADAM_F32, 2052, 205000000, 4}, {"complete", 96, 96, DADAM_F32, 2044, 205000000, 4}, {"complete", 96, 96, DADAM_F32, 6148, 205000000, 4},
      {"complete", 128, 128, DADAM_F32, 6148, 205000000, 4}, {"complete", 96, 96, DADAM_BF16, 8200, 205000000, 4}, {"complete", 96, 96, DADAM_BF16, 8184, 205000000, 4},
      {"ring", 18, 3, DADAM_BF16, 20004, 205000000, 4}, {"ring", 24, 3, DADAM_BF16, 4100, 205000000, 4}, {"ring", 24, 3, DADAM_BF16, 4092, 205000000, 4},
      {"ring", 32, 3, DADAM_BF16, 2564, 205000000, 4}, {"ring", 32, 3, DADAM_BF16, 2556, 205000000, 4}, {"ring", 48, 3, DADAM_BF16, 12292, 101000000, 4},
      {"ring", 48, 3, DADAM_BF16, 12284, 101000000, 4}, {"ring", 48, 3, DADAM_BF16, 20004, 79000000, 4}, {"ring", 72, 3, DADAM_BF16, 20004, 205000000, 4},
      {"ring", 32, 3, DADAM_F32, 20004, 205000000, 4}, {"ring", 96, 7, DADAM_F32, 5124, 205000000, 4}, {"ring", 96, 7, DADAM_F32, 5116, 205000000, 4},
      {"ring", 72, 7, DADAM_F32, 5124, 205000000, 4}, {"ring", 96, 7, DADAM_F32, 5124, 190000000, 4}};
  for (const auto& c : cases) {
    Rows r;
    if (c.degree == 0) r = halves(c.rows);
    for (int i = 0; i < c.rows && c.degree > 0; ++i) {
      std::vector<int32_t> cols;
      for (int k = 0; k < c.degree; ++k) cols.push_back(c.rows == 1 ? k : (i + k) % c.rows);
      add_row(r, cols);
    }
    std::vector<dadam_tensor_desc> ts;
    for (uint64_t at = 0; at < c.total / c.rows; at += c.each + c.gap) ts.push_back({at, c.each, 0.f, 0});
    ts.push_back({ts.back().offset_elems + c.each + c.gap, 0, 0.f, 0});  // d is a multiple of four
    Sim s(c.rows, c.rows == 1 ? 3 : c.rows, ts, r, c.dtype);
    s.bind();
    const std::string n = std::to_string(ts.size() - 1) + " segments";
    std::string answers;
    auto told = [&](const std::string& what) {
      answers += (answers.empty() ? "" : ", ") + (what.substr(0, 5) == "error" ? what : walk == n ? "segments" : walk) + (what.find("whole") != std::string::npos ? " whole" : "");
    };
    told(s.step(DADAM_FUSE_ACCUM));
    told(s.mix(0));
    double out = 0.0;
    if (c.rows > 1) told(dadam_mix_consensus(s.h, 0, 0, &out, nullptr) == DADAM_OK ? route : "error");
    told(dadam_accumulate(s.h, s.g.data(), 1, nullptr) == DADAM_OK ? route : "error");
    say((std::string(c.kind) + std::to_string(c.rows) + " of " + std::to_string(c.degree) + (c.dtype == DADAM_BF16 ? " bf16 " : " f32 ") + std::to_string(c.each) + "+" + std::to_string(c.gap) +
         " " + std::to_string(c.total / 1000000) + "e6").c_str(), answers);
  }
}

// The same of given layouts: lines of a name, rows, sources, whether bfloat16, d, and of every tensor its offset, elements and decay.
static void map_of() {
  char name[64];
  unsigned rows, cols, wide, n;
  unsigned long long d;
  while (scanf("%63s %u %u %u %llu %u", name, &rows, &cols, &wide, &d, &n) == 6) {
    std::vector<dadam_tensor_desc> ts;
    for (unsigned k = 0; k < n; ++k) {
      unsigned long long offset, numel;
      float decay;
      if (scanf("%llu %llu %f", &offset, &numel, &decay) != 3) exit(1);
      ts.push_back({offset, numel, decay, 0});
    }
    ts.push_back({d, 0, 0.f, 0});
    Rows r;
    for (unsigned i = 0; i < rows; ++i) {
      std::vector<int32_t> of;
      for (unsigned k = 0; k < (cols < 3 ? cols : 3u); ++k) of.push_back((int32_t)((i + k) % cols));
      add_row(r, of);
    }
    Sim s(rows, cols, ts, r, wide ? DADAM_BF16 : DADAM_F32);
    s.bind();
    std::string answers = s.step(DADAM_FUSE_ACCUM).substr(0, 5) == "error" ? "error" : walk;
    if (dadam_accumulate(s.h, s.g.data(), 1, nullptr) == DADAM_OK) answers += ", " + walk;
    if (s.mix(0).substr(0, 5) != "error") answers += ", " + walk;
    say(name, answers);
  }
}

// Steps of few rows on both sides of 344 MB of what they touch.
static void few_rows() {
  struct { const char* name; uint32_t rows, cols, read, dtype, bytes; bool in_place; uint64_t outside; } cases[] = {
      {"share of 3", 1, 3, 3, DADAM_F32, 28, true, 0},          // sources (the first is the output), gradient, two moments, accumulator
      {"share of 3, apart", 1, 3, 3, DADAM_F32, 32, false, 0},
      {"share of 3, one neighbour", 1, 3, 2, DADAM_F32, 24, true, 0},
      {"share of 64, 3 read", 1, 64, 3, DADAM_F32, 28, true, 0},
      {"share of 3, bf16", 1, 3, 3, DADAM_BF16, 20, true, 0},
      {"2 rows", 2, 2, 2, DADAM_F32, 48, false, 0},
      {"2 rows in place", 2, 2, 2, DADAM_F32, 40, true, 0},
      {"3 rows, bf16", 3, 3, 3, DADAM_BF16, 54, false, 0},
      {"share of 3, a part of d", 1, 3, 3, DADAM_F32, 28, true, 3000000},
      {"4 rows", 4, 4, 3, DADAM_F32, 92, false, 0}};
  for (const auto& c : cases) {
    std::string answers;
    for (uint64_t more : {0, 1}) {
      const uint64_t n = (344ull << 20) / c.bytes + more;
      Rows r;
      for (uint32_t i = 0; i < c.rows; ++i) {
        std::vector<int32_t> cols;
        for (uint32_t k = 0; k < c.read; ++k) cols.push_back((int32_t)((i + k) % c.cols));
        add_row(r, cols);
      }
      Sim s(c.rows, c.cols, {{0, n, 0.f, 0}, {n + c.outside, 0, 0.f, 0}}, r, c.dtype);
      if (c.in_place)
        for (uint32_t i = 0; i < c.rows; ++i) s.xd[i] = const_cast<void*>(s.xs[i]);
      s.bind();
      auto told = [&answers](const std::string& route) { answers += route.substr(0, 5) == "error" ? " error" : streams ? " yes" : " no"; };
      told(s.step(DADAM_FUSE_ACCUM));
      told(s.step(0, 0, 1));
      told(s.mix(0));
      told(dadam_accumulate(s.h, s.g.data(), 1, nullptr) == DADAM_OK ? "" : "error");
      dadam_plan_info info;
      dadam_get_plan_info(s.h, &info);
      answers += " plan " + std::to_string(info.streaming) + (more ? "" : ",");
    }
    say(c.name, answers.substr(1));
  }
}

// How many tiles a launch of rows that share sources may have and still go row by row.
static void few() {
  for (uint32_t dtype : {DADAM_F32, DADAM_BF16})
    for (int degree : {3, 12, 13, 24, 25, 64}) {
      Rows r;
      for (int i = 0; i < 64; ++i) {
        std::vector<int32_t> cols;
        for (int k = 0; k < degree; ++k) cols.push_back((i + k) % 64);
        add_row(r, cols, 0.001f * (float)(i % 7));
      }
      uint64_t most = 0;
      for (uint64_t tiles = 120; tiles <= 260; ++tiles) {
        Sim s(64, 64, {{0, tiles * (dtype == DADAM_BF16 ? 512 : 256), 0.f, 0}}, r, dtype);
        s.bind();
        if (s.step(DADAM_FUSE_ACCUM) != "tile") most = tiles;
      }
      say(((dtype == DADAM_BF16 ? "bf16 " : "f32 ") + std::to_string(degree)).c_str(), std::to_string(most));
    }
}

// The order in which large direct launches of rows in pairs walk rows and pieces: from how many million elements of all
// rows together a step keeps a piece's rows on one die.
static void die_order() {
  for (uint32_t dtype : {DADAM_F32, DADAM_BF16})
    for (int n : {32, 33, 63, 64, 71, 72, 79, 80, 95, 96, 128, 129, 160}) {
      Rows r;
      for (int i = 0; i < n; ++i) add_row(r, {i, (i + 1) % n});
      uint32_t from = 0;
      std::string other = "none";
      uint32_t whole_from = 0;
      for (uint32_t million = 90; million <= 1200 && !from; million += 5) {
        const uint64_t d = (million * 1000000ull + n - 1) / n;
        Sim s(n, n, {{0, d, 0.f, 0}}, r, dtype);
        s.bind();
        const std::string step = s.step(DADAM_FUSE_ACCUM);
        if (step == "direct-blocks") from = million; else other = step;
        if (step == "direct-groups whole" && !whole_from) whole_from = million;
        if (s.mix(0) != "direct-groups whole") other = "mixing " + s.mix(0);
      }
      say(((dtype == DADAM_BF16 ? "bf16 " : "f32 ") + std::to_string(n)).c_str(), other + ", whole items from " + std::to_string(whole_from) + ", blocks from " + std::to_string(from));
    }
}

// From how many million elements of all rows together accumulation goes by whole items.
static void accumulation() {
  for (int n : {1, 32, 33, 64, 65, 80, 81, 127, 128, 160}) {
    Rows r;
    for (int i = 0; i < n; ++i) add_row(r, {i});
    uint32_t from = 0;
    for (uint32_t million = 20; million <= 400 && !from; million += 5) {
      Sim s(n, n, {{0, (million * 1000000ull + n - 1) / n, 0.f, 0}}, r);
      s.bind();
      if (dadam_accumulate(s.h, s.g.data(), 1, nullptr) != DADAM_OK) { printf("refused\n"); exit(1); }
      if (route == "whole") from = million;
    }
    say(std::to_string(n).c_str(), std::to_string(from));
  }
}

// Large layouts of one long segment, or of segments of `each` elements: which kernel, in which shape and order.
static void large(uint64_t each, uint64_t total) {
  struct { int rows, degree; } cases[] = {{4, 3}, {8, 3}, {16, 3}, {18, 2}, {24, 3}, {32, 2}, {33, 2}, {32, 3}, {32, 6}, {40, 2}, {64, 3}, {96, 2}, {96, 3}, {96, 4}, {96, 5}, {96, 6}, {96, 7}};
  for (uint32_t dtype : {DADAM_F32, DADAM_BF16})
    for (const auto& c : cases) {
      Rows r;
      for (int i = 0; i < c.rows; ++i) {
        std::vector<int32_t> cols;
        for (int k = 0; k < c.degree; ++k) cols.push_back((i + k) % c.rows);
        add_row(r, cols);
      }
      const uint64_t d = total / c.rows;
      std::vector<dadam_tensor_desc> ts;
      for (uint64_t at = 0; at < d; at += each + 8) ts.push_back({at, at + each < d ? each : d - at, 0.f, 0});
      Sim s(c.rows, c.rows, ts, r, dtype);
      s.bind();
      auto told = [&](const std::string& kind) { return (kind.substr(0, 6) == "direct" ? "direct " : kind + " ") + how; };
      const std::string step = told(s.step(DADAM_FUSE_ACCUM)), mix = told(s.mix(0));
      double out = 0.0;
      if (dadam_mix_consensus(s.h, 0, 0, &out, nullptr) != DADAM_OK) { printf("refused\n"); exit(1); }
      const std::string error = how;
      if (dadam_accumulate(s.h, s.g.data(), 1, nullptr) != DADAM_OK) { printf("refused\n"); exit(1); }
      say(((dtype == DADAM_BF16 ? "bf16 " : "f32 ") + std::to_string(c.rows) + " of " + std::to_string(c.degree)).c_str(),
          step + "; mix " + mix + "; error " + error + "; accumulate " + how);
    }
}

int main(int argc, char** argv) {
  const std::string what = argc > 1 ? argv[1] : "";
  if (what == "foreign_in_place") foreign_in_place();
  else if (what == "consensus") consensus();
  else if (what == "loops") loops();
  else if (what == "sparse_loops") sparse_loops();
  else if (what == "few_rows") few_rows();
  else if (what == "loop_shares") loop_shares();
  else if (what == "maps") maps();
  else if (what == "map_of") map_of();
  else if (what == "few") few();
  else if (what == "die_order") die_order();
  else if (what == "accumulation") accumulation();
  else if (what == "long") large(1ull << 40, 120000000);       // streams
  else if (what == "short") large(1100, 120000000);            // streams
  else if (what == "ordinary11") large(1ull << 40, 11000000);  // does not
  else if (what == "ordinary20") large(1ull << 40, 20000000);
  else { printf("unknown question\n"); return 2; }
  return 0;
}
