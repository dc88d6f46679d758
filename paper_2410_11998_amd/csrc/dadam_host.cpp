// Host side of libdadam: the C ABI of include/dadam.h - argument validation, the segment/tile
// planner, neighbour-list slots, per-iteration scalars and launch set-up.  No arithmetic of the
// method happens here except the scalar bias corrections of Algorithm 3 line 8, which are the same
// for every element of an iteration.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <new>
#include <string>
#include <utility>
#include <vector>

#include "dadam_internal.h"

using namespace dadam;

namespace {

thread_local std::string g_init_error;

struct Slot {
  bool set = false;
  std::vector<int32_t> row_ptr, col;
  std::vector<float> w;
  int32_t max_degree = 0;             // longest row
  uint32_t n_read = 0;                // sources that some row lists
  std::vector<int32_t> order;         // rows ordered so that neighbours share sources (empty: nothing is shared)
  bool reuse = false;                 // some source is read by two or more rows
  // Loops: rows that list the same sources with the same weights.  Filled only where the loop kernel may take the
  // slot (see find_loops).
  std::vector<Loop> loops;
  std::vector<int32_t> loop_of_row, loop_of_source;  // the loop a row is in / that reads a source (-1: none)
  std::vector<int32_t> sole_reader;   // per source: the only row reading it, -1 none, -2 several
  // one device allocation holding everything the kernels read (see StepArgs)
  char* d_lists = nullptr;
  const int32_t *d_row_ptr = nullptr, *d_col = nullptr;                                    // tile kernel
  const float* d_w = nullptr;
  const int32_t *d_row_len = nullptr, *d_list_col = nullptr, *d_row_order = nullptr;        // direct kernel
  const float* d_list_w = nullptr;
  const int32_t *d_loop_col = nullptr, *d_loop_rows = nullptr;                              // loop kernel
  const float* d_loop_w = nullptr;
  const Loop* d_loops = nullptr;
};

struct DeviceGuard {
  int prev = -1;
  bool switched = false;
  hipError_t err = hipSuccess;
  explicit DeviceGuard(int dev) {
    err = hipGetDevice(&prev);
    if (err == hipSuccess && prev != dev) {
      err = hipSetDevice(dev);
      switched = (err == hipSuccess);
    }
  }
  ~DeviceGuard() {
    if (switched) (void)hipSetDevice(prev);
  }
};

}  // namespace

struct dadam_handle {
  dadam_config cfg{};
  std::vector<dadam_tensor_desc> tensors;
  std::vector<uint32_t> tensor_seg;  // segment of each non-empty tensor, UINT32_MAX for empty ones
  std::vector<Segment> segs;
  std::vector<uint32_t> seg_work[kNumGrids];  // per Grid: number of work items (tiles; per row in direct mode) in earlier segments
  // Layouts of many short tensors side by side: no search and no tile launched twice, but one dense grid over the whole vector and a byte
  // for every four elements that says which are stored and decay (build_map).
  bool mapped = false;
  float map_decay = 0.f;      // of the tensors that decay
  uint8_t* d_map = nullptr;
  Segment* d_segs = nullptr;     // the segments, and behind them
  uint32_t* d_seg_work = nullptr;  // their first work items, per Grid (what the kernels search)
  double* d_partials = nullptr;  // kConsensusPartials doubles of scratch for the consensus error
  // Cleared when the handle is made and by every pass after use; false after a pass that could not be enqueued whole,
  // and the next one clears them itself.  Passes that are recorded into a graph neither rely on it nor change it.
  bool partials_clear = true;
  // Handles with more than kInlineRows rows or sources: device copies of the bound pointer tables, two per
  // binding (as bound, and with x_src / x_dst exchanged), DADAM_BINDINGS_KEPT bindings in a ring.
  BoundTables* d_tables = nullptr;
  uint32_t binding = 0;  // ring position of the current binding
  bool swapped = false;  // dadam_swap_x flips between the binding's two copies
  double* d_static_partials = nullptr;  // the same in the library's device image (dadam_mix_consensus_static)
  uint32_t static_capacity = 0;         // doubles it holds
  TileShape shape{4, 1, false};
  TileShape mix_shape{4, 1, false};  // shape of the mixing-only launch (more bytes in flight per wavefront)
  uint32_t mix_tile_elems = 0, mix_lds_bytes = 0;
  uint64_t n_work_m = 0;
  bool nontemporal = false;  // every launch streams (steps of few rows may all the same, see few_rows_stream)
  bool decays = false;  // some tensor carries weight decay
  // Segments of fewer than 65536 elements on average: lanes are hardly ever spread and most tiles need their segment searched, so
  // streaming launches keep the shapes and orders of contiguous lanes.  (By the share of elements in whole blocks, which takes a long tensor
  // beside many short ones for long, steps of GPT-2 shapes with decay gain nothing and unfused steps lose up to 7 % at 16 rows.)  Fraction of 8 TB/s, contiguous / spread choices, segments of
  // 1100 elements: exp. graph of 16 0.74 / 0.70, of 64 0.68 / 0.66, pairs of 64 0.53 / 0.51.
  bool short_segments = false;
  int vec = 4;
  uint32_t tile_elems = 0, direct_elems = 0, lds_bytes = 0;
  bool tile_possible = false;
  uint64_t n_elems = 0;  // elements of the tensors
  uint64_t n_work_t = 0, n_work_d = 0, n_work_v = 0;
  Slot slots[DADAM_MAX_SLOTS];
  bool bound = false;
  const void* x_src[kMaxRows] = {};
  void* x_dst[kMaxRows] = {};
  float* m_hat[kMaxRows] = {};
  float* v_hat[kMaxRows] = {};
  float* acc[kMaxRows] = {};
  std::vector<int32_t> inplace_cols[kMaxRows];  // every source buffer that x_dst[i] coincides with
  uint32_t lds_limit = 65536;  // LDS one workgroup may use
  uint32_t n_xcds = 8;         // dies consecutive workgroup ids are dealt over
  // Gradient tables that passed check_grads against the current outputs: a caller that cycles a few
  // gradient sets (or issues a step bucket by bucket) is checked once per set, not once per call.
  struct CheckedGrads { uint64_t gen; std::vector<const void*> ptrs; };
  std::vector<CheckedGrads> checked;
  size_t checked_next = 0;
  // Names the set of output buffers: dadam_bind moves on to the next even number, dadam_swap_x flips
  // the lowest bit (two exchanges give back the same tables).
  uint64_t outputs_gen = 0;
  std::vector<std::pair<uintptr_t, uintptr_t>> outputs_sorted[2];  // [lo, hi) of x_dst, m_hat, v_hat, b, by lo
  uint64_t outputs_sorted_gen[2] = {~0ull, ~0ull};
  float lr = 0.f;
  double betav = 0.0;
  mutable std::string err;
};

namespace {

int fail(const dadam_handle* h, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof(buf), fmt, ap);
  va_end(ap);
  if (h) h->err = buf; else g_init_error = buf;
  return code;
}

size_t dtype_bytes(uint32_t dt) { return dt == DADAM_BF16 ? 2 : 4; }

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

struct Interval {
  uintptr_t lo, hi;
  int kind;  // 0 x_src, 1 x_dst, 2 state
  int index;
};

bool overlaps(const Interval& a, const Interval& b) { return a.lo < b.hi && b.lo < a.hi; }

// Measurement builds (-DDADAM_TUNING, never what build() makes) let the environment override kernel
// shapes when a handle is created; the shipped library has no such switches.
#ifdef DADAM_TUNING
int env_int(const char* name, int fallback) {
  const char* v = getenv(name);
  if (!v || !*v) return fallback;
  return atoi(v);
}
#else
constexpr int env_int(const char*, int fallback) { return fallback; }
#endif

// Elements of a tile of one vector a lane: what the loop kernel walks, and what the rules below count launches in.
uint32_t vector_elems(const dadam_handle* h) { return (uint32_t)(kWave * h->vec); }

// Build maximal runs of contiguous tensors.
void find_segments(dadam_handle* h) {
  h->segs.clear();
  h->tensor_seg.assign(h->tensors.size(), UINT32_MAX);
  for (size_t k = 0; k < h->tensors.size(); ++k) {
    const dadam_tensor_desc& t = h->tensors[k];
    if (t.numel == 0) continue;
    if (!h->segs.empty() && h->segs.back().hi == t.offset_elems && h->segs.back().weight_decay == t.weight_decay) {
      h->segs.back().hi = t.offset_elems + t.numel;
    } else {
      Segment s{};
      s.lo = t.offset_elems;
      s.hi = t.offset_elems + t.numel;
      s.weight_decay = t.weight_decay;
      h->segs.push_back(s);
    }
    h->tensor_seg[k] = (uint32_t)(h->segs.size() - 1);
  }
  for (const Segment& s : h->segs) h->n_elems += s.hi - s.lo;
  h->short_segments = h->segs.size() * (uint64_t)kLongSegment > h->cfg.d;
}

// Does the layout get a map?  Segments of 65536 elements on average or fewer, a gap of at most 7 elements between two (what packing to
// multiples of 8 leaves; wider gaps, whose padding a dense grid loads too, were not measured and keep the walk by segments), one value of decay beside 0,
// four elements never with and without it, d a multiple of 4 (the last group of a buffer is whole), and at most 2^28 elements (64 MB of map).  Such layouts
// then count as one segment, but in launches that are faster by segments (segments_are_faster).  What a map gives stands at MapTile.
bool can_map(const dadam_handle* h, float* decay) {
  if (!h->short_segments || h->segs.size() < 2 || h->cfg.d % 4 != 0 || h->cfg.d > kMostMapped) return false;
  *decay = 0.f;
  for (size_t k = 0; k < h->segs.size(); ++k) {
    const Segment& s = h->segs[k];
    if (s.weight_decay != 0.f && *decay != 0.f && s.weight_decay != *decay) return false;
    if (s.weight_decay != 0.f) *decay = s.weight_decay;
    if (k == 0) continue;
    const Segment& before = h->segs[k - 1];
    if (s.lo - before.hi > kWidestGap) return false;
    if (s.lo / 4 == (before.hi - 1) / 4 && (s.weight_decay != 0.f) != (before.weight_decay != 0.f)) return false;
  }
  return true;
}

// The map (see StepArgs::map), zero behind the layout up to the end of the last tile of any grid.
std::vector<uint8_t> build_map(const dadam_handle* h) {
  std::vector<uint8_t> map((h->cfg.d + kLongSegment) / 4, 0);
  for (const Segment& s : h->segs) {
    const uint8_t decays = s.weight_decay != 0.f ? 0x10 : 0;
    const uint64_t first = (s.lo + 3) / 4, last = s.hi / 4;  // whole groups [first, last)
    if (first < last) memset(map.data() + first, 0x0F | decays, last - first);
    for (uint64_t e = s.lo; e < std::min(s.hi, 4 * first); ++e) map[e / 4] |= (uint8_t)(1u << e % 4) | decays;
    for (uint64_t e = std::max(s.lo, 4 * std::max(first, last)); e < s.hi; ++e) map[e / 4] |= (uint8_t)(1u << e % 4) | decays;
  }
  return map;
}

// Number the tiles of every tile grid.
int plan(dadam_handle* h) {
  uint64_t wt = 0, wd = 0, wm = 0, wv = 0;
  for (Segment& s : h->segs) {
    if (s.weight_decay != 0.f) h->decays = true;
    s.first_tile[kGridTile] = s.lo / h->tile_elems;
    s.first_tile[kGridDirect] = s.lo / h->direct_elems;
    s.first_tile[kGridMix] = s.lo / h->mix_tile_elems;
    s.first_tile[kGridVector] = s.lo / vector_elems(h);
    if (wv > 0x7fffffffull || wd > 0x7fffffffull) break;
    h->seg_work[kGridTile].push_back((uint32_t)wt);
    h->seg_work[kGridDirect].push_back((uint32_t)wd);
    h->seg_work[kGridMix].push_back((uint32_t)wm);
    h->seg_work[kGridVector].push_back((uint32_t)wv);
    wt += (s.hi - 1) / h->tile_elems - s.first_tile[kGridTile] + 1;
    wd += (s.hi - 1) / h->direct_elems - s.first_tile[kGridDirect] + 1;
    wv += (s.hi - 1) / vector_elems(h) - s.first_tile[kGridVector] + 1;
    wm += (s.hi - 1) / h->mix_tile_elems - s.first_tile[kGridMix] + 1;
  }
  h->n_work_t = wt;
  h->n_work_d = wd;
  h->n_work_m = wm;
  h->n_work_v = wv;
  if (wv > 0x7fffffffull || wd * (h->cfg.n_rows + h->n_xcds) > 0x7fffffffull)  // direct mode pads rows up to the dies
    return fail(nullptr, DADAM_EINVAL, "layout too large: more than 2^31-1 work items");
  return DADAM_OK;
}

// Work-item range [w0, w1) of the tiles that intersect elements [lo, hi), which start in segment
// s0 and end in segment s1.
// by_map: over the dense grid of a layout with a map.
void work_range(const dadam_handle* h, bool by_map, Grid grid, uint32_t s0, uint32_t s1, uint64_t lo,
                uint64_t hi, uint32_t* w0, uint32_t* w1) {
  const uint64_t T = grid == kGridTile ? h->tile_elems : grid == kGridDirect ? h->direct_elems : grid == kGridMix ? h->mix_tile_elems : vector_elems(h);
  if (by_map) {
    *w0 = (uint32_t)(lo / T);
    *w1 = (uint32_t)((hi - 1) / T) + 1;
    return;
  }
  const Segment& a = h->segs[s0];
  const Segment& b = h->segs[s1];
  *w0 = h->seg_work[grid][s0] + (uint32_t)(lo / T - a.first_tile[grid]);
  *w1 = h->seg_work[grid][s1] + (uint32_t)((hi - 1) / T - b.first_tile[grid]) + 1;
}

int check_bound(const dadam_handle* h) {
  if (!h->bound) return fail(h, DADAM_ESTATE, "no buffers bound: call dadam_bind first");
  return DADAM_OK;
}

// The last check before a launch, after every argument has been validated (so that a host-only
// handle reports what is wrong with a call exactly as a device handle would).
int check_device(const dadam_handle* h) {
  if (h->cfg.device == DADAM_DEVICE_NONE)
    return fail(h, DADAM_ESTATE, "host-only handle (device = DADAM_DEVICE_NONE) cannot launch");
  return DADAM_OK;
}

// Gradients are read-only; what they must not overlap is anything the call writes.  The outputs are
// pairwise disjoint (dadam_bind checked that), so they are kept sorted and each gradient is located
// with a binary search; a table that passed is remembered until the outputs change.
int check_grads(dadam_handle* h, const void* const* grads) {
  if (!grads) return fail(h, DADAM_EINVAL, "grads is null");
  const uint32_t R = h->cfg.n_rows;
  for (const auto& ok : h->checked)
    if (ok.gen == h->outputs_gen && std::equal(ok.ptrs.begin(), ok.ptrs.end(), grads)) return DADAM_OK;
  const size_t gb = h->cfg.d * dtype_bytes(h->cfg.grad_dtype);
  const size_t xb = h->cfg.d * dtype_bytes(h->cfg.param_dtype);
  const size_t sb = h->cfg.d * 4;
  const int par = (int)(h->outputs_gen & 1u);
  auto& o = h->outputs_sorted[par];
  if (h->outputs_sorted_gen[par] != h->outputs_gen) {
    o.clear();
    for (uint32_t j = 0; j < R; ++j) {
      o.push_back({(uintptr_t)h->x_dst[j], (uintptr_t)h->x_dst[j] + xb});
      o.push_back({(uintptr_t)h->m_hat[j], (uintptr_t)h->m_hat[j] + sb});
      o.push_back({(uintptr_t)h->v_hat[j], (uintptr_t)h->v_hat[j] + sb});
      if (h->acc[j]) o.push_back({(uintptr_t)h->acc[j], (uintptr_t)h->acc[j] + sb});
    }
    std::sort(o.begin(), o.end());
    h->outputs_sorted_gen[par] = h->outputs_gen;
  }
  for (uint32_t i = 0; i < R; ++i) {
    if (!grads[i]) return fail(h, DADAM_EINVAL, "grads[%u] is null", i);
    if (!aligned16(grads[i])) return fail(h, DADAM_EALIGN, "grads[%u] is not 16-byte aligned", i);
    const uintptr_t lo = (uintptr_t)grads[i], hi = lo + gb;
    // first output that ends beyond lo; it overlaps iff it starts below hi
    auto it = std::upper_bound(o.begin(), o.end(), lo,
                               [](uintptr_t v, const std::pair<uintptr_t, uintptr_t>& iv) { return v < iv.second; });
    if (it != o.end() && it->first < hi)
      return fail(h, DADAM_EALIAS, "grads[%u] overlaps an output buffer (x_dst, m_hat, v_hat or acc)", i);
  }
  dadam_handle::CheckedGrads ok{h->outputs_gen, std::vector<const void*>(grads, grads + R)};
  if (h->checked.size() < 8) h->checked.push_back(std::move(ok));
  else { h->checked[h->checked_next] = std::move(ok); h->checked_next = (h->checked_next + 1) % 8; }
  return DADAM_OK;
}

void fill_args(const dadam_handle* h, bool by_map, const void* const* grads, StepArgs* a) {
  memset(a, 0, sizeof(*a));
  const uint32_t R = h->cfg.n_rows, C = h->cfg.n_cols;
  if (h->d_tables) {
    a->ext = h->d_tables + 2 * h->binding + (h->swapped ? 1 : 0);
  } else if (R <= (uint32_t)kInlineRows && C <= (uint32_t)kInlineRows) {
    for (uint32_t c = 0; c < C; ++c) a->x_src[c] = h->x_src[c];
    for (uint32_t i = 0; i < R; ++i) {
      a->x_dst[i] = h->x_dst[i];
      a->m_hat[i] = h->m_hat[i];
      a->v_hat[i] = h->v_hat[i];
      a->acc[i] = h->acc[i];
    }
  }
  for (uint32_t i = 0; i < R; ++i) a->grad[i] = grads ? grads[i] : nullptr;
  a->seg = h->d_segs;
  a->seg_work = h->d_seg_work;
  a->map = by_map ? h->d_map : nullptr;
  a->n_seg = by_map ? 1u : (uint32_t)h->segs.size();
  a->n_rows = R;
  a->n_cols = C;
  a->n_xcd = h->n_xcds;
  a->d = h->cfg.d;
  a->die_run = 1;
  a->xcd_block = (uint32_t)env_int("DADAM_XCD_BLOCK", (int)kDieBlockTiles);
}

// Scalars of iteration t (Algorithm 3 lines 4 and 8), computed in double and rounded once.
void fill_scalars(const dadam_handle* h, uint64_t t, Scalars* s) {
  const double b1 = (double)h->cfg.beta1, b2 = (double)h->cfg.beta2, bv = h->betav;
  const uint64_t S = h->cfg.accum_s;
  const double th = (double)((t + S - 1) / S);  // t_hat = ceil(t / s)
  s->beta1 = (float)b1;
  s->omb1 = (float)(1.0 - b1);
  s->beta2 = (float)b2;
  s->omb2 = (float)(1.0 - b2);
  s->betav = (float)bv;
  s->ombv = (float)(1.0 - bv);
  s->inv_c1 = (float)(1.0 / (1.0 - std::pow(b1, th)));
  s->inv_c2 = (float)(1.0 / (1.0 - std::pow(b2, th)));
  s->eps = h->cfg.eps;
  s->lr = h->lr;
  s->inv_s = (float)(1.0 / (double)S);
}

Phase fused_phase(const dadam_handle* h, uint64_t t) {
  const uint64_t S = h->cfg.accum_s;
  if (S == 1) return kAlg1;
  if (t % S == 0) return kFold;
  if ((t - 1) % S == 0) return kLoopStart;
  return kPlain;
}

// A row updated in place overwrites every source buffer that shares its memory (two source
// entries may name one buffer); the direct kernel may do that only if nobody but the row itself
// reads any of them: neither from a list nor, where the launch decays, as the row whose own parameters they are.
bool direct_is_legal(const dadam_handle* h, const Slot& slot, bool decays) {
  for (uint32_t i = 0; i < h->cfg.n_rows; ++i)
    for (int32_t c : h->inplace_cols[i]) {
      const int32_t sr = slot.sole_reader[c];
      if (!(sr == -1 || sr == (int32_t)i)) return false;
      if (decays && (uint32_t)c < h->cfg.n_rows && c != (int32_t)i) return false;
    }
  return true;
}

// Does a step over tensors [tb, te) of the layout (whole: all of them) apply weight decay?
bool range_decays(const dadam_handle* h, bool whole, uint32_t tb, uint32_t te) {
  if (whole || !h->decays) return h->decays;
  for (size_t k = tb; k < te && k < h->tensors.size(); ++k)
    if (h->tensors[k].numel && h->tensors[k].weight_decay != 0.f) return true;
  return false;
}

// Streaming float32 steps over short segments: cut tiles load element by element where that is faster.  (Where every row's loads are
// few lines, groups that lie outside a segment cost more than waiting does.)  us, elements / groups, 2e8 elements in segments of 1100, by the tile
// kernel: 4 rows 1876 / 1926, 6 rows 1905 / 1962, 8 rows 2013 / 1982, 12 rows 1942 / 1943, 16 rows 1969 / 2000, 24 rows 1957 / 2010, 32 rows 1992 / 2031,
// 48 rows 2069 / 2092, 64 rows 2102 / 2091; 1.5e8 elements in segments of 1000: 50 rows 3937 / 3974, 56 rows 4415 / 4372, 60 rows 4780 / 4746;
// by the loop kernel: 16 rows 3877 / 3780, 24 rows 3795 / 3845, 32 rows 3802 / 3882, 48 rows 3997 / 4044.  In
// bfloat16, mixing and by the direct kernel groups are ahead, by 1 to 20 %.
bool cut_by_elements(const dadam_handle* h, bool mix_only, bool by_loops) {
  const uint32_t R = h->cfg.n_rows;
  return h->nontemporal && h->short_segments && h->vec == 4 && !mix_only && (by_loops ? R >= 24 && R < 64 : R < 8 || (R >= 16 && R < 56));
}

// Large launches in die blocks: a die takes runs of `run` pieces (or items), row after row (see rows_stay_on_one_die).
void set_die_run(uint32_t run, StepArgs* a) { a->die_run = a->xcd_block = run; }

// Do direct launches of this slot walk its rows in the sharing order?
bool ordered_rows(const dadam_handle* h, const Slot& slot) { return !slot.order.empty() && h->n_xcds > 1; }

// decays: the launch applies weight decay.
void set_range(const dadam_handle* h, bool by_map, bool decays, Grid grid, uint32_t work_begin, uint64_t lo, uint64_t hi, StepArgs* a) {
  a->grid = grid;
  a->work_begin = work_begin;
  a->clip_lo = lo;
  a->clip_hi = hi;
  a->first_tile = by_map ? 0 : h->segs.front().first_tile[grid];
  a->weight_decay = !by_map ? h->segs.front().weight_decay : decays ? h->map_decay : 0.f;
}

// Does a compute unit hold one workgroup of the tile, even with one vector a lane?
bool lone_tile(const dadam_handle* h) { return 2 * (uint64_t)h->cfg.n_cols * kWave * 16u > h->lds_limit; }

// Decide tile or direct mode for this slot and these flags; checks in-place legality.  decays: the launch applies
// weight decay.
int choose_mode(const dadam_handle* h, const Slot& slot, uint32_t flags, bool decays, bool* tile_mode) {
  if ((flags & DADAM_FORCE_DIRECT) && (flags & DADAM_FORCE_TILE))
    return fail(h, DADAM_EINVAL, "DADAM_FORCE_DIRECT and DADAM_FORCE_TILE are exclusive");
  const bool direct_legal = direct_is_legal(h, slot, decays);
  if (flags & DADAM_FORCE_TILE) {
    if (!h->tile_possible) return fail(h, DADAM_EINVAL, "tile mode needs the source tile to fit in LDS");
    *tile_mode = true;
  } else if (flags & DADAM_FORCE_DIRECT) {
    if (!direct_legal)
      return fail(h, DADAM_EALIAS, "in-place update of a source that another row reads needs tile mode");
    *tile_mode = false;
  } else {
    // Shared sources normally mean tile mode.  Two exceptions, where the rows stream directly and the dies
    // take them in the sharing order, so that the second reader of a source finds it in its die's L2:
    // (1) rows of at most two sources over more sources than the two-vector tile holds (64 replicas of a
    // one-peer graph: mixing 0.77 against 0.75 of peak, the whole step 0.792 against 0.788; with three
    // sources a row, a ring, the tile is as fast or faster);
    // (2) a tile so large that a CU holds one workgroup of it (more than 80 sources on 160 KB), with rows of
    // at most eight sources (128 replicas, launches that do not stream: the step of seven sources 0.60 against 0.48; launches that stream
    // are decided in staging_is_faster).
    const bool ordered = slot.reuse && direct_legal && h->n_xcds > 1;
    const bool pairs_stream = ordered && slot.max_degree <= 2 && h->cfg.n_cols > 16;
    const bool alone_streams = ordered && slot.max_degree <= 8 && lone_tile(h);
    *tile_mode = h->tile_possible && ((slot.reuse && !pairs_stream && !alone_streams) || !direct_legal);
    if (!*tile_mode && !direct_legal)
      return fail(h, DADAM_EALIAS, "in-place update of a shared source is impossible: tile does not fit in LDS");
  }
  return DADAM_OK;
}

// Do steps of up to three rows stream in a handle whose other launches do not (see dadam_init)?  From 344 MB (2^20) of buffers that an
// iteration touches: the sources that rows list, outputs that are not updated in place, gradients and state.  One row with two receive
// buffers, updated in place, has 28 bytes an element in float32 and is past the last-level cache (256 MB) from 1.29e7 elements on, where
// ordinary accesses with lanes side by side lose.  Four steps, time of streaming accesses over ordinary ones, by MB:
//   one row of 2 sources 320 1.03, 332 0.98, 343 0.95, 366 0.90; of 3 320 1.04, 334 1.01, 344 0.97, 360 0.94, 401 0.87 (bfloat16 324 1.00, 334 0.97, 343
//   0.96, 362 0.90; s = 1 320 1.02, 343 0.97, 366 0.91); of 5 326 1.05, 343 1.00, 360 0.93, 412 0.87; of 3 in 64 buffers 133 1.03, 339 0.88
//   two rows 320 1.00, 343 0.97, 366 0.93, 412 0.86 (bfloat16 326 0.97, 343 0.92, 378 0.88); three 326 0.97, 343 0.94, 412 0.84 (335 0.94, 360 0.90)
// With an accumulation behind every step, at 343 MB, steps alone / both streaming: 0.96 / 1.00, two rows 0.97 / 1.00, three 0.94 / 0.99, and so up to the
// handle's line, so accumulation keeps to that; mixing was not measured and does too.  (Steps of more rows would gain between 15 and 22 million elements
// as well, but pairs in bfloat16 and loops lose there; they were not measured by bytes, nor were short segments without a map.)
bool few_rows_stream(const dadam_handle* h, uint32_t sources) {
  const uint32_t R = h->cfg.n_rows;
  if (R > 3 || h->short_segments) return false;
  uint32_t outputs = 0;
  for (uint32_t i = 0; i < R; ++i) outputs += h->inplace_cols[i].empty() ? 1 : 0;
  const uint64_t row = dtype_bytes(h->cfg.grad_dtype) + (h->cfg.accum_s > 1 ? 12u : 8u);
  return h->n_elems * ((sources + outputs) * dtype_bytes(h->cfg.param_dtype) + R * row) > kStreamedBytes;
}

uint32_t loop_lds_bytes(const dadam_handle* h, int waves) { return (uint32_t)(waves * kWave * h->vec * 4); }

// Tiles of one vector a lane of a launch over the whole layout.
uint64_t vector_tiles(const dadam_handle* h) {
  if (!h->mapped) return h->n_work_v;
  const uint64_t T = vector_elems(h);
  return (h->segs.back().hi - 1) / T - h->segs.front().lo / T + 1;
}

// Wavefronts of a loop kernel's workgroup, 0: another kernel takes the launch.  Depends on the slot and on the whole
// layout, never on the range of a launch: the order in which a loop is summed follows from it, and a step issued
// range by range has the bits of the whole one.
// Legal: a row updated in place overwrites sources that only its own loop may read (the loop reads them all before
// it writes), and with weight decay a row reads its own parameters again after that; the partial sums fit the LDS the
// configuration grants.
// Faster: with 16 rows to a loop on average.  us, other kernels / 4 / 8 / 16 wavefronts, 3e8 elements, mixing:
// 32 rows in one loop 1349 / 862 / 837 / 900, 64 rows 3163 / 881 / 871 / 865, 96 rows in loops of 48, 24, 24 8486 /
// 1764 / 1737 / 2091, but 32 rows in loops of 16, 8, 8 1756 / 1667 / 1933 / 3531 and 16 rows in loops of 8, 4, 4
// 1709 / 1850 / 3098.  Steps, tile / this, four of 3e8 elements, one loop of 16, 32, 48, 64 rows: 6288 / 6167, 6512 / 6419,
// 6749 / 6654, 7978 / 6561 (bfloat16 5069 / 4905, 5256 / 5095, 5650 / 5241, 6710 / 5201), 64 rows in loops of 32, 16, 16 6428 /
// 6541 (5257 / 5175), 96 in loops of 48, 24, 24 13221 / 6635.  In small launches each wavefront walks its rows in turn, so
// more of them, from 8 rows a loop on: 64 rows 4e5 elements 85 / 121 / 75 / 52, 4e6 225 / 176 / 118 / 84; 32 rows in
// loops of 16, 8, 8 4e5 36 / 44 / 32 / 27.  One loop of fewer than 28 rows leaves 16 of them little to do beyond one tile
// per compute unit: tile time over 8 / 16, 16 rows of 366, 488 tiles 1.00 / 0.88, 0.98 / 0.88 (bfloat16 1.08 / 0.96, 1.02 /
// 0.88), 24 rows of 488 1.22 / 1.11, 28 rows 1.20 / 1.26, 64 rows in three loops of 275 1.98 / 2.29.
// A step with decay reads each row's own parameters again, from memory: 12 % of it.  In large layouts that is more than the
// shared sum saves, until the tile kernel's own sums get long or few workgroups of its tile share a compute unit: tile /
// this, 3e8 elements, one loop of 32, 48, 52, 56, 64 rows 6489 / 7311, 0.91, 0.92, 1.01, 8000 / 7442; 64 rows in loops of
// 32, 16, 16 6433 / 7332, but 72, 80, 96 rows of such loops 1.01, 1.05, 13239 / 7536 (bfloat16 0.95 / 1.03 / 1.06 / 1.14 /
// 1.18 and 0.93, 0.94, 0.98, 1.47).  In small ones the tile kernel has other troubles; they are even at about 32 tiles for
// every row of a loop: 24 rows 1.21, 1.07, 1.04, 1.00, 0.97 at 400, 500, 700, 1000, 1500 tiles, 48 rows 1.62, 1.37, 1.33,
// 1.21, 1.13, 64 in loops of 32, 16, 16 1.14, 1.02, 1.08, 0.92, 0.83.
int loop_kernel_waves(const dadam_handle* h, const Slot& slot, bool mix_only) {
  const uint64_t R = h->cfg.n_rows, G = slot.loops.size();
  if (G == 0 || (R < 16 * G && (R < 8 * G || vector_tiles(h) > kFewTiles))) return 0;
  if (!mix_only && h->decays && vector_tiles(h) * G > 32 * R && R < 56 * G && h->cfg.n_cols <= (uint32_t)kInlineRows) return 0;
  for (uint32_t i = 0; i < R; ++i)
    for (int32_t c : h->inplace_cols[i])
      if ((slot.loop_of_source[c] != -1 && slot.loop_of_source[c] != slot.loop_of_row[i]) || h->decays) return 0;
  const int waves = vector_tiles(h) * G <= (G == 1 && R < 28 ? 1 : 2) * kFewTiles ? 16 : 8;
  return loop_lds_bytes(h, waves) <= h->lds_limit ? waves : 0;
}

// How many workgroups share the rows of one tile of a loop.  The order of the sums does not depend on it.  A row updated in place
// overwrites a source that the other workgroups may still read, so there it is one; and one in streaming mixing, which has no kernel of
// shares (whether a handle streams follows from d, its tiles from what the tensors cover of it, so a streaming launch may well be small).
// Launches that leave compute units idle: as many as keep it at one workgroup a unit (sixteen wavefronts then walk 6 rows of 96 in turn
// otherwise).  us of two steps from a graph, one / two / four / as many as this gives, 16 tiles: 32 rows 16.4 / 13.0 / 13.1 / 13.0, 64 rows 25.4 / 19.0 / 15.5 /
// 15.4, 96 rows 39.3 / 27.5 / 22.3 / 18.6 (bfloat16 58.8 / 38.0 / 31.2 / 25.0), in loops of 48, 24, 24 24.1 / 19.8 / 16.1 / 16.0; 128 tiles, two or none fit: 32 rows
// 18.3 / 15.4, 96 rows 60 / 45 (82 / 62), loops 49.2 / 54.6.  17 rows, one of them in the second workgroup, 0.86 to 0.95 of the time of one.  Of unequal loops
// the longest decides, and the others have workgroups that sum and own no row: of 48, 24, 24 by three 16.0, by the two that the shorter ones fill 19.8.
// Mixing, half of whose bytes are sources, gains from 32 rows on, and only where the tiles divide among the dies: then the workgroups of a tile run on one
// and find the sources in its L2.  Time of two over that of one, 32 / 64 / 96 rows: 24 tiles 0.96 / 0.95 / 0.89, 64 tiles 0.98 / 0.97 (56 rows), but 4 tiles 1.16 / 1.17 (56
// rows), 31 tiles 1.07 / 1.10 / 1.15, 42 tiles 1.10 / 1.10 / 1.19, 85 tiles 1.11 / 1.13 / 1.19; 17 to 20 rows of 24 to 128 tiles 0.98 to 1.02.
// Streaming steps of one loop of 96 rows and more, whose workgroups are few and long (12 rows to a wavefront): two where the last round of workgroups
// would be short of them, at most a quarter of one (three to a compute unit in float32, two in bfloat16, by registers).  In the first two rounds a tile
// that the layout's end cuts, which takes longer than others, counts too (see begin_with_last): there up to half a round.  Time of two over that of one, whole tiles /
// one cut, 96 to 160 rows: float32 769 to 960 tiles 0.92 to 1.00 / 0.85 to 0.93, 1024 to 1100 1.00 / 0.92 to 0.95, 1200 to 1536 0.99 to 1.07 / 1.00 to 1.04, 1540 to 1728 0.96 to
// 1.00 / 0.97 to 1.01, 1900 1.00 / 0.98, 2048 and more 0.99 to 1.10 / 0.99 to 1.03; bfloat16 513 to 640 0.92 to 0.95 / 0.76 to 0.83, 700 to 768 1.01 to 1.07 / 0.85 to 0.95, 800 to 1000
// 1.03 to 1.07 / 0.96 to 1.04, 1025 to 1152 0.94 to 0.99 / 0.94 to 0.99, 1200 to 1400 1.00 to 1.04 / 0.98 to 1.04, 1537 to 1664 0.97 to 1.01 / 0.97 to 1.01, 1700 and more 0.98 to 1.05.
// s = 1, decay, accumulation apart and mixed types the same or more (0.86 to 0.98 at 560, 860, 1100 tiles).  Fewer rows gain nothing sure (float32 32 rows
// 0.93 to 1.06, 64 rows 0.93 to 1.05, bfloat16 70 rows 0.91 to 1.12); loops of 48, 24, 24 lose, and so does most of what does not stream.
// With a map 96 and 128 rows of float32 by two over one 0.88 to 0.97 at 800 to 1100 tiles, 0.96 at 1300, as where a tile is cut, bfloat16 0.88 to 0.94 at 560, 0.96 to 1.02 at 640
// to 768, 0.94 to 0.97 at 1100, as where none is.  cut: some tile of the launch is not whole, or it has a map in float32.
uint32_t loop_shares(const dadam_handle* h, const Slot& slot, int waves, uint32_t n_tiles, bool cut, bool mix_only) {
  if (mix_only && h->nontemporal) return 1;
  for (uint32_t i = 0; i < h->cfg.n_rows; ++i)
    if (!h->inplace_cols[i].empty()) return 1;
  uint32_t rows = 0;
  for (const Loop& l : slot.loops) rows = std::max(rows, (uint32_t)l.n_rows);
  const uint32_t most = (rows + (uint32_t)waves - 1) / (uint32_t)waves;
  const uint32_t units = n_tiles * (uint32_t)slot.loops.size();
  if (2 * units <= kFewTiles) return mix_only && (rows < 32 || n_tiles % h->n_xcds != 0) ? 1 : std::min(most, kFewTiles / units);
  if (!h->nontemporal || slot.loops.size() > 1 || rows < 96 || n_tiles >= kLongLaunch) return 1;
  const uint32_t round = kFewTiles * (h->vec == 4 ? 3u : 2u), last = n_tiles % round;
  return n_tiles > round && last > 0 && last <= (cut && n_tiles < 2 * round ? round / 2 : round / 4) ? 2 : 1;
}

// A launch of few tiles leaves compute units idle, and each workgroup walks its rows in turn: up to this many tiles and with
// more rows than a workgroup has wavefronts, the direct kernel's one wavefront per row takes the launch from the tile
// kernel, with the same sums in the same order.  A loop of four steps, us, tile / direct, by tiles: 16 rows of 5 sources 98:
// 27 / 24, 488: 48 / 48; 32 rows of 6 sources 49: 45 / 24, 244: 65 / 48, 977: 158 / 165; 64 rows of 7 sources 24: 82 / 27,
// 122: 108 / 48, 488: 173 / 171; 8 rows the same up to 195 tiles.  Every row reads its sources through the caches, so long
// rows and the wider vectors of bfloat16 end this sooner; direct time over tile time at 128, 192, 256 tiles: float32 rows
// of 12 at most 0.76, 0.85, 1.00, 24 of 128 rows 0.59, 0.80, 1.01, 64 of 128 0.67, 0.94, 1.22, 128 of 128 0.69, 1.00, 1.32;
// bfloat16 rows of 6 at most 0.77, 0.96, 1.02, 24 of 128 0.63, 0.87, 1.21, 64 of 128 0.74, 1.06, 1.43.
uint32_t few_tiles_limit(const dadam_handle* h, const Slot& slot) {
  return slot.max_degree > 24 ? kFewTiles / 2 : slot.max_degree > 12 || h->vec == 8 ? kFewTiles * 3 / 4 : kFewTiles;
}

// From how many tiles on a launch is large for the rules below.  Launches that stream have that few tiles only with many rows (or by ranges), and one wavefront to
// a piece and row in no order, as small launches go, serves spread lanes badly.  Time by the rules for large launches over that by those for small
// ones, 640 to 1000 tiles of 44 to 160 rows: mixing in pairs and of three sources 0.59 to 0.88, of seven 0.45 to 0.72 (81 to 128 rows), steps of two 0.78 to 0.99, of three
// 0.74 to 0.98, of seven 0.62 to 0.89, the others the same kernel; 560 tiles 0.68 to 1.02.  With a map, which has fewer tiles than its segments have, the
// same: 128 rows of seven sources, tensors of 2000 elements, 1000 tiles, two steps 624 / 412 us (by segments 529), mixing 149 / 69 (88).
// Without a map segments of 1100 elements 0.52 to 0.94, but steps of seven float32 sources 1.02, which keep to the old line (see staging_is_faster).
bool many_tiles(const dadam_handle* h, uint32_t n_tiles) { return n_tiles >= (h->nontemporal ? kManyStreamed : kManyTiles); }

// Direct launches of rows that share sources: does every row of a piece run on one die (die blocks), or does each die have a
// group of the rows (die groups)?  Small launches, us, groups / blocks: 64 rows of two sources 244 tiles 87 / 83; 96 rows
// of 7 sources 81 tiles 74 / 53, 325 tiles 215 / 186.  Large ones: mixing is far slower in blocks (0.75 to 0.9 of the rate).
// Steps of 64 rows and more, groups' time over blocks' on the same buffers by elements of all rows together, rows of two:
//   float32    5e7   1.5e8  6e8   1.8e9        bfloat16   5e7   1.5e8  6e8   1.8e9
//   64 rows    0.98  1.10   1.03               64 rows    0.94  1.05   0.99
//   65 rows    1.00  1.16   1.11  1.10         65 rows    0.98  1.14   1.06  1.08     (9 rows on one die, 8 on the others)
//   72 rows    0.97  0.95   0.98  1.01         72 rows    0.96  0.95   0.98  0.99
//   80 rows    0.95  0.96   1.07  1.02         80 rows    0.94  0.93   1.05  1.03
//   96 rows    0.95  1.04   1.03  1.01         96 rows    0.97  1.00   1.06  1.02     (3e8: 1.07)
//   112 rows   0.90  1.05   0.99  0.99         112 rows   0.94  1.02   1.00  0.99
//   128 rows   1.00  1.03   0.98  0.98         128 rows   0.95  1.04   1.02  1.01     (3e8: 1.08)
//   160 rows   0.98  0.99   1.04  0.99         160 rows   0.88  0.99   0.98  0.98
// That was with all rows of a piece one after the other.  Since large launches walk runs of 256 pieces a die row after row,
// blocks are ahead of groups in every streaming launch of at least 1024 tiles (640, see many_tiles): a die has the arrays of few rows in use at a time
// instead of those of all, and rows that do not divide among the dies leave none waiting.  Fraction of 8 TB/s, groups / piece by piece / runs of 64 / 256 / 512, two rows to a source: 64 rows of 26 million elements
// 0.83 / 0.78 / 0.83 / 0.84 / 0.84, 18 rows 0.67 / - / 0.81 / 0.80 / 0.81, 32 rows 0.82 / 0.82 / 0.83 / 0.83 / 0.84, 40 rows 0.79 / - / 0.79 / 0.82 /
// 0.82, bfloat16 18 rows 0.67 / - / 0.78 / 0.80 / 0.80; rings of 48 in bfloat16 0.79 / - / 0.80 / 0.80 / 0.80, of 64 0.80 / 0.72 / 0.80 /
// 0.80 / 0.80, of 128 0.80 / 0.76 / 0.79 / 0.78 / 0.79 (bfloat16 0.76 / 0.78 / 0.79 / 0.79 / 0.79).  Launches that do not stream, groups' time
// over that of runs of 256: 18 rows 1.24, 26 rows (bfloat16) 1.04, 64 rows 1.03-1.07, ring of 100 1.03-1.07, 20 rows of 250 thousand
// elements 1.02, 32 rows 1.03 and 0.96.
// Pairs of 32 to 63 rows and the larger numbers of rows below the sizes of the table have stayed with groups.  us of a loop of two,
// groups / runs, float32 of 4e7, 1.2e8, 4e8 elements of all rows: 32 rows 372 / 366, 1104 / 1081, 3620 / 3586, 33 rows 415 / 370, 1240 / 1086, 4111 / 3583,
// 36 rows 390 / 371, 1152 / 1084, 3849 / 3597, 48 rows 380 / 371, 1101 / 1082, 3642 / 3606, 63 rows 375 / 370, 1114 / 1078, 3666 / 3577, 72 rows 385 / 372,
// 1115 / 1086, 3773 / 3605, 80 rows 381 / 371, 1103 / 1085, 3693 / 3596 (bfloat16 33 rows 341 / 305, 1004 / 884, 3336 / 2911, 48 rows 308 / 303, 912 / 881, 2978 /
// 2947, 160 rows of 1.2e8, 4e8 931 / 882, 3043 / 2918).  Launches of fewer tiles go piece by piece.
// Launches that do not stream, us, groups / runs, 1.1e7 and 1.6e7 elements: float32 32 rows 106 / 112, 170 / 163, 33 rows 120 / 107, 182 / 159, 40 rows 107 /
// 107, 171 / 164, 48 rows 108 / 109, 168 / 155; bfloat16 of 1.6e7 32 rows 121 / 125, 40 rows 132 / 141, 48 rows 124 / 132, 56 rows 124 / 129, 33 rows 140 / 126.
bool rows_stay_on_one_die(const dadam_handle* h, const Slot& slot, bool mix_only, uint32_t n_tiles) {
  if (!many_tiles(h, n_tiles)) return true;
  const uint32_t R = h->cfg.n_rows;
  if (mix_only) return false;
  if (!h->nontemporal) {
    const bool even = R >= 32 && R < 64 && R % h->n_xcds == 0 && slot.max_degree <= 2;
    return !(even && (h->vec == 8 || (uint64_t)n_tiles * vector_elems(h) * R < kPairElems));
  }
  if (R < 64) return !h->short_segments && (R < 32 || slot.max_degree > 2);
  const bool wide = h->vec == 8;
  if (wide && R >= 72 && (R < 80 || R > 128)) return false;
  const uint64_t elems = (uint64_t)n_tiles * vector_elems(h) * R;
  return elems >= (R < 72 ? kManyElems : R < 96 ? 5 * kManyElems : wide ? kManyElems * 5 / 2 : kManyElems);
}

// Do workgroups of four wavefronts take whole items of a launch over die groups, instead of eight workgroups of one?
// Mixing always (see k_rows).  Steps of 33 to 63 float32 rows of 1e8 elements and more: time of one-wavefront pieces over
// this, 3e8 elements, rows in pairs, update only / whole step: 24 rows 0.98 / 0.99, 32 rows 0.99 / 1.00, 40 rows 1.04 / 1.03,
// 48 rows 1.01 / 1.01, 56 rows 1.00 / 1.01, 72 rows 1.00 / 0.98; 3e7 elements 0.98 to 1.00; bfloat16 0.98 to 1.01, 3e7 0.95 to 0.98.
bool whole_items(const dadam_handle* h, bool mix_only, uint32_t order, uint64_t elems) {
  if (order != kOrderDieGroups) return false;
  if (h->mapped && !mix_only) return false;  // (k_rows has no body for maps: with it 74 registers became 87, a wavefront per SIMD)
  return mix_only || (h->cfg.n_rows > 32 && h->cfg.n_rows < 64 && h->vec == 4 && h->d_tables == nullptr && h->nontemporal && elems >= kManyElems);
}

// The same question for accumulation.  Time of one-wavefront pieces over whole items, 3e8 elements: 1 row 0.90, 16 rows 0.96,
// 24 rows 0.98, 32 rows 0.98, 40 rows 1.03, 48 rows 1.02, 64 rows 1.01, 72 rows 0.99, 96 rows 1.03, 128 rows 1.00, 160 rows
// 1.00 (bfloat16 0.96, 0.93, 0.97, 0.97, 1.00, 1.00, 1.01, 0.98, 1.01, 0.99, 0.99); 3e7 elements 0.92 to 1.01.
// Segments of 1100 elements, us, pieces / whole items, 2e8 elements: 40 rows 2300 / 1804, 64 rows 2352 / 1894, 90 rows 2250 / 1960, 110 rows
// 2222 / 1996, with bfloat16 parameters (eight elements a lane) 1789 / 1975, 1847 / 2007, 1966 / 2558, 2018 / 2566.
bool accumulate_whole_items(const dadam_handle* h, uint64_t elems) {
  const uint32_t R = h->cfg.n_rows;
  if (h->mapped || (h->short_segments && h->vec == 8)) return false;  // (as in whole_items)
  return h->nontemporal && elems >= kManyElems && ((R > 32 && R <= 64) || (R > 80 && R < 128));
}

// Streaming launches of rows that share sources for which the tile kernel and the direct one have changed places since
// lanes are spread, sixteen wavefronts share a tile and dies walk runs of pieces.  usual: what choose_mode says.
// Fraction of 8 TB/s, tile / direct, 3e8 elements:
//   steps of rows of three sources: 24 of them 0.80 / 0.80, 32 0.78 / 0.80, 48 0.78 / 0.80, 64 0.78 / 0.80, bfloat16 32 0.78 / 0.80, 48 0.77 /
//   0.80; of six (32 rows) and seven (64 rows) the tile stays ahead, 0.80 / 0.74;
//   mixing in pairs: 18 rows 0.81 / 0.57, 24 rows 0.80 / 0.74, 28 rows 0.80 / 0.72 (bfloat16 0.72 / 0.58, 0.73 / 0.70, 0.75 / 0.70);
//   96 rows, whose tile leaves a compute unit one workgroup: steps with four sources a row 0.71 / 0.71, five 0.71 / 0.67, six 0.70 /
//   0.64, seven 0.70 / 0.60 (bfloat16 four 0.73 / 0.75, five 0.73 / 0.74, six 0.74 / 0.73, seven 0.73 / 0.68), mixing with
//   three (128 rows) 0.63 / 0.66, four 0.59 / 0.48, seven 0.51 / 0.36 (bfloat16 four 0.46 / 0.48, six 0.41 / 0.39).
// Launches that do not stream stay: 128 rows of seven, 1e7 elements, 0.48 / 0.60.
// Segments of 1100 elements, us, tile / direct: steps of bfloat16 rows of seven, 96 of them 1263 / 1091, 128 rows 1292 / 1107 (float32 1352 / 1503, 1376 /
// 1577); mixing in pairs 24 rows 898 / 1673, 32 rows 910 / 1606, 48 rows 1088 / 1902, 64 rows 1068 / 1891 (bfloat16 545 / 1801, 514 / 1797, 655 / 2123, 717 / 2120), 96 and
// 160 rows 1712 / 2405, 1791 / 2808 (1321 / 2578, 1555 / 2957), with three sources 504 / 791, 468 / 812 (398 / 881, 409 / 884).
bool staging_is_faster(const dadam_handle* h, const Slot& slot, bool mix_only, uint32_t n_tiles, bool usual) {
  if (!many_tiles(h, n_tiles)) return usual;
  const uint32_t C = h->cfg.n_cols;
  if (h->short_segments && (usual || mix_only)) return true;
  if (usual) return mix_only || slot.max_degree > 3 || C < 32;
  if (lone_tile(h)) return h->shape.waves == 16 && slot.max_degree >= (h->vec == 8 ? 6 : mix_only ? 4 : 5) && (!h->short_segments || (h->vec == 4 && n_tiles >= kManyTiles));
  return mix_only && C < 32;
}

// Launches over a layout with a map that go by its segments all the same, because these are long: what a map saves is cut tiles and the search for a
// segment, and where the tile and loop kernels are bound by more than that, its byte for every four elements and its tests at every store, and lanes
// that it lets spread over segments (bfloat16 mixing by the tile has them side by side where segments end), cost more.  The sums are the same.  From which
// average length on, by time by segments over time by the map, 3e8 elements of all rows in tensors of 1500, 3000, 6000, 12000, 24000 (30000 of the tile) elements:
//   loops in float32   32 rows steps 1.13 1.10 1.07 1.03 0.97, mixing 1.06 1.03 1.05 1.00 0.96   64 rows 1.16 1.11 1.09 1.08 1.00, 1.10 1.07 1.08 1.04 0.95 (in loops of 32, 16, 16
//     1.13 1.11 1.06 1.02 0.97, 1.05 0.96 0.95 0.98 0.95)
//     72 rows 1.07 1.01 0.98 0.94 0.89, 1.01 0.98 0.93 0.97 0.90   96 rows 1.07 1.03 1.00 0.96 0.91, 1.01 0.96 0.93 0.91 0.89 (in loops of 48, 24, 24 1.09 1.02 1.00 0.95
//     0.92, 1.02 0.93 0.90 0.88 0.89)   128 rows 1.11 1.05 1.02 1.00 0.95, 1.09 1.05 1.03 0.98 0.96
//   loops in bfloat16  72 to 128 rows steps 1.5 to 1.12, mixing 1.33 1.11 1.01 0.95 0.92, 96 rows 1.39 1.16 1.04 1.00 0.96
//   mixing by the tile in bfloat16, three sources  18 rows 1.35 1.19 1.11 1.07 1.08   24 rows 1.13 1.00 0.94 0.93 0.90   32 rows 1.04 0.93 0.92 0.92 0.91   48 rows 1.04 0.92
//     0.89 0.88 0.86   64 rows 1.08 1.00 0.89 0.90 0.90 (1e8 elements 24 rows 1.19 1.08 1.03 1.02 1.00, 48 rows 1.14 1.03 0.99 0.96 0.96, 56 rows 1.21 1.07 1.03 0.98 0.98; 3e7
//     1.17 and less to 0.98; 81 rows and more 1.4 to 1.07)
//   steps by the tile in float32, seven sources  72 rows 1.24 to 1.11   96 rows - 1.02 0.97 0.95 1.00   128 rows - 1.03 0.98 0.96 0.99   160 rows - 1.03 1.00 0.98 1.00
// 24000, 40000 elements, less in all: loops in float32 32 rows of 9.6e7 steps 0.98 0.96, mixing 0.96 0.94, 64 rows of 1.9e8 0.99 0.97, 0.95 0.94, bfloat16 mixing 0.97 0.97; from 1.9e7 to
// 6e7 1.00 to 1.3.  What else has a map loses nothing by it or 1 to 3 % at most (of 1.2e8 elements and less, segments of 12000 and more).
// n_loops: of a launch of the loop kernel, otherwise 0.
bool segments_are_faster(const dadam_handle* h, bool tile_mode, size_t n_loops, bool mix_only, uint64_t elems) {
  if (!h->nontemporal || !tile_mode || elems < kSegmentElems) return false;
  const uint32_t R = h->cfg.n_rows, C = h->cfg.n_cols;
  const bool most = elems >= 2 * kManyElems, tables = R > (uint32_t)kInlineRows || C > (uint32_t)kInlineRows;  // (in device memory)
  uint64_t from = 0;  // 0: never
  if (n_loops > 0 && h->vec == 8 && mix_only) from = most ? 8192 : tables ? 0 : 20480;
  if (n_loops > 0 && h->vec == 4 && !tables) from = !most ? 20480 : mix_only && n_loops > 1 ? 2560 : 16384;
  if (n_loops > 0 && h->vec == 4 && tables && most) from = !mix_only ? 6144 : R < 112 ? 2048 : 8192;
  if (n_loops == 0 && h->vec == 8 && mix_only && !tables && C >= 24) from = !most ? 12288 : C < 32 ? 4096 : 2560;
  if (n_loops == 0 && h->vec == 4 && !mix_only && tables && lone_tile(h) && most) from = 5120;
  return from != 0 && h->n_elems >= from * h->segs.size();
}

// LDS a workgroup of a large one-row step reserves without using it, to bound how many wavefronts a compute unit
// holds: with all 32 of them the row's 8 or 9 streams are requested over too wide a window of memory.  What counts
// is the bytes of loads in flight per unit; about 90 KB is best.  Fraction of 8 TB/s, by wavefronts per unit,
// one row with three sources, 3e8 elements: float32 (7 KB a wavefront) 32: 0.772, 18: 0.791, 14: 0.800, 11: 0.809,
// 9: 0.780; bfloat16 (10 KB) 32: 0.744, 14: 0.770, 11: 0.787, 9: 0.805; s = 1 0.767 -> 0.809.  Short launches need
// every wavefront (12000 pieces: 0.725 -> 0.670; 25000 in buckets 0.743 -> 0.713; 117000: 0.755 -> 0.779), and so do
// the passes that load little (mixing 0.828 -> 0.625, accumulation).  Only one row was measured.
uint32_t bounded_occupancy_lds(const dadam_handle* h, const Slot& slot, Phase phase, bool streams, uint32_t n_pieces) {
  if (h->cfg.n_rows != 1 || phase == kMixOnly || !streams || n_pieces < kBoundedPieces) return 0;
  if (h->lds_limit < kLdsPerUnit) return 0;  // the configuration keeps LDS for other kernels
  const uint32_t state = kWave * 4 * (uint32_t)h->vec;
  const uint32_t loads = 16 * kWave * (uint32_t)std::min(slot.max_degree, 8) + kWave * (uint32_t)h->vec * (uint32_t)dtype_bytes(h->cfg.grad_dtype) +
                         state * (phase == kPlain || phase == kFold ? 3u : 2u);
  const uint32_t waves = std::max(4u, kInFlightBytes / loads);
  if (waves >= 20) return 0;
  return kLdsPerUnit / waves / kLdsGranule * kLdsGranule;
}

int resolve_range(const dadam_handle* h, uint32_t tb, uint32_t te, bool whole, uint64_t* lo,
                  uint64_t* hi, uint32_t* s0, uint32_t* s1, bool* empty) {
  *empty = false;
  if (whole) {
    if (h->segs.empty()) { *empty = true; return DADAM_OK; }
    *lo = h->segs.front().lo;
    *hi = h->segs.back().hi;
    *s0 = 0;
    *s1 = (uint32_t)h->segs.size() - 1;
    return DADAM_OK;
  }
  if (tb > te || te > h->tensors.size())
    return fail(h, DADAM_EINVAL, "tensor range [%u, %u) outside [0, %zu]", tb, te, h->tensors.size());
  uint32_t first = UINT32_MAX, last = UINT32_MAX;
  for (uint32_t k = tb; k < te; ++k)
    if (h->tensor_seg[k] != UINT32_MAX) { if (first == UINT32_MAX) first = k; last = k; }
  if (first == UINT32_MAX) { *empty = true; return DADAM_OK; }
  *lo = h->tensors[first].offset_elems;
  *hi = h->tensors[last].offset_elems + h->tensors[last].numel;
  *s0 = h->tensor_seg[first];
  *s1 = h->tensor_seg[last];
  return DADAM_OK;
}

int step_impl(dadam_handle* h, uint32_t slot_id, const void* const* grads, uint64_t t, uint32_t flags,
              bool whole, uint32_t tb, uint32_t te, bool mix_only, void* stream, double* consensus_out = nullptr,
              double* partials = nullptr) {
  if (!h) return DADAM_EINVAL;
  int rc = check_bound(h);
  if (rc) return rc;
  if (slot_id >= DADAM_MAX_SLOTS || !h->slots[slot_id].set)
    return fail(h, DADAM_ESTATE, "topology slot %u is not set", slot_id);
  if (flags & ~(DADAM_FUSE_ACCUM | DADAM_FORCE_DIRECT | DADAM_FORCE_TILE))
    return fail(h, DADAM_EINVAL, "unknown flag bits 0x%x", flags);
  const Slot& slot = h->slots[slot_id];
  Phase phase = kMixOnly;
  if (!mix_only) {
    if (t == 0) return fail(h, DADAM_EINVAL, "iterations are numbered from 1");
    rc = check_grads(h, grads);
    if (rc) return rc;
    phase = (flags & DADAM_FUSE_ACCUM) ? fused_phase(h, t) : kUpdateOnly;
    if (h->cfg.accum_s > 1 && (flags & DADAM_FUSE_ACCUM))
      for (uint32_t i = 0; i < h->cfg.n_rows; ++i)
        if (!h->acc[i]) return fail(h, DADAM_ESTATE, "accumulator of row %u is not bound", i);
  }
  bool tile_mode = false;
  // the consensus error is computed from the staged tile: ask for tile mode unless the caller chose
  if (consensus_out && !(flags & DADAM_FORCE_DIRECT) && h->tile_possible && slot.reuse) flags |= DADAM_FORCE_TILE;
  const bool decays = !mix_only && range_decays(h, whole, tb, te);
  rc = choose_mode(h, slot, flags, decays, &tile_mode);
  if (rc) return rc;
  if (consensus_out) {
    if (!tile_mode)
      return fail(h, DADAM_ESTATE, "the consensus error is a by-product of tile mode (shared sources that fit in LDS)");
    phase = kMixConsensus;
  }
  uint64_t lo = 0, hi = 0;
  uint32_t s0 = 0, s1 = 0;
  bool empty = false;
  rc = resolve_range(h, tb, te, whole, &lo, &hi, &s0, &s1, &empty);
  if (rc) return rc;
  rc = check_device(h);
  if (rc) return rc;
  if (!partials) partials = h->d_partials;
  DeviceGuard guard(h->cfg.device);
  if (guard.err != hipSuccess) return fail(h, DADAM_EHIP, "hipSetDevice: %s", hipGetErrorString(guard.err));
  // The handle's own partial sums are clear after every pass that ran whole, so the next one needs no launch to clear
  // them.  What a pass under stream capture records runs later, any number of times and behind whatever came in
  // between: it always clears first, and says nothing about what the memory holds now.
  const bool own_partials = consensus_out && partials == h->d_partials;
  bool recorded = false;
  if (own_partials) {
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(reinterpret_cast<hipStream_t>(stream), &capture) != hipSuccess) {
      (void)hipGetLastError();
      recorded = true;
    }
    if (capture != hipStreamCaptureStatusNone) recorded = true;
  }
  if (consensus_out && !(own_partials && !recorded && h->partials_clear)) {
    int e0 = launch_consensus_zero(partials, stream);
    if (e0 != (int)hipSuccess) return fail(h, DADAM_EHIP, "kernel launch failed: %s", hipGetErrorString((hipError_t)e0));
  }
  if (own_partials && !recorded) h->partials_clear = false;
  if (empty) {
    if (consensus_out) (void)launch_consensus_sum(partials, consensus_out, stream);
    return DADAM_OK;
  }
  uint32_t w0 = 0, w1 = 0;
  work_range(h, h->mapped, kGridVector, s0, s1, lo, hi, &w0, &w1);
  const uint32_t n_tiles = w1 - w0;
  const int loop_waves = consensus_out || (flags & (DADAM_FORCE_TILE | DADAM_FORCE_DIRECT)) ? 0 : loop_kernel_waves(h, slot, mix_only);
  const bool by_loops = loop_waves > 0;
  const bool few_tiles = !by_loops && tile_mode && !consensus_out && !(flags & DADAM_FORCE_TILE) && h->cfg.n_rows > 8 &&
                         n_tiles <= few_tiles_limit(h, slot) && direct_is_legal(h, slot, decays);
  if (h->nontemporal && !by_loops && !few_tiles && !consensus_out &&
      !(flags & (DADAM_FORCE_TILE | DADAM_FORCE_DIRECT)) && slot.reuse && h->n_xcds > 1 && h->tile_possible && direct_is_legal(h, slot, decays))
    tile_mode = staging_is_faster(h, slot, mix_only, n_tiles, tile_mode);
  if (few_tiles) tile_mode = false;
  if (by_loops) tile_mode = true;
  const bool streams = h->nontemporal || (!mix_only && few_rows_stream(h, slot.n_read));
  // streaming float32 steps take two vectors a lane (see dadam_init): in a handle whose other launches do not stream, the mixing tile has them
  const bool mixing_tile = mix_only || (streams && !h->nontemporal && h->vec == 4 && h->mix_shape.ut == 2);
  const Grid grid = !tile_mode ? kGridDirect : by_loops ? kGridVector : mixing_tile ? kGridMix : kGridTile;
  const bool by_map = h->mapped && !segments_are_faster(h, tile_mode, by_loops ? slot.loops.size() : 0, mix_only, (uint64_t)n_tiles * vector_elems(h) * h->cfg.n_rows);
  work_range(h, by_map, grid, s0, s1, lo, hi, &w0, &w1);
  StepArgs a;
  fill_args(h, by_map, mix_only ? nullptr : grads, &a);
  if (!tile_mode && ordered_rows(h, slot)) a.order = rows_stay_on_one_die(h, slot, mix_only, n_tiles) ? kOrderDieBlocks : kOrderDieGroups;
  if (a.order == kOrderDieBlocks && many_tiles(h, n_tiles) && !(h->nontemporal && h->short_segments)) set_die_run(kDieRunPieces, &a);
  set_range(h, by_map, decays, grid, w0, lo, hi, &a);
  if (tile_mode && cut_by_elements(h, mix_only, by_loops)) a.d = 0;
  a.partials = partials;
  if (!tile_mode) a.reserve_lds = bounded_occupancy_lds(h, slot, phase, streams, (w1 - w0) * kDirectItem);
  fill_scalars(h, mix_only ? 1 : t, &a.s);
  TileShape shape = mixing_tile ? h->mix_shape : h->shape;
  shape.nontemporal = streams;
  uint32_t lds = mixing_tile ? h->mix_lds_bytes : h->lds_bytes;
  if (by_loops) {
    a.loops = slot.d_loops;
    a.n_loops = (uint32_t)slot.loops.size();
    const uint64_t T = vector_elems(h);
    a.loop_shares = loop_shares(h, slot, loop_waves, n_tiles, a.n_seg > 1 || (by_map ? h->vec == 4 : lo % T != 0 || hi % T != 0), mix_only);
    a.col = slot.d_loop_col;
    a.w = slot.d_loop_w;
    a.row_order = slot.d_loop_rows;
    shape.ut = 1;
    shape.waves = loop_waves;
    if (h->nontemporal) a.xcd_block = kDieBlockLoops;
    lds = loop_lds_bytes(h, shape.waves);
  } else if (tile_mode) {
    if (mix_only && h->nontemporal && shape.ut == 2) a.xcd_block = kDieBlockMix;
    a.row_ptr = slot.d_row_ptr;
    a.col = slot.d_col;
    a.w = slot.d_w;
  } else {
    a.row_len = slot.d_row_len;
    a.col = slot.d_list_col;
    a.w = slot.d_list_w;
    a.row_order = slot.d_row_order;
    a.list_stride = (uint32_t)slot.max_degree;
    a.order_group = (h->cfg.n_rows + h->n_xcds - 1) / h->n_xcds;
  }
  const uint64_t wavefronts = (uint64_t)(w1 - w0) * (tile_mode ? shape.waves * (by_loops ? slot.loops.size() * a.loop_shares : 1) : kDirectItem * (uint64_t)h->cfg.n_rows);
  a.wide_search = wavefronts <= kWideSearchWaves ? 1u : 0u;
  int e = tile_mode
              ? launch_tile((int)h->cfg.param_dtype, (int)h->cfg.grad_dtype, phase, shape, a, w1 - w0, lds, stream)
              : launch_direct((int)h->cfg.param_dtype, (int)h->cfg.grad_dtype, phase,
                              // where rows share sources the re-reads must find them in the cache
                              streams, slot.reuse, whole_items(h, mix_only, a.order, (uint64_t)n_tiles * vector_elems(h) * h->cfg.n_rows),
                              a, w1 - w0, stream);
  if (e == (int)hipSuccess && consensus_out) e = launch_consensus_sum(partials, consensus_out, stream);
  if (e == (int)hipSuccess && own_partials && !recorded) h->partials_clear = true;
  if (e != (int)hipSuccess)
    return fail(h, DADAM_EHIP, "kernel launch failed: %s", hipGetErrorString((hipError_t)e));
  return DADAM_OK;
}

// Rows in an order in which consecutive rows share as many sources as possible (greedy: from the current row
// to the unvisited row that shares most sources with it, the lowest-numbered on a tie; when nothing is shared
// any more, on to the lowest unvisited row).  A one-peer graph with hop h comes out as its chains
// 0, h, 2h, ..., a ring as 0, 1, 2, ...  The direct kernels hand contiguous groups of this order to the dies.
std::vector<int32_t> sharing_order(uint32_t R, uint32_t C, const int32_t* row_ptr, const int32_t* col) {
  std::vector<std::vector<int32_t>> readers(C);
  for (uint32_t i = 0; i < R; ++i)
    for (int32_t k = row_ptr[i]; k < row_ptr[i + 1]; ++k) readers[col[k]].push_back((int32_t)i);
  std::vector<int32_t> order;
  std::vector<char> visited(R, 0);
  std::vector<int32_t> shared(R);
  uint32_t lowest = 0;
  int32_t cur = 0;
  while (true) {
    order.push_back(cur);
    visited[cur] = 1;
    if (order.size() == R) break;
    std::fill(shared.begin(), shared.end(), 0);
    for (int32_t k = row_ptr[cur]; k < row_ptr[cur + 1]; ++k)
      for (int32_t j : readers[col[k]])
        if (!visited[j]) ++shared[j];
    int32_t best = -1;
    for (uint32_t j = 0; j < R; ++j)
      if (shared[j] > 0 && (best < 0 || shared[j] > shared[best])) best = (int32_t)j;
    if (best < 0) {
      while (visited[lowest]) ++lowest;
      best = (int32_t)lowest;
    }
    cur = best;
  }
  return order;
}

// The loops of a neighbour list, for the loop kernel: at least eight rows to a loop on average, so that a
// workgroup's wavefronts have rows to share, and no source in two loops, so that each is read once.
// col / w / rows: the loops' entries, in source order, and their rows.
void find_loops(uint32_t R, uint32_t C, Slot& s, std::vector<int32_t>& col, std::vector<float>& w, std::vector<int32_t>& rows) {
  std::map<std::vector<std::pair<int32_t, float>>, std::vector<int32_t>> by_list;
  for (uint32_t i = 0; i < R; ++i) {
    std::vector<std::pair<int32_t, float>> list;
    for (int32_t k = s.row_ptr[i]; k < s.row_ptr[i + 1]; ++k) list.push_back({s.col[k], s.w[k]});
    std::sort(list.begin(), list.end());
    by_list[list].push_back((int32_t)i);
    if (by_list.size() * 8 > R) return;
  }
  std::vector<int32_t> of_row(R, -1), of_source(C, -1);
  std::vector<Loop> loops;
  for (const auto& it : by_list) {
    const int32_t id = (int32_t)loops.size();
    loops.push_back({(int32_t)col.size(), (int32_t)it.first.size(), (int32_t)rows.size(), (int32_t)it.second.size()});
    for (const auto& e : it.first) {
      if (of_source[e.first] != -1) return;
      of_source[e.first] = id;
      col.push_back(e.first);
      w.push_back(e.second);
    }
    for (int32_t i : it.second) { of_row[i] = id; rows.push_back(i); }
  }
  s.loops = loops;
  s.loop_of_row = of_row;
  s.loop_of_source = of_source;
}

// Device copies of everything the kernels read of a slot, in one allocation.
hipError_t upload_lists(const dadam_handle* h, Slot& s, const std::vector<int32_t>& loop_col, const std::vector<float>& loop_w,
                        const std::vector<int32_t>& loop_rows) {
  const int32_t R = (int32_t)h->cfg.n_rows, stride = s.max_degree;
  std::vector<int32_t> rows(R), len(R), lcol((size_t)R * stride, 0);
  std::vector<float> lw((size_t)R * stride, 0.0f);
  for (int32_t p = 0; p < R; ++p) {
    const int32_t i = ordered_rows(h, s) ? s.order[p] : p;
    rows[p] = i;
    len[p] = s.row_ptr[i + 1] - s.row_ptr[i];
    std::copy_n(s.col.begin() + s.row_ptr[i], len[p], lcol.begin() + (size_t)p * stride);
    std::copy_n(s.w.begin() + s.row_ptr[i], len[p], lw.begin() + (size_t)p * stride);
  }
  std::vector<char> image;
  auto add = [&image](const auto& v) {
    const size_t at = image.size();
    image.resize(at + (v.size() * sizeof(v[0]) + 255) / 256 * 256);
    memcpy(image.data() + at, v.data(), v.size() * sizeof(v[0]));
    return at;
  };
  const size_t row_ptr = add(s.row_ptr), col = add(s.col), w = add(s.w);
  const size_t row_len = add(len), list_col = add(lcol), list_w = add(lw), row_order = add(rows);
  const bool has_loops = !s.loops.empty();
  const size_t l = has_loops ? add(s.loops) : 0, lc = has_loops ? add(loop_col) : 0, lww = has_loops ? add(loop_w) : 0,
               lr = has_loops ? add(loop_rows) : 0;
  hipError_t e = hipMalloc((void**)&s.d_lists, image.size());
  if (e == hipSuccess) e = hipMemcpy(s.d_lists, image.data(), image.size(), hipMemcpyHostToDevice);
  if (e != hipSuccess) return e;
  auto ints = [&s](size_t at) { return reinterpret_cast<const int32_t*>(s.d_lists + at); };
  auto floats = [&s](size_t at) { return reinterpret_cast<const float*>(s.d_lists + at); };
  s.d_row_ptr = ints(row_ptr); s.d_col = ints(col); s.d_w = floats(w);
  s.d_row_len = ints(row_len); s.d_list_col = ints(list_col); s.d_list_w = floats(list_w); s.d_row_order = ints(row_order);
  if (has_loops) {
    s.d_loops = reinterpret_cast<const Loop*>(s.d_lists + l);
    s.d_loop_col = ints(lc); s.d_loop_w = floats(lww); s.d_loop_rows = ints(lr);
  }
  return hipSuccess;
}

void free_slot(Slot& s) {
  if (s.d_lists) (void)hipFree(s.d_lists);
  s = Slot();
}

}  // namespace

// -------------------------------------------------------------------------------------------------
// C ABI
// -------------------------------------------------------------------------------------------------
extern "C" {

int dadam_init(const dadam_config* cfg, dadam_handle** out) {
  if (!cfg || !out) return fail(nullptr, DADAM_EINVAL, "cfg or out is null");
  if (cfg->abi_version != DADAM_ABI_VERSION)
    return fail(nullptr, DADAM_EINVAL, "abi_version %u, library has %u", cfg->abi_version, DADAM_ABI_VERSION);
  if (cfg->n_rows == 0 || cfg->n_rows > DADAM_MAX_ROWS || cfg->n_cols == 0 || cfg->n_cols > DADAM_MAX_ROWS)
    return fail(nullptr, DADAM_EINVAL, "n_rows and n_cols must be in [1, %u]", DADAM_MAX_ROWS);
  if (cfg->d == 0) return fail(nullptr, DADAM_EINVAL, "d is zero");
  if (cfg->d > (1ull << 40)) return fail(nullptr, DADAM_EINVAL, "d too large");
  if (cfg->param_dtype > DADAM_BF16 || cfg->grad_dtype > DADAM_BF16)
    return fail(nullptr, DADAM_EINVAL, "unknown dtype");
  if (cfg->accum_s == 0) return fail(nullptr, DADAM_EINVAL, "accum_s must be >= 1");
  if (!std::isfinite(cfg->lr)) return fail(nullptr, DADAM_EINVAL, "lr is not finite");
  if (!(cfg->beta1 >= 0.f && cfg->beta1 < 1.f) || !(cfg->beta2 >= 0.f && cfg->beta2 < 1.f))
    return fail(nullptr, DADAM_EINVAL, "betas must be in [0, 1)");
  if (!(cfg->eps >= 0.f) || !std::isfinite(cfg->eps)) return fail(nullptr, DADAM_EINVAL, "eps must be finite and >= 0");
  if (cfg->n_tensors > 0 && !cfg->tensors) return fail(nullptr, DADAM_EINVAL, "tensors is null");
  if (cfg->n_tensors == 0) return fail(nullptr, DADAM_EINVAL, "the layout has no tensors");
  if (cfg->device < 0 && cfg->device != DADAM_DEVICE_NONE) return fail(nullptr, DADAM_EINVAL, "bad device ordinal");
  double betav = (double)cfg->beta2;
  if (!std::isnan(cfg->beta_vhat) && cfg->beta_vhat >= 0.f) {
    if (!(cfg->beta_vhat < 1.f)) return fail(nullptr, DADAM_EINVAL, "beta_vhat must be in [0, 1)");
    betav = (double)cfg->beta_vhat;
  }
  uint64_t prev_end = 0;
  for (uint32_t k = 0; k < cfg->n_tensors; ++k) {
    const dadam_tensor_desc& t = cfg->tensors[k];
    if (t.offset_elems < prev_end)
      return fail(nullptr, DADAM_EINVAL, "tensor %u starts before tensor %u ends (list must be ordered and disjoint)", k, k ? k - 1 : 0);
    if (t.numel > cfg->d || t.offset_elems > cfg->d - t.numel)
      return fail(nullptr, DADAM_EINVAL, "tensor %u reaches beyond d", k);
    if (!(t.weight_decay >= 0.f) || !std::isfinite(t.weight_decay))
      return fail(nullptr, DADAM_EINVAL, "tensor %u: weight_decay must be finite and >= 0", k);
    if (t.flags != 0) return fail(nullptr, DADAM_EINVAL, "tensor %u: flags is reserved and must be 0", k);
    if (t.weight_decay > 0.f && cfg->n_rows > cfg->n_cols)
      return fail(nullptr, DADAM_EINVAL, "weight decay needs source buffer i to be row i's own parameters (n_rows <= n_cols)");
    prev_end = t.offset_elems + t.numel;
  }
  dadam_handle* h = new (std::nothrow) dadam_handle();
  if (!h) return fail(nullptr, DADAM_EINVAL, "out of host memory");
  h->cfg = *cfg;
  h->tensors.assign(cfg->tensors, cfg->tensors + cfg->n_tensors);
  h->cfg.tensors = nullptr;
  h->lr = cfg->lr;
  h->betav = betav;

  // What the chip offers: LDS one workgroup may use and the number of dies (XCDs), asked of the
  // device; a host-only handle plans for 64 KB and 8 dies unless the configuration says otherwise.
  if (cfg->device != DADAM_DEVICE_NONE) {
    int lds = 0, xcc = 0;
    hipError_t e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, cfg->device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&xcc, hipDeviceAttributeNumberOfXccs, cfg->device);
    if (e != hipSuccess || lds <= 0) {
      delete h;
      return fail(nullptr, DADAM_EHIP, "cannot read the device's LDS size / die count: %s", hipGetErrorString(e));
    }
    h->lds_limit = (uint32_t)lds;
    h->n_xcds = xcc > 0 ? (uint32_t)xcc : 1u;
    if (cfg->lds_limit_bytes > h->lds_limit) {
      delete h;
      return fail(nullptr, DADAM_EINVAL, "lds_limit_bytes %u exceeds the device's %u", cfg->lds_limit_bytes, h->lds_limit);
    }
  }
  if (cfg->lds_limit_bytes) h->lds_limit = cfg->lds_limit_bytes;
  if (cfg->n_xcds) h->n_xcds = cfg->n_xcds;
  h->n_xcds = (uint32_t)env_int("DADAM_XCDS", (int)h->n_xcds);
  if (h->n_xcds > 64) { delete h; return fail(nullptr, DADAM_EINVAL, "n_xcds out of range"); }

  // tile geometry: 16 bytes per lane and vector, `ut` vectors per lane, all source buffers' slices
  // of one tile resident in LDS.  One vector per lane (many small workgroups) and eight wavefronts per group, four when there
  // are fewer than eight rows to deal out; larger launches below.
  h->vec = vec_elems((int)cfg->param_dtype);
  TileShape shape;
  shape.ut = 1;
  shape.waves = cfg->n_rows >= 8 ? 8 : 4;
  // Non-temporal accesses pay off when an iteration's working set cannot stay in the last-level
  // cache anyway; small problems keep ordinary accesses so that one iteration finds the previous
  // one's output on chip (steps of up to three rows go by what they touch, see few_rows_stream).
  const double touched = (double)cfg->d * cfg->n_rows * 24.0;
  h->nontemporal = env_int("DADAM_NT", touched > 512.0 * 1024 * 1024 ? 1 : 0) != 0;
  shape.nontemporal = h->nontemporal;
  shape.ut = env_int("DADAM_TILE_UT", shape.ut);
  shape.waves = env_int("DADAM_TILE_WAVES", shape.waves);
  // Streaming float32 steps: two vectors a lane, which lie the way the memory serves best (see lane_start), up to the
  // sources whose tile fits; sixteen wavefronts from 16 rows on.  Fraction of 8 TB/s, one vector by eight wavefronts / two by
  // eight / two by sixteen, 3e8 to 2e9 elements: 16 rows 0.710 / 0.802 / 0.814, 24 rows 0.801 / 0.802 / 0.809, 48 rows 0.783 / 0.806 /
  // 0.805, 72 rows 0.72 / 0.725 / 0.779; 8 rows 0.817 / 0.825 / 0.802, 4 rows by four wavefronts 0.816 / 0.820, by sixteen 0.794.
  // In bfloat16 one vector has that layout already, and sixteen wavefronts lose (8 rows 0.813 / 0.783, 16 rows 0.780 / 0.770).
  find_segments(h);
  h->mapped = env_int("DADAM_MAP", 1) && can_map(h, &h->map_decay);
  if (h->mapped) h->short_segments = false;
  if (env_int("DADAM_TILE_UT", 0) == 0 && h->nontemporal && !h->short_segments && h->vec == 4 && cfg->n_cols * 2u * kWave * 16u <= h->lds_limit) {
    shape.ut = 2;
    if (cfg->n_rows >= 16) shape.waves = env_int("DADAM_TILE_WAVES", 16);
  } else if (cfg->n_cols > (uint32_t)kInlineRows && lone_tile(h) && cfg->n_rows >= 16) {
    // A compute unit holds one workgroup of the tile: sixteen wavefronts keep more of it busy.  us, eight / sixteen: steps of 96
    // rows with 16 sources each, 3e8 elements 9850 / 6860, 1e7 elements 430 / 295; 128 rows of 12 in bfloat16, 3e7 elements 910 / 690; mixing of
    // 96 rows with 7 sources, 3e8 elements 1730 / 1190, with the error 1e8 elements 650 / 460.
    shape.waves = env_int("DADAM_TILE_WAVES", 16);
  }
  if (!tile_shape_supported(shape)) {
    delete h;
    return fail(nullptr, DADAM_EINVAL, "unsupported tile shape (waves %d, ut %d)", shape.waves, shape.ut);
  }
  h->shape = shape;
  h->tile_elems = (uint32_t)(kWave * h->vec * shape.ut);
  h->direct_elems = (uint32_t)(kWave * h->vec * kDirectItem);
  h->lds_bytes = cfg->n_cols * (uint32_t)shape.ut * kWave * 16u;
  h->tile_possible = h->lds_bytes <= h->lds_limit;
  // The mixing-only launch moves few bytes per row, so it wants more of them in flight per
  // wavefront: two vectors per lane and four wavefronts, as long as that tile stays small enough
  // (32 KB) for five workgroups to share a CU's LDS.  Measured: 16 sources (32 KB) +3 % over the
  // step's shape; with 64 sources (128 KB, one workgroup per CU) and contiguous lanes 0.68-0.75 of peak against 0.76 with the
  // step's one-vector tile, so larger source counts keep the step's shape.  Streaming float32 passes spread the lanes and take eight
  // wavefronts up to 32 sources, then the step's sixteen (four / eight / sixteen: 12 sources 0.815 / 0.814, 16 sources 0.810 / 0.819, with
  // the error 0.750 / 0.778, 24 sources 0.797 / 0.812 / 0.809, with the error 0.73 / 0.80 / 0.74, 48 sources 0.63 / 0.745 / 0.780).
  h->mix_shape = shape;
  if (cfg->n_cols * 2u * kWave * 16u <= 32768u && h->lds_limit >= 32768u && env_int("DADAM_TILE_UT", 0) == 0 &&
      env_int("DADAM_TILE_WAVES", 0) == 0) {
    h->mix_shape.ut = 2;
    h->mix_shape.waves = 4;
  }
  if (h->nontemporal && !h->short_segments && h->vec == 4 && cfg->n_rows >= 8 && cfg->n_cols <= 32 && h->mix_shape.ut == 2)
    h->mix_shape.waves = 8;
  h->mix_shape.ut = env_int("DADAM_MIX_UT", h->mix_shape.ut);
  h->mix_shape.waves = env_int("DADAM_MIX_WAVES", h->mix_shape.waves);
  if (!tile_shape_supported(h->mix_shape) || cfg->n_cols * (uint32_t)h->mix_shape.ut * kWave * 16u > h->lds_limit)
    h->mix_shape = shape;
  h->mix_tile_elems = (uint32_t)(kWave * h->vec * h->mix_shape.ut);
  h->mix_lds_bytes = cfg->n_cols * (uint32_t)h->mix_shape.ut * kWave * 16u;
  int rc = plan(h);
  if (rc) { delete h; return rc; }

  if (cfg->device != DADAM_DEVICE_NONE) {
    DeviceGuard guard(cfg->device);
    hipError_t e = guard.err;
    if (e == hipSuccess && !h->segs.empty()) {
      const size_t n = h->segs.size(), bytes = n * sizeof(Segment);
      std::vector<char> image(bytes + kNumGrids * n * sizeof(uint32_t));
      memcpy(image.data(), h->segs.data(), bytes);
      for (int g = 0; g < (int)kNumGrids; ++g)
        memcpy(image.data() + bytes + g * n * sizeof(uint32_t), h->seg_work[g].data(), n * sizeof(uint32_t));
      e = hipMalloc((void**)&h->d_segs, image.size());
      if (e == hipSuccess) e = hipMemcpy(h->d_segs, image.data(), image.size(), hipMemcpyHostToDevice);
      h->d_seg_work = reinterpret_cast<uint32_t*>(h->d_segs + n);
    }
    if (e == hipSuccess && h->mapped) {
      const std::vector<uint8_t> map = build_map(h);
      e = hipMalloc((void**)&h->d_map, map.size());
      if (e == hipSuccess) e = hipMemcpy(h->d_map, map.data(), map.size(), hipMemcpyHostToDevice);
    }
    if (e == hipSuccess && (cfg->n_rows > (uint32_t)kInlineRows || cfg->n_cols > (uint32_t)kInlineRows))
      e = hipMalloc((void**)&h->d_tables, 2 * DADAM_BINDINGS_KEPT * sizeof(BoundTables));
    if (e == hipSuccess) e = hipMalloc((void**)&h->d_partials, kConsensusPartials * sizeof(double));
    if (e == hipSuccess) {
      const std::vector<double> zeros(kConsensusPartials, 0.0);
      e = hipMemcpy(h->d_partials, zeros.data(), kConsensusPartials * sizeof(double), hipMemcpyHostToDevice);
    }
    // the array in the device image: its address on THIS device (the guard has made it current)
    if (e == hipSuccess) e = (hipError_t)static_partials(&h->d_static_partials, &h->static_capacity);
    if (e != hipSuccess) {
      if (h->d_segs) (void)hipFree(h->d_segs);
      if (h->d_map) (void)hipFree(h->d_map);
      if (h->d_partials) (void)hipFree(h->d_partials);
      if (h->d_tables) (void)hipFree(h->d_tables);
      delete h;
      return fail(nullptr, DADAM_EHIP, "device set-up failed: %s", hipGetErrorString(e));
    }
  }
  *out = h;
  return DADAM_OK;
}

int dadam_set_topology(dadam_handle* h, uint32_t slot_id, const int32_t* row_ptr, const int32_t* col_idx,
                       const float* w, uint32_t* warn) {
  if (!h) return DADAM_EINVAL;
  if (warn) *warn = 0;
  if (slot_id >= DADAM_MAX_SLOTS) return fail(h, DADAM_EINVAL, "slot %u out of range", slot_id);
  if (!row_ptr || !col_idx || !w) return fail(h, DADAM_EINVAL, "null neighbour list");
  const uint32_t R = h->cfg.n_rows, C = h->cfg.n_cols;
  if (row_ptr[0] != 0) return fail(h, DADAM_ETOPO, "row_ptr[0] must be 0");
  for (uint32_t i = 0; i < R; ++i) {
    if (row_ptr[i + 1] <= row_ptr[i]) return fail(h, DADAM_ETOPO, "row %u is empty or row_ptr decreases", i);
    if ((uint32_t)(row_ptr[i + 1] - row_ptr[i]) > C) return fail(h, DADAM_ETOPO, "row %u has more entries than sources", i);
  }
  const int32_t nnz = row_ptr[R];
  std::vector<double> colsum(C, 0.0);
  std::vector<int32_t> sole(C, -1);
  bool reuse = false;
  for (uint32_t i = 0; i < R; ++i) {
    double sum = 0.0;
    std::vector<char> seen(C, 0);
    for (int32_t k = row_ptr[i]; k < row_ptr[i + 1]; ++k) {
      int32_t c = col_idx[k];
      if (c < 0 || (uint32_t)c >= C) return fail(h, DADAM_ETOPO, "row %u: column %d out of range", i, c);
      if (seen[c]) return fail(h, DADAM_ETOPO, "row %u lists source %d twice", i, c);
      seen[c] = 1;
      if (!(w[k] > 0.f) || !std::isfinite(w[k])) return fail(h, DADAM_ETOPO, "row %u: weight %d is not finite and positive", i, k);
      sum += (double)w[k];
      colsum[c] += (double)w[k];
      if (sole[c] == -1) sole[c] = (int32_t)i; else { sole[c] = -2; reuse = true; }
    }
    if (std::fabs(sum - 1.0) > 1e-5) return fail(h, DADAM_ETOPO, "row %u sums to %.9g, not 1", i, sum);
  }
  if (R == C && warn)
    for (uint32_t c = 0; c < C; ++c)
      if (std::fabs(colsum[c] - 1.0) > 1e-5) *warn |= DADAM_WARN_NOT_COLUMN_STOCHASTIC;

  Slot fresh;
  fresh.set = true;
  fresh.row_ptr.assign(row_ptr, row_ptr + R + 1);
  fresh.col.assign(col_idx, col_idx + nnz);
  fresh.w.assign(w, w + nnz);
  fresh.reuse = reuse;
  fresh.sole_reader = sole;
  for (uint32_t c = 0; c < C; ++c) fresh.n_read += sole[c] != -1 ? 1 : 0;
  for (uint32_t i = 0; i < R; ++i) fresh.max_degree = std::max(fresh.max_degree, row_ptr[i + 1] - row_ptr[i]);
  if (reuse) fresh.order = sharing_order(R, C, row_ptr, col_idx);
  std::vector<int32_t> loop_col, loop_rows;
  std::vector<float> loop_w;
  find_loops(R, C, fresh, loop_col, loop_w, loop_rows);
  if (h->cfg.device != DADAM_DEVICE_NONE) {
    DeviceGuard guard(h->cfg.device);
    hipError_t e = guard.err;
    if (e == hipSuccess) e = upload_lists(h, fresh, loop_col, loop_w, loop_rows);
    if (e != hipSuccess) {
      free_slot(fresh);
      return fail(h, DADAM_EHIP, "uploading the neighbour list failed: %s", hipGetErrorString(e));
    }
  }
  if (h->cfg.device != DADAM_DEVICE_NONE) {
    DeviceGuard guard(h->cfg.device);
    free_slot(h->slots[slot_id]);
  }
  h->slots[slot_id] = fresh;
  return DADAM_OK;
}

int dadam_bind(dadam_handle* h, const dadam_buffers* b) {
  if (!h) return DADAM_EINVAL;
  if (!b || !b->x_src || !b->x_dst || !b->m_hat || !b->v_hat) return fail(h, DADAM_EINVAL, "null buffer table");
  const uint32_t R = h->cfg.n_rows, C = h->cfg.n_cols;
  if (!b->acc && h->cfg.accum_s > 1) return fail(h, DADAM_EINVAL, "acc table is null but accum_s > 1");
  const size_t xb = h->cfg.d * dtype_bytes(h->cfg.param_dtype);
  const size_t sb = h->cfg.d * 4;
  std::vector<Interval> iv;
  for (uint32_t c = 0; c < C; ++c) {
    if (!b->x_src[c]) return fail(h, DADAM_EINVAL, "x_src[%u] is null", c);
    if (!aligned16(b->x_src[c])) return fail(h, DADAM_EALIGN, "x_src[%u] is not 16-byte aligned", c);
    iv.push_back({(uintptr_t)b->x_src[c], (uintptr_t)b->x_src[c] + xb, 0, (int)c});
  }
  for (uint32_t i = 0; i < R; ++i) {
    const void* ps[4] = {b->x_dst[i], b->m_hat[i], b->v_hat[i], b->acc ? b->acc[i] : nullptr};
    const char* names[4] = {"x_dst", "m_hat", "v_hat", "acc"};
    for (int q = 0; q < 4; ++q) {
      if (!ps[q]) {
        if (q == 3 && h->cfg.accum_s == 1) continue;
        return fail(h, DADAM_EINVAL, "%s[%u] is null", names[q], i);
      }
      if (!aligned16(ps[q])) return fail(h, DADAM_EALIGN, "%s[%u] is not 16-byte aligned", names[q], i);
      iv.push_back({(uintptr_t)ps[q], (uintptr_t)ps[q] + (q == 0 ? xb : sb), q == 0 ? 1 : 2, (int)i});
    }
  }
  std::vector<int32_t> inplace[kMaxRows];
  for (size_t p = 0; p < iv.size(); ++p)
    for (size_t q = p + 1; q < iv.size(); ++q) {
      const Interval& a = iv[p];
      const Interval& c = iv[q];
      if (!overlaps(a, c)) continue;
      if (a.kind == 0 && c.kind == 0) continue;  // two read-only sources may coincide
      if (a.kind == 0 && c.kind == 1 && a.lo == c.lo) {  // update in place
        inplace[c.index].push_back(a.index);
        continue;
      }
      return fail(h, DADAM_EALIAS, "buffers overlap: kind %d index %d and kind %d index %d (0 x_src, 1 x_dst, 2 state)",
                  a.kind, a.index, c.kind, c.index);
    }
  if (h->d_tables) {
    // The tables do not fit the kernel arguments: two immutable device copies for this binding (as bound,
    // and as dadam_swap_x would leave it), in the ring slot after the current one, so that launches in
    // flight keep reading the copies they were given.
    std::vector<BoundTables> t(2);
    memset(t.data(), 0, 2 * sizeof(BoundTables));
    for (int v = 0; v < 2; ++v) {
      for (uint32_t c = 0; c < C; ++c) t[v].x_src[c] = (uint64_t)(uintptr_t)b->x_src[c];
      for (uint32_t i = 0; i < R; ++i) {
        t[v].x_dst[i] = (uint64_t)(uintptr_t)b->x_dst[i];
        t[v].m_hat[i] = (uint64_t)(uintptr_t)b->m_hat[i];
        t[v].v_hat[i] = (uint64_t)(uintptr_t)b->v_hat[i];
        t[v].acc[i] = b->acc ? (uint64_t)(uintptr_t)b->acc[i] : 0;
      }
    }
    if (R == C)
      for (uint32_t i = 0; i < R; ++i)
        if (inplace[i].empty()) {  // what dadam_swap_x does
          t[1].x_src[i] = (uint64_t)(uintptr_t)b->x_dst[i];
          t[1].x_dst[i] = (uint64_t)(uintptr_t)b->x_src[i];
        }
    const uint32_t next = h->bound ? (h->binding + 1) % DADAM_BINDINGS_KEPT : h->binding;
    DeviceGuard guard(h->cfg.device);
    hipError_t e = guard.err;
    if (e == hipSuccess) e = hipMemcpy(h->d_tables + 2 * next, t.data(), 2 * sizeof(BoundTables), hipMemcpyHostToDevice);
    if (e != hipSuccess) return fail(h, DADAM_EHIP, "copying the pointer tables to the device failed: %s", hipGetErrorString(e));
    h->binding = next;
  }
  h->swapped = false;
  for (uint32_t c = 0; c < C; ++c) h->x_src[c] = b->x_src[c];
  for (uint32_t i = 0; i < R; ++i) {
    h->x_dst[i] = b->x_dst[i];
    h->m_hat[i] = b->m_hat[i];
    h->v_hat[i] = b->v_hat[i];
    h->acc[i] = b->acc ? b->acc[i] : nullptr;
    h->inplace_cols[i] = inplace[i];
  }
  h->bound = true;
  h->outputs_gen = (h->outputs_gen | 1u) + 1u;
  return DADAM_OK;
}

int dadam_swap_x(dadam_handle* h) {
  if (!h) return DADAM_EINVAL;
  if (!h->bound) return fail(h, DADAM_ESTATE, "no buffers bound");
  if (h->cfg.n_rows != h->cfg.n_cols) return fail(h, DADAM_ESTATE, "swap needs n_rows == n_cols");
  for (uint32_t i = 0; i < h->cfg.n_rows; ++i) {
    if (!h->inplace_cols[i].empty()) continue;  // in-place rows stay as they are
    void* s = const_cast<void*>(h->x_src[i]);
    h->x_src[i] = h->x_dst[i];
    h->x_dst[i] = s;
  }
  h->outputs_gen ^= 1u;
  h->swapped = !h->swapped;
  return DADAM_OK;
}

int dadam_gossip_step(dadam_handle* h, uint32_t slot, const void* const* grads, uint64_t t, uint32_t flags,
                      void* hip_stream) {
  return step_impl(h, slot, grads, t, flags, true, 0, 0, false, hip_stream);
}

int dadam_gossip_step_range(dadam_handle* h, uint32_t slot, const void* const* grads, uint64_t t,
                            uint32_t flags, uint32_t tensor_begin, uint32_t tensor_end, void* hip_stream) {
  return step_impl(h, slot, grads, t, flags, false, tensor_begin, tensor_end, false, hip_stream);
}

int dadam_mix(dadam_handle* h, uint32_t slot, uint32_t flags, void* hip_stream) {
  if (h && (flags & DADAM_FUSE_ACCUM)) return fail(h, DADAM_EINVAL, "dadam_mix takes only the FORCE flags");
  return step_impl(h, slot, nullptr, 1, flags, true, 0, 0, true, hip_stream);
}

int dadam_mix_consensus(dadam_handle* h, uint32_t slot, uint32_t flags, double* consensus_out, void* hip_stream) {
  if (!h) return DADAM_EINVAL;
  if (flags & DADAM_FUSE_ACCUM) return fail(h, DADAM_EINVAL, "dadam_mix_consensus takes only the FORCE flags");
  if (!consensus_out || (reinterpret_cast<uintptr_t>(consensus_out) & 7u))
    return fail(h, DADAM_EINVAL, "consensus_out must be a non-null, 8-byte aligned device pointer");
  return step_impl(h, slot, nullptr, 1, flags, true, 0, 0, true, hip_stream, consensus_out);
}

int dadam_mix_consensus_static(dadam_handle* h, uint32_t slot, uint32_t flags, double* consensus_out, void* hip_stream) {
  if (!h) return DADAM_EINVAL;
  if (flags & DADAM_FUSE_ACCUM) return fail(h, DADAM_EINVAL, "dadam_mix_consensus_static takes only the FORCE flags");
  if (!consensus_out || (reinterpret_cast<uintptr_t>(consensus_out) & 7u))
    return fail(h, DADAM_EINVAL, "consensus_out must be a non-null, 8-byte aligned device pointer");
  if (h->cfg.device != DADAM_DEVICE_NONE) {
    if (!h->d_static_partials) return fail(h, DADAM_ESTATE, "the static scratch array was not resolved on this device");
    if (kConsensusPartials > h->static_capacity)
      return fail(h, DADAM_EINVAL, "the pass needs %u partial sums, the static scratch array holds %u (DADAM_STATIC_SCRATCH_BYTES = %u)",
                  kConsensusPartials, h->static_capacity, DADAM_STATIC_SCRATCH_BYTES);
  }
  return step_impl(h, slot, nullptr, 1, flags, true, 0, 0, true, hip_stream, consensus_out, h->d_static_partials);
}

int dadam_accumulate(dadam_handle* h, const void* const* grads, uint64_t t, void* hip_stream) {
  if (!h) return DADAM_EINVAL;
  int rc = check_bound(h);
  if (rc) return rc;
  if (t == 0) return fail(h, DADAM_EINVAL, "iterations are numbered from 1");
  rc = check_grads(h, grads);
  if (rc) return rc;
  if (h->cfg.accum_s > 1)
    for (uint32_t i = 0; i < h->cfg.n_rows; ++i)
      if (!h->acc[i]) return fail(h, DADAM_ESTATE, "accumulator of row %u is not bound", i);
  rc = check_device(h);
  if (rc) return rc;
  if (h->segs.empty()) return DADAM_OK;
  StepArgs a;
  fill_args(h, h->mapped, grads, &a);
  uint32_t w0 = 0, w1 = 0;
  work_range(h, h->mapped, kGridDirect, 0, (uint32_t)h->segs.size() - 1, h->segs.front().lo, h->segs.back().hi, &w0, &w1);
  set_range(h, h->mapped, false, kGridDirect, w0, h->segs.front().lo, h->segs.back().hi, &a);
  a.wide_search = (uint64_t)(w1 - w0) * kDirectItem * h->cfg.n_rows <= kWideSearchWaves ? 1u : 0u;
  fill_scalars(h, t, &a.s);
  DeviceGuard guard(h->cfg.device);
  if (guard.err != hipSuccess) return fail(h, DADAM_EHIP, "hipSetDevice: %s", hipGetErrorString(guard.err));
  const bool whole_items = accumulate_whole_items(h, (uint64_t)(w1 - w0) * h->direct_elems * h->cfg.n_rows);
  // Rows share nothing here, but with many of them a die that walks run after run row by row has few arrays in use at a time.  us of a
  // loop of four, one row of a piece after the other / runs, 5e8 elements: float32 4 rows 4790 / 5136, 8 rows 4752 / 4984, 16 rows 4712 / 4853,
  // 24 rows 4649 / 4773, 32 rows 4869 / 4901, 40 rows 4581 / 4606 (2e9 elements 4 rows 18602 / 19346, 16 rows 19031 / 19612, 32 rows 19324 / 19491, but with arrays that lie badly 11040 / 10966 of a whole loop);
  // bfloat16 8 rows 4092 / 4096, 16 rows 4048 / 3984, 24 rows 4013 / 3979, 32 rows 4167 / 4034.  Where the arrays lie badly runs gain more (fraction of
  // 8 TB/s, 40 rows 0.61 / 0.81, 64 rows 0.67 / 0.81, 100 rows 0.63 / 0.80, bfloat16 parameters 24 rows 0.66 / 0.73, 128 rows 0.56 / 0.75).
  if (h->nontemporal && !h->short_segments && h->cfg.n_rows >= (h->vec == 8 ? 16u : 32u)) {
    a.order = kOrderDieBlocks;
    set_die_run(whole_items ? kDieRunPieces / kDirectItem : kDieRunPieces, &a);
  }
  int e = launch_accumulate((int)h->cfg.grad_dtype, fused_phase(h, t), h->nontemporal, whole_items, a, w1 - w0, hip_stream, h->vec);
  if (e != (int)hipSuccess)
    return fail(h, DADAM_EHIP, "kernel launch failed: %s", hipGetErrorString((hipError_t)e));
  return DADAM_OK;
}

int dadam_set_lr(dadam_handle* h, float lr) {
  if (!h) return DADAM_EINVAL;
  if (!std::isfinite(lr)) return fail(h, DADAM_EINVAL, "lr is not finite");
  h->lr = lr;
  return DADAM_OK;
}

int dadam_get_plan_info(const dadam_handle* h, dadam_plan_info* out) {
  if (!h || !out) return DADAM_EINVAL;
  out->n_segments = (uint32_t)h->segs.size();
  out->tile_elems = h->tile_elems;
  out->direct_elems = h->direct_elems;
  out->n_tiles_tile = h->n_work_t;
  out->n_tiles_direct = h->n_work_d;
  out->lds_bytes_tile = h->lds_bytes;
  out->tile_mode_possible = h->tile_possible ? 1u : 0u;
  out->lds_limit_bytes = h->lds_limit;
  out->n_xcds = h->n_xcds;
  out->mix_tile_elems = h->mix_tile_elems;
  out->lds_bytes_mix = h->mix_lds_bytes;
  out->n_tiles_mix = h->n_work_m;
  out->tile_waves = (uint32_t)h->shape.waves;
  out->tile_vectors = (uint32_t)h->shape.ut;
  out->mix_waves = (uint32_t)h->mix_shape.waves;
  out->mix_vectors = (uint32_t)h->mix_shape.ut;
  out->streaming = h->nontemporal ? 1u : 0u;
  return DADAM_OK;
}

int dadam_slot_uses_tile_mode(const dadam_handle* h, uint32_t slot) {
  if (!h) return DADAM_EINVAL;
  if (slot >= DADAM_MAX_SLOTS || !h->slots[slot].set) return fail(h, DADAM_ESTATE, "topology slot %u is not set", slot);
  bool tile = false;
  int rc = choose_mode(h, h->slots[slot], 0, h->decays, &tile);
  if (rc) return rc;
  return tile ? 1 : 0;
}

int dadam_get_row_order(const dadam_handle* h, uint32_t slot, int32_t* order_out) {
  if (!h || !order_out) return DADAM_EINVAL;
  if (slot >= DADAM_MAX_SLOTS || !h->slots[slot].set) return fail(h, DADAM_ESTATE, "topology slot %u is not set", slot);
  const Slot& s = h->slots[slot];
  const uint32_t R = h->cfg.n_rows;
  const bool used = !s.order.empty() && h->n_xcds > 1;
  for (uint32_t i = 0; i < R; ++i) order_out[i] = used ? s.order[i] : (int32_t)i;
  return used ? 1 : 0;
}

int dadam_pack_offsets(const uint64_t* numel, uint32_t n, uint32_t align_elems, uint64_t* offsets, uint64_t* d_out) {
  if (!numel || !offsets || !d_out || align_elems == 0) return DADAM_EINVAL;
  uint64_t cur = 0;
  for (uint32_t k = 0; k < n; ++k) {
    offsets[k] = cur;
    cur += (numel[k] + align_elems - 1) / align_elems * align_elems;
  }
  *d_out = cur;
  return DADAM_OK;
}

int dadam_spread_offsets(const uint64_t* nbytes, uint32_t n, uint64_t arena_bytes, uint64_t* offsets) {
  if (!nbytes || !offsets || n == 0) return DADAM_EINVAL;
  const uint64_t unit = 2ull << 20;
  uint64_t packed = 0;
  for (uint32_t k = 0; k < n; ++k) {
    if (nbytes[k] > (1ull << 46)) return DADAM_EINVAL;
    packed += (nbytes[k] + unit - 1) / unit * unit;
  }
  if (packed > arena_bytes + (((nbytes[n - 1] + unit - 1) / unit * unit) - nbytes[n - 1])) return DADAM_EINVAL;
  const uint64_t slack = arena_bytes > packed ? arena_bytes - packed : 0;
  const uint64_t gap = n > 1 ? slack / (n - 1) / unit * unit : 0;
  uint64_t cur = 0;
  for (uint32_t k = 0; k < n; ++k) {
    offsets[k] = cur;
    cur += (nbytes[k] + unit - 1) / unit * unit + gap;
  }
  return DADAM_OK;
}

int dadam_deal_offsets(const uint64_t* nbytes, uint32_t n, uint64_t lo0, uint64_t hi0, uint64_t lo1, uint64_t hi1,
                       uint32_t every, uint64_t* offsets) {
  if (!nbytes || !offsets || n == 0 || every < 2 || every > 8) return DADAM_EINVAL;
  const uint64_t unit = 2ull << 20;
  const uint64_t lo[2] = {lo0, lo1}, hi[2] = {hi0, hi1};
  for (int r = 0; r < 2; ++r)
    if (lo[r] % unit || hi[r] % unit || lo[r] > hi[r] || hi[r] > (1ull << 50)) return DADAM_EINVAL;
  if (lo0 < hi1 && lo1 < hi0 && lo0 != hi0 && lo1 != hi1) return DADAM_EINVAL;  // the regions overlap
  std::vector<uint64_t> side[2];
  std::vector<uint32_t> number[2];  // which buffers a side holds
  for (uint32_t k = 0; k < n; ++k) {
    if (nbytes[k] > (1ull << 46)) return DADAM_EINVAL;
    const int r = k % every == every - 1 ? 1 : 0;
    side[r].push_back(nbytes[k]);
    number[r].push_back(k);
  }
  for (int r = 0; r < 2; ++r) {
    if (side[r].empty()) continue;
    std::vector<uint64_t> off(side[r].size());
    const int rc = dadam_spread_offsets(side[r].data(), (uint32_t)side[r].size(), hi[r] - lo[r], off.data());
    if (rc != DADAM_OK) return rc;
    // Stagger the buffers inside their gaps by a fixed pseudo-random number of 2 MiB steps, so that their
    // bases do not form an arithmetic progression: for some distances (660 MiB, 884 MiB between 476 MiB
    // buffers) a progression costs 3-4 % of bandwidth, staggered bases never did.  A buffer moves forward
    // by less than the gap behind it; the last one stays where it is.
    for (size_t j = 0; j + 1 < off.size(); ++j) {
      const uint64_t end = off[j] + (side[r][j] + unit - 1) / unit * unit;
      const uint64_t slots = off[j + 1] > end ? (off[j + 1] - end) / unit : 0;
      uint64_t z = ((uint64_t)j + 1) * 0x9E3779B97F4A7C15ull;  // a fixed 64-bit mix of the buffer's number
      z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
      z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
      z ^= z >> 31;
      if (slots > 1) off[j] += z % slots * unit;
    }
    for (size_t j = 0; j < off.size(); ++j) offsets[number[r][j]] = lo[r] + off[j];
  }
  return DADAM_OK;
}

int dadam_place_offsets(const uint64_t* nbytes, uint32_t n, uint64_t arena_bytes, uint64_t device_total_bytes,
                        uint64_t* offsets, uint64_t* regions_out, uint32_t* advice_out) {
  if (!nbytes || !offsets || n == 0) return DADAM_EINVAL;
  const uint64_t unit = 2ull << 20, gib = 1ull << 30;
  std::vector<uint64_t> side[2];
  uint64_t need[2] = {0, 0};
  for (uint32_t k = 0; k < n; ++k) {
    if (nbytes[k] > (1ull << 46)) return DADAM_EINVAL;
    side[k & 1].push_back(nbytes[k]);
    need[k & 1] += (nbytes[k] + unit - 1) / unit * unit;
  }
  if (arena_bytes > (1ull << 50) || device_total_bytes > (1ull << 50)) return DADAM_EINVAL;
  const uint64_t third = (device_total_bytes + 3 * gib / 2) / (3 * gib) * gib;  // a third, to the nearest GiB
  const uint64_t margin = 2 * gib;
  // Region 0 ends `margin` below the boundary between the first two thirds, region 1 starts `margin`
  // above it and ends no later than `margin` below the next boundary (or where the arena ends).
  const uint64_t top = arena_bytes < 2 * third - margin ? arena_bytes : 2 * third - margin;
  uint32_t advice = 0;
  uint64_t lo[2] = {0, 0}, width[2] = {0, 0};
  if (n < 2 || third <= 2 * margin) {
    advice = 0;  // nothing to deal over two sides
  } else if (arena_bytes + 16 * gib < device_total_bytes) {
    advice = DADAM_PLACE_ARENA_ELSEWHERE;
  } else if (need[0] > third - margin || third + margin + need[1] > top) {
    advice = DADAM_PLACE_TOO_LARGE;
  } else {
    for (int r = 0; r < 2; ++r) {
      uint64_t want = (need[r] + need[r] / 5 + unit - 1) / unit * unit;  // 20 % of room for the stagger
      if (want < 64 * gib) want = 64 * gib;
      const uint64_t room = r == 0 ? third - margin : top - (third + margin);
      width[r] = (want < room ? want : room) / unit * unit;  // >= need[r] by the tests above
      lo[r] = r == 0 ? third - margin - width[r] : third + margin;
    }
    advice = DADAM_PLACE_TWO_REGIONS;
  }
  if (advice_out) *advice_out = advice;
  if (advice == DADAM_PLACE_TWO_REGIONS) {
    const int rc = dadam_deal_offsets(nbytes, n, lo[0], lo[0] + width[0], lo[1], lo[1] + width[1], 2, offsets);
    if (rc != DADAM_OK) return rc;
    if (regions_out) {
      regions_out[0] = lo[0]; regions_out[1] = lo[0] + width[0];
      regions_out[2] = lo[1]; regions_out[3] = lo[1] + width[1];
    }
    return DADAM_OK;
  }
  if (regions_out) {
    regions_out[0] = 0; regions_out[1] = arena_bytes;
    regions_out[2] = 0; regions_out[3] = 0;
  }
  return dadam_spread_offsets(nbytes, n, arena_bytes, offsets);
}

const char* dadam_last_error(const dadam_handle* h) { return h ? h->err.c_str() : g_init_error.c_str(); }

void dadam_destroy(dadam_handle* h) {
  if (!h) return;
  if (h->cfg.device != DADAM_DEVICE_NONE) {
    DeviceGuard guard(h->cfg.device);
    for (Slot& s : h->slots) free_slot(s);
    if (h->d_segs) (void)hipFree(h->d_segs);
    if (h->d_map) (void)hipFree(h->d_map);
    if (h->d_partials) (void)hipFree(h->d_partials);
    if (h->d_tables) (void)hipFree(h->d_tables);
  }
  delete h;
}

}  // extern "C"
