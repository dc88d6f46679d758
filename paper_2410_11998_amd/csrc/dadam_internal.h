// Internal interface between the host side of libdadam (validation, planning, launch set-up) and
// the gfx950 kernels.  Nothing in here is part of the public C ABI (see include/dadam.h).
#ifndef DADAM_INTERNAL_H_
#define DADAM_INTERNAL_H_

#include <stdint.h>

#include "dadam.h"

namespace dadam {

constexpr int kMaxRows = DADAM_MAX_ROWS;  // rows / source buffers a handle may have
constexpr int kInlineRows = 64;           // up to this many, every pointer table travels in the kernel arguments
constexpr int kWave = 64;            // gfx950 wavefront
constexpr int kDirectItem = 8;  // direct and accumulate kernels: wavefronts (16-byte vectors per lane) per work item

// Which of the four tile grids a launch walks: the fused step's tiles, the direct/accumulate
// kernels' tiles, the tiles of the mixing-only launch, or tiles of one vector a lane (loop kernel).
enum Grid : uint32_t { kGridTile = 0, kGridDirect = 1, kGridMix = 2, kGridVector = 3, kNumGrids = 4 };

// A maximal run of contiguous tensors with the same hyper-parameters: elements [lo, hi) of every buffer.  Work items are tiles of a
// fixed grid anchored at element 0, so that vector accesses are 16-byte aligned whenever the
// buffers are; a tile that sticks out of [lo, hi) is stored, and at the end of a buffer loaded, element by element.
struct alignas(64) Segment {
  uint64_t lo, hi;
  uint64_t first_tile[kNumGrids];  // per Grid: index of the first tile of that grid that intersects the segment
  float weight_decay;      // decoupled weight decay of the tensors in this segment
};
static_assert(sizeof(Segment) == 64, "a work item finds all of its segment in one line");

// How the workgroups of a direct-kernel launch walk the (piece, row) pairs.
enum Order : uint32_t { kOrderLinear = 0, kOrderDieGroups = 1, kOrderDieBlocks = 2 };

// Scalars of one iteration, computed on the host in double and rounded once.
struct Scalars {
  float beta1, omb1;     // beta1, 1 - beta1
  float beta2, omb2;     // beta2, 1 - beta2
  float betav, ombv;     // decay of v_hat in the fold and its complement
  float inv_c1, inv_c2;  // 1 / (1 - beta1^t_hat), 1 / (1 - beta2^t_hat)
  float eps, lr, inv_s;
};

// What a step does with the optimizer state (Algorithm 3, lines 6-13).
enum Phase : int {
  kMixOnly = 0,     // x_dst = W x_src
  kUpdateOnly = 1,  // lines 6-8 only
  kPlain = 2,       // lines 6-9, inside a loop
  kLoopStart = 3,   // lines 6-9, first iteration of a loop: b is known to be zero and not read
  kFold = 4,        // lines 6-13, last iteration of a loop (s > 1)
  kAlg1 = 5,        // s == 1: Algorithm 1, moments updated every iteration, no accumulator
  kMixConsensus = 6,  // x_dst = W x_src and, on the side, sum_c ||x_src[c] - mean||^2 (tile mode only)
  kNumPhases = 7
};

constexpr uint32_t kConsensusPartials = 1024;  // partial sums the tiles scatter their contributions over
static_assert(kConsensusPartials * sizeof(double) == DADAM_STATIC_SCRATCH_BYTES, "the header states the static scratch size");

// Rows that list the same sources with the same weights.
struct Loop {
  int32_t first_entry, n_entries;  // in StepArgs::col / w
  int32_t first_row, n_rows;       // in StepArgs::row_order
};
constexpr int kMaxLoopWaves = 16;  // wavefronts of a loop kernel's workgroup

// Pointer tables of the bound buffers of a handle with more than kInlineRows rows or sources: they do not
// fit the 4 KB kernel-argument segment and live in device memory, one immutable copy per binding and
// exchange state (see dadam_bind).
// Addresses are held as 64-bit integers on purpose: see the kernels' table helpers.
struct BoundTables {
  uint64_t x_src[kMaxRows];
  uint64_t x_dst[kMaxRows];
  uint64_t m_hat[kMaxRows];
  uint64_t v_hat[kMaxRows];
  uint64_t acc[kMaxRows];
};

// Kernel argument block (passed by value; 3.9 KB of the 4 KB kernarg segment).  The tables of the bound
// buffers are used when `ext` is null (at most kInlineRows rows and sources); otherwise `ext` holds them.
// The gradient pointers change from call to call and always travel here.
// N rows and sources travel in the block's tables, G gradients.
template <int N, int G>
struct StepArgsFor {
  const void* x_src[N];
  void* x_dst[N];
  float* m_hat[N];
  float* v_hat[N];
  float* acc[N];
  const void* grad[G];
  const BoundTables* ext;
  // The slot's neighbour lists (device).  Tile kernel: CSR.  Direct kernel: the lists by position, list_stride
  // entries apart, row_len their lengths and row_order the rows: where rows share sources, positions follow an order
  // in which neighbours share them, so that the rows which read a source run on the die whose L2 already holds it.
  // Loop kernel: the loops' entries, row_order their rows.
  const int32_t* row_ptr;
  const int32_t* row_len;
  const int32_t* col;
  const float* w;
  const int32_t* row_order;
  const Loop* loops;
  uint32_t list_stride;
  uint32_t n_loops;      // > 0: the loop kernel's launch (see launch_tile)
  uint32_t loop_shares;  // workgroups that share the rows of one tile of a loop (see loop_shares)
  uint32_t order;        // Order: how a launch of the row kernel walks pieces and rows
  uint32_t n_pieces;     // pieces of this launch (kOrderDieBlocks)
  uint32_t die_run;      // pieces a die walks row after row (kOrderDieBlocks)
  uint32_t order_group;  // kOrderDieGroups: rows per die, ceil(n_rows / n_xcd); the launch has n_xcd * order_group
                         // workgroups per tile, of which those beyond a die's share of the rows have nothing to do
  uint32_t reserve_lds;  // direct kernels: LDS a workgroup reserves (see bounded_occupancy_lds)
  // Device, null where the launch walks segments: a byte for every four elements of the packed vector, kept by layouts of
  // short segments side by side (see build_map).  Bits 0 to 3: which of them belong to a tensor; bit 4: they decay.
  const uint8_t* map;
  const Segment* seg;        // device
  const uint32_t* seg_work;  // device: per Grid, the first work item of every segment (tiles; per row in direct mode)
  uint32_t wide_search;      // small launch: all lanes search the segments (see locate)
  uint64_t first_tile;       // one segment: its first tile of this launch's grid ...
  float weight_decay;        // ... and its decay
  uint32_t n_seg;
  uint32_t n_rows, n_cols;
  uint32_t grid;        // Grid: which tile numbering work items refer to
  uint32_t work_begin;  // first work item (in tiles) of this launch
  uint32_t n_xcd;       // dies that consecutive workgroup ids are dealt over (tile order)
  uint32_t xcd_block;   // tile mode: tiles per block; blocks go to the dies in turn (0: one contiguous share each)
  uint64_t d;                 // elements of a buffer (0: cut tiles load element by element, see cut_by_elements)
  uint64_t clip_lo, clip_hi;  // element range of this launch (whole layout or a tensor range)
  double* partials;           // kConsensusPartials doubles (device), used by kMixConsensus only
  Scalars s;
};

using StepArgs = StepArgsFor<kInlineRows, kMaxRows>;
// The block of handles with few rows and sources whose launches are small: the runtime copies it to the device on every
// launch, which for 4 KB takes 1.1 us longer than for 1 KB (of 5.5 us a call through the binding).
constexpr int kFewRows = 16;
using StepArgsFew = StepArgsFor<kFewRows, kFewRows>;

static_assert(sizeof(StepArgs) <= 4096, "the argument block of a launch holds 4 KB");

constexpr uint32_t kDieBlockTiles = 32;  // measured, see k_tile
constexpr uint32_t kLongSegment = 65536;  // elements of two blocks of spread lanes; measured, see dadam_handle::short_segments
constexpr uint64_t kSegmentElems = 80000000;  // elements of all rows of a launch; measured, see segments_are_faster
constexpr uint64_t kMostMapped = 1ull << 28, kWidestGap = 7;  // elements; see can_map
constexpr uint64_t kStreamedBytes = 344ull << 20;  // measured, see few_rows_stream
constexpr uint32_t kDieRunPieces = 256;  // large direct launches in die blocks; measured, see rows_stay_on_one_die
constexpr uint32_t kDieBlockMix = 256, kDieBlockLoops = 2;  // streaming launches; measured, see k_tile, k_loop
constexpr uint32_t kFewTiles = 256;      // compute units of the chip; measured, see few_tiles_limit, loop_kernel_waves
constexpr uint32_t kLongLaunch = 2048;   // tiles; measured, see loop_shares
constexpr uint32_t kManyTiles = 1024, kManyStreamed = 640;  // measured, see rows_stay_on_one_die, many_tiles
constexpr uint64_t kManyElems = 100000000;  // elements of all rows of a launch; measured, see there, whole_items, accumulate_whole_items
constexpr uint64_t kPairElems = 13000000;   // the same, of launches that do not stream; measured, see rows_stay_on_one_die
constexpr uint32_t kWideSearchWaves = 16384;  // up to two rounds of wavefronts on the chip; see locate
constexpr uint32_t kBoundedPieces = 65536, kInFlightBytes = 90 * 1024;  // measured, see bounded_occupancy_lds
constexpr uint32_t kLdsPerUnit = 160 * 1024, kLdsGranule = 1280;        // LDS of a compute unit; it is given out in granules

typedef const void* KernelFn;  // address of a kernel taking a StepArgs, or a StepArgsFew where the name says so

struct TileShape {
  int waves;  // wavefronts per workgroup (rows are dealt round-robin to them)
  int ut;     // 16-byte vectors per lane and row
  bool nontemporal;  // streaming hint on every full-vector global access
};

// The pass that the placement probe times: float32 streams of it, elements of a stream to a workgroup.
constexpr uint32_t kProbeStreams = 16, kProbeTile = 512;

// Launchers.  All of them enqueue on `stream` and return the hipError_t of the launch as int.
// xdt / gdt are DADAM_F32 | DADAM_BF16.  n_work is the number of tiles in this launch.
// launch_tile with a.n_loops > 0 launches the loop kernel, shape.waves wavefronts a workgroup.
int launch_tile(int xdt, int gdt, Phase phase, TileShape shape, const StepArgs& a, uint32_t n_work,
                uint32_t lds_bytes, void* stream);
// shared: rows share sources; a streaming launch then keeps the hint off the source loads.
// whole_items: one workgroup of four wavefronts takes a work item instead of eight of one (see k_rows).
int launch_direct(int xdt, int gdt, Phase phase, bool nontemporal, bool shared, bool whole_items, const StepArgs& a,
                  uint32_t n_work_tiles, void* stream);
// vec = elements per direct-mode parameter vector of the handle (fixes the tile grid).
int launch_accumulate(int gdt, Phase phase, bool nontemporal, bool whole_items, const StepArgs& a, uint32_t n_work_tiles,
                      void* stream, int vec);

// Consensus error: clear the partial sums / add them up in a fixed order into *out (device) and clear them.
int launch_consensus_zero(double* partials, void* stream);
int launch_consensus_sum(double* partials, double* out, void* stream);

// The placement probe's pass: dst[k] = src[k] for kProbeStreams streams of `elems` (a multiple of kProbeTile) float32 elements.
int launch_probe(const void* const* src, void* const* dst, uint64_t elems, uint32_t n_xcd, void* stream);

// The partial-sum array that lives in the library's device image (no allocation): its address on the
// current device and its capacity in doubles.  Returns a hipError_t as int.
int static_partials(double** out, uint32_t* capacity);

// Geometry the host planner needs.
int vec_elems(int xdt);              // elements per 16-byte parameter vector: 4 (f32) or 8 (bf16)
bool tile_shape_supported(TileShape s);

}  // namespace dadam

#endif  // DADAM_INTERNAL_H_
