// Launchers of the gfx950 kernels, the accumulate-only and consensus kernels, and the scratch array of the
// entry point that does not allocate.  The tile and direct kernels are compiled in parts
// (dadam_kernels_part.hip, once per pair of element types and streaming hint) from dadam_device.h.
#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstring>
#include <map>
#include <mutex>
#include <utility>

#include "dadam_device.h"

// Scratch memory of the entry point that may not allocate (dadam_mix_consensus_static): the partial sums
// of the consensus error, in the library's own image instead of a hipMalloc'ed buffer.  Every GPU the
// library runs on holds its own copy at its own address; host code never uses this name as an
// address, only what hipGetSymbolAddress returned for the current device (static_partials below).
// The compiler makes a static device variable visible to the runtime only once it has seen host code
// refer to it, at the end of the translation unit: nothing may force it out earlier (no `used`
// attribute), or the symbol stays local to the code object and the look-up by name aborts.
static __device__ __align__(256) double scratch[dadam::kConsensusPartials];

namespace dadam {

// what the parts define
#define DADAM_PART(name)                                       \
  KernelFn tile_kernel_##name(int phase, TileShape s, bool map);         \
  KernelFn direct_kernel_##name(int phase, bool shared, bool map);       \
  KernelFn rows_kernel_##name(int phase, bool map);                      \
  KernelFn rows_kernel_##name##_ext(int phase, bool map);                \
  KernelFn loop_kernel_##name(int phase, bool shared, bool map);         \
  KernelFn loop_kernel_##name##_ext(int phase, bool shared, bool map);   \
  KernelFn tile_kernel_##name##_ext(int phase, TileShape s, bool map);   \
  KernelFn direct_kernel_##name##_ext(int phase, bool shared, bool map)
DADAM_PART(f32_f32_nt);
DADAM_PART(f32_f32);
DADAM_PART(bf16_bf16_nt);
DADAM_PART(bf16_bf16);
DADAM_PART(bf16_f32_nt);
DADAM_PART(bf16_f32);
DADAM_PART(f32_bf16_nt);
DADAM_PART(f32_bf16);
#undef DADAM_PART
#define DADAM_PART(name)                                   \
  KernelFn tile_kernel_##name##_few(int phase, TileShape s, bool map); \
  KernelFn direct_kernel_##name##_few(int phase, bool map)
DADAM_PART(f32_f32);
DADAM_PART(bf16_bf16);
DADAM_PART(bf16_f32);
DADAM_PART(f32_bf16);
#undef DADAM_PART

namespace {

// ---------------------------------------------------------------------------------------------
// consensus error: partial sums are cleared by a kernel (not a memset, so that the sequence can be
// captured in a graph) and added up and cleared again by one workgroup in a fixed order
// ---------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_consensus_zero(double* partials) {
  for (uint32_t i = threadIdx.x; i < kConsensusPartials; i += 256) partials[i] = 0.0;
}

// Leaves the partial sums cleared: the next pass over the same array needs no launch to clear them (a launch in
// sequence costs 4.6 us, 3 % of a pass over 16 sources of 25 MB).  Bound by its latency: the sums of a wavefront meet
// in lane exchanges, one barrier in all (4.7 us with a tree of eight barriers).
__global__ __launch_bounds__(256) void k_consensus_sum(double* partials, double* out) {
  __shared__ double red[256 / kWave];
  static_assert(kConsensusPartials == 4 * 256, "four partial sums a thread");
  double p[4], s = 0.0;
#pragma unroll
  for (int k = 0; k < 4; ++k) p[k] = partials[threadIdx.x + k * 256];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    partials[threadIdx.x + k * 256] = 0.0;
    s += p[k];
  }
#pragma unroll
  for (int off = kWave / 2; off > 0; off >>= 1) s += __shfl_xor(s, off);
  if ((threadIdx.x & (kWave - 1)) == 0) red[threadIdx.x / kWave] = s;
  __syncthreads();
  if (threadIdx.x == 0) {
    s = (red[0] + red[1]) + (red[2] + red[3]);
    out[0] = s < 0.0 ? 0.0 : s;
  }
}

// ---------------------------------------------------------------------------------------------
// the pass that the placement probe times: sixteen streams in, sixteen out
// ---------------------------------------------------------------------------------------------
// Two contiguous kilobytes of every stream to a workgroup of four wavefronts, all of them read before any is written.  Bound by
// HBM, and with lanes side by side by where the arrays lie: 0.81 of 8 TB/s across two thirds of the memory, 0.72-0.75 inside
// one.  (Mixing passes of the library spread their lanes, see lane_start, and run alike everywhere: timed in place of
// this one they show no thirds.  LDS reserved to hold fewer workgroups a unit brings the two levels closer, 0.815 / 0.75 with 53 KB.)
struct ProbeArgs {
  const float* src[kProbeStreams];
  float* dst[kProbeStreams];
  uint32_t n_xcd;
};
__global__ __launch_bounds__(256) void k_probe(const ProbeArgs a) {
  const uint32_t lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t tile = die_block_order(blockIdx.x, gridDim.x, a.n_xcd, kDieBlockTiles);
  const uint64_t e = (uint64_t)tile * kProbeTile + 4 * lane;
  f4 v[kProbeStreams / 4][2];
#pragma unroll
  for (uint32_t k = 0; k < kProbeStreams / 4; ++k)
#pragma unroll
    for (uint32_t u = 0; u < 2; ++u) v[k][u] = vload<true>(reinterpret_cast<const f4*>(a.src[4 * k + wave] + e + u * 4 * kWave));
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < kProbeStreams / 4; ++k)
#pragma unroll
    for (uint32_t u = 0; u < 2; ++u) vstore<true>(reinterpret_cast<f4*>(a.dst[4 * k + wave] + e + u * 4 * kWave), v[k][u]);
}

// ---------------------------------------------------------------------------------------------
// dispatch tables
// ---------------------------------------------------------------------------------------------
template <typename GT, int VEC, bool NT, bool EXT>
KernelFn acc_kernel_for_phase(int phase, bool map) {
  switch (phase) {
    case kPlain: return map ? (KernelFn)k_acc_map<GT, VEC, kPlain, NT, EXT> : (KernelFn)k_acc<GT, VEC, kPlain, NT, EXT>;
    case kLoopStart: return map ? (KernelFn)k_acc_map<GT, VEC, kLoopStart, NT, EXT> : (KernelFn)k_acc<GT, VEC, kLoopStart, NT, EXT>;
    case kFold: return map ? (KernelFn)k_acc_map<GT, VEC, kFold, NT, EXT> : (KernelFn)k_acc<GT, VEC, kFold, NT, EXT>;
    case kAlg1: return map ? (KernelFn)k_acc_map<GT, VEC, kAlg1, NT, EXT> : (KernelFn)k_acc<GT, VEC, kAlg1, NT, EXT>;
  }
  return nullptr;
}

template <typename GT, int VEC, bool EXT>  // only streaming launches are large enough
KernelFn acc_rows_kernel(int phase) {
  switch (phase) {
    case kPlain: return (KernelFn)k_acc_rows<GT, VEC, kPlain, true, EXT>;
    case kLoopStart: return (KernelFn)k_acc_rows<GT, VEC, kLoopStart, true, EXT>;
    case kFold: return (KernelFn)k_acc_rows<GT, VEC, kFold, true, EXT>;
    case kAlg1: return (KernelFn)k_acc_rows<GT, VEC, kAlg1, true, EXT>;
  }
  return nullptr;
}

template <typename GT, int VEC>
KernelFn few_acc_kernel(int phase, bool map) {
  switch (phase) {
    case kPlain: return map ? (KernelFn)k_acc_few_map<GT, VEC, kPlain> : (KernelFn)k_acc_few<GT, VEC, kPlain>;
    case kLoopStart: return map ? (KernelFn)k_acc_few_map<GT, VEC, kLoopStart> : (KernelFn)k_acc_few<GT, VEC, kLoopStart>;
    case kFold: return map ? (KernelFn)k_acc_few_map<GT, VEC, kFold> : (KernelFn)k_acc_few<GT, VEC, kFold>;
    case kAlg1: return map ? (KernelFn)k_acc_few_map<GT, VEC, kAlg1> : (KernelFn)k_acc_few<GT, VEC, kAlg1>;
  }
  return nullptr;
}

// Does this launch go out on the short argument block?
bool few(const StepArgs& a, bool nt) {
  return !nt && a.ext == nullptr && a.n_loops == 0 && a.n_rows <= (uint32_t)kFewRows && a.n_cols <= (uint32_t)kFewRows;
}

// The short block of a launch: the used part of every table, and everything behind the tables.
StepArgsFew shortened(const StepArgs& a) {
  StepArgsFew f;
  memcpy(f.x_src, a.x_src, sizeof(f.x_src));
  memcpy(f.x_dst, a.x_dst, sizeof(f.x_dst));
  memcpy(f.m_hat, a.m_hat, sizeof(f.m_hat));
  memcpy(f.v_hat, a.v_hat, sizeof(f.v_hat));
  memcpy(f.acc, a.acc, sizeof(f.acc));
  memcpy(f.grad, a.grad, sizeof(f.grad));
  static_assert(sizeof(StepArgs) - offsetof(StepArgs, ext) == sizeof(StepArgsFew) - offsetof(StepArgsFew, ext),
                "the two blocks are alike behind the tables");
  memcpy((void*)&f.ext, (const void*)&a.ext, sizeof(f) - offsetof(StepArgsFew, ext));
  return f;
}

// A kernel may use more than 64 KB of dynamic LDS only after its limit has been raised; that is done
// once per (device, kernel), up to the largest size asked for so far.
int raise_lds_limit(KernelFn fn, uint32_t lds) {
  static std::mutex mu;
  static std::map<std::pair<int, const void*>, uint32_t> raised;
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  std::lock_guard<std::mutex> lock(mu);
  uint32_t& have = raised[{dev, fn}];
  if (have >= lds) return (int)hipSuccess;
  e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e == hipSuccess) have = lds;
  return (int)e;
}

// The status of the launch itself.  The runtime also keeps a failure for whoever asks for the last error next: it is
// taken away here, because the call that reports it is this one.
int enqueue(KernelFn fn, uint32_t grid, uint32_t block, void** args, uint32_t lds, void* stream) {
  const hipError_t e = hipLaunchKernel(fn, dim3(grid), dim3(block), args, lds, reinterpret_cast<hipStream_t>(stream));
  if (e != hipSuccess) (void)hipGetLastError();
  return (int)e;
}

int launch(KernelFn fn, bool short_block, uint32_t grid, uint32_t block, uint32_t lds, const StepArgs& a, void* stream) {
  if (fn == nullptr) return (int)hipErrorInvalidDeviceFunction;
  if (grid == 0) return (int)hipSuccess;
  if (lds > 65536u) {
    const int e = raise_lds_limit(fn, lds);
    if (e != (int)hipSuccess) return e;
  }
  if (short_block) {
    StepArgsFew f = shortened(a);
    void* args[] = {&f};
    return enqueue(fn, grid, block, args, lds, stream);
  }
  void* args[] = {const_cast<StepArgs*>(&a)};
  return enqueue(fn, grid, block, args, lds, stream);
}

// Launch of a kernel whose workgroups are one-wavefront pieces of work items (wide: whole items), for every row.  A grid holds less
// than 2^32 threads (17 billion float32 elements), so what is larger goes out in several launches.
int launch_pieces(KernelFn fn, bool short_block, StepArgs a, uint32_t n_items, void* stream, bool wide = false) {
  // with a sharing order every die gets the same number of workgroups (see k_direct)
  const uint32_t X = a.n_xcd;
  const uint32_t threads = wide ? kWave * kWideWaves : kWave, per_item = wide ? 1 : kDirectItem;  // workgroups per item and row
  const uint64_t per_piece = a.order == kOrderDieGroups ? X * a.order_group : a.n_rows;
  const uint32_t most = (uint32_t)(((1ull << 32) - 1) / threads / per_piece / per_item - X);
  int e = (int)hipSuccess;
  while (n_items > 0 && e == (int)hipSuccess) {
    const uint32_t now = n_items < most ? n_items : most;
    a.n_pieces = now * per_item;
    const uint32_t pieces = a.order == kOrderDieBlocks ? (a.n_pieces + X - 1) / X * X : a.n_pieces;
    e = launch(fn, short_block, (uint32_t)(pieces * per_piece), threads, a.reserve_lds, a, stream);
    a.work_begin += now;
    n_items -= now;
  }
  return e;
}

}  // namespace

// Address and capacity (in doubles) of `scratch` on the CURRENT device, resolved once per device.
int static_partials(double** out, uint32_t* capacity) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static double* addr[kMaxDevices] = {};
  *out = nullptr;
  *capacity = (uint32_t)(sizeof(scratch) / sizeof(double));
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!addr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    addr[dev] = static_cast<double*>(p);
  }
  *out = addr[dev];
  return (int)hipSuccess;
}

int launch_consensus_zero(double* partials, void* stream) {
  void* args[] = {&partials};
  return enqueue((KernelFn)k_consensus_zero, 1, 256, args, 0, stream);
}

int launch_consensus_sum(double* partials, double* out, void* stream) {
  void* args[] = {&partials, &out};
  return enqueue((KernelFn)k_consensus_sum, 1, 256, args, 0, stream);
}

int launch_probe(const void* const* src, void* const* dst, uint64_t elems, uint32_t n_xcd, void* stream) {
  if (elems % kProbeTile != 0 || n_xcd == 0) return (int)hipErrorInvalidValue;
  ProbeArgs a;
  for (uint32_t k = 0; k < kProbeStreams; ++k) {
    a.src[k] = static_cast<const float*>(src[k]);
    a.dst[k] = static_cast<float*>(dst[k]);
  }
  a.n_xcd = n_xcd;
  void* args[] = {&a};
  return enqueue((KernelFn)k_probe, (uint32_t)(elems / kProbeTile), 256, args, 0, stream);
}

int vec_elems(int xdt) { return xdt == DADAM_BF16 ? TBF16::vec : TF32::vec; }
bool tile_shape_supported(TileShape s) {
  if (s.ut == 2 && (s.waves == 8 || s.waves == 16)) return s.nontemporal;  // of float32 parameters
  if (s.ut == 1 && s.waves == 16) return true;                            // of more than 64 sources
  return (s.waves == 4 && s.ut == 2) || ((s.waves == 4 || s.waves == 8) && s.ut == 1);
}

// Loop kernel: a.loop_shares workgroups per tile and loop, in several launches where a grid would reach 2^32 threads.
static int launch_loops(int xdt, int gdt, Phase phase, TileShape shape, StepArgs a, uint32_t n_tiles, uint32_t lds_bytes,
                        void* stream) {
  KernelFn fn = nullptr;
  const bool nt = shape.nontemporal, ext = a.ext != nullptr, shared = a.loop_shares > 1, map = a.map != nullptr;
#define DADAM_PICK(name) (ext ? (nt ? loop_kernel_##name##_nt_ext(phase, shared, map) : loop_kernel_##name##_ext(phase, shared, map)) \
                              : (nt ? loop_kernel_##name##_nt(phase, shared, map) : loop_kernel_##name(phase, shared, map)))
  if (xdt == DADAM_F32 && gdt == DADAM_F32) fn = DADAM_PICK(f32_f32);
  if (xdt == DADAM_BF16 && gdt == DADAM_BF16) fn = DADAM_PICK(bf16_bf16);
  if (xdt == DADAM_BF16 && gdt == DADAM_F32) fn = DADAM_PICK(bf16_f32);
  if (xdt == DADAM_F32 && gdt == DADAM_BF16) fn = DADAM_PICK(f32_bf16);
#undef DADAM_PICK
  const uint32_t threads = (uint32_t)(kWave * shape.waves);
  const uint32_t most = (uint32_t)(((1ull << 32) - 1) / threads / (a.n_loops * a.loop_shares));
  int e = (int)hipSuccess;
  while (n_tiles > 0 && e == (int)hipSuccess) {
    const uint32_t now = n_tiles < most ? n_tiles : most;
    e = launch(fn, false, now * a.n_loops * a.loop_shares, threads, lds_bytes, a, stream);
    a.work_begin += now;
    n_tiles -= now;
  }
  return e;
}

int launch_tile(int xdt, int gdt, Phase phase, TileShape shape, const StepArgs& a, uint32_t n_work,
                uint32_t lds_bytes, void* stream) {
  if (a.n_loops > 0) return launch_loops(xdt, gdt, phase, shape, a, n_work, lds_bytes, stream);
  // A handle with more than 64 rows or sources keeps its pointer tables in device memory and runs kernels
  // compiled for that (kernels of their own, so that the small handles' register budget is not theirs).
  KernelFn fn = nullptr;
  const bool nt = shape.nontemporal, ext = a.ext != nullptr, map = a.map != nullptr;
  const bool short_block = few(a, nt);
#define DADAM_PICK(name) (short_block ? tile_kernel_##name##_few(phase, shape, map) : ext ? (nt ? tile_kernel_##name##_nt_ext(phase, shape, map) : tile_kernel_##name##_ext(phase, shape, map)) \
                              : (nt ? tile_kernel_##name##_nt(phase, shape, map) : tile_kernel_##name(phase, shape, map)))
  if (xdt == DADAM_F32 && gdt == DADAM_F32) fn = DADAM_PICK(f32_f32);
  if (xdt == DADAM_BF16 && gdt == DADAM_BF16) fn = DADAM_PICK(bf16_bf16);
  if (xdt == DADAM_BF16 && gdt == DADAM_F32) fn = DADAM_PICK(bf16_f32);
  if (xdt == DADAM_F32 && gdt == DADAM_BF16) fn = DADAM_PICK(f32_bf16);
#undef DADAM_PICK
  return launch(fn, short_block, n_work, (uint32_t)(kWave * shape.waves), lds_bytes, a, stream);
}

int launch_direct(int xdt, int gdt, Phase phase, bool nt, bool shared, bool whole_items, const StepArgs& a,
                  uint32_t n_work_tiles, void* stream) {
  KernelFn fn = nullptr;
  const bool ext = a.ext != nullptr, map = a.map != nullptr;
  if (whole_items) {
    if (phase == kMixOnly) gdt = xdt;  // no gradient: one kernel per parameter type
#define DADAM_PICK(name) (ext ? (nt ? rows_kernel_##name##_nt_ext(phase, map) : rows_kernel_##name##_ext(phase, map)) \
                              : (nt ? rows_kernel_##name##_nt(phase, map) : rows_kernel_##name(phase, map)))
    if (xdt == DADAM_F32 && gdt == DADAM_F32) fn = DADAM_PICK(f32_f32);
    if (xdt == DADAM_BF16 && gdt == DADAM_BF16) fn = DADAM_PICK(bf16_bf16);
    if (xdt == DADAM_F32 && gdt == DADAM_BF16) fn = DADAM_PICK(f32_bf16);
#undef DADAM_PICK
    return launch_pieces(fn, false, a, n_work_tiles, stream, true);
  }
  const bool short_block = few(a, nt);
#define DADAM_PICK(name) (short_block ? direct_kernel_##name##_few(phase, map) : ext ? (nt ? direct_kernel_##name##_nt_ext(phase, shared, map) : direct_kernel_##name##_ext(phase, shared, map)) \
                              : (nt ? direct_kernel_##name##_nt(phase, shared, map) : direct_kernel_##name(phase, shared, map)))
  if (xdt == DADAM_F32 && gdt == DADAM_F32) fn = DADAM_PICK(f32_f32);
  if (xdt == DADAM_BF16 && gdt == DADAM_BF16) fn = DADAM_PICK(bf16_bf16);
  if (xdt == DADAM_BF16 && gdt == DADAM_F32) fn = DADAM_PICK(bf16_f32);
  if (xdt == DADAM_F32 && gdt == DADAM_BF16) fn = DADAM_PICK(f32_bf16);
#undef DADAM_PICK
  return launch_pieces(fn, short_block, a, n_work_tiles, stream);
}

int launch_accumulate(int gdt, Phase phase, bool nt, bool whole_items, const StepArgs& a, uint32_t n_work_tiles, void* stream,
                      int vec) {
  KernelFn fn = nullptr;
  const bool ext = a.ext != nullptr, map = a.map != nullptr;
  const bool short_block = !whole_items && few(a, nt);
#define DADAM_PICK(GT, VEC)                                                                                      \
  (whole_items ? (ext ? acc_rows_kernel<GT, VEC, true>(phase) : acc_rows_kernel<GT, VEC, false>(phase))             \
   : short_block ? few_acc_kernel<GT, VEC>(phase, map) : ext ? (nt ? acc_kernel_for_phase<GT, VEC, true, true>(phase, map) : acc_kernel_for_phase<GT, VEC, false, true>(phase, map)) \
       : (nt ? acc_kernel_for_phase<GT, VEC, true, false>(phase, map) : acc_kernel_for_phase<GT, VEC, false, false>(phase, map)))
  if (gdt == DADAM_F32 && vec == 4) fn = DADAM_PICK(TF32, 4);
  if (gdt == DADAM_F32 && vec == 8) fn = DADAM_PICK(TF32, 8);
  if (gdt == DADAM_BF16 && vec == 4) fn = DADAM_PICK(TBF16, 4);
  if (gdt == DADAM_BF16 && vec == 8) fn = DADAM_PICK(TBF16, 8);
#undef DADAM_PICK
  return launch_pieces(fn, short_block, a, n_work_tiles, stream, whole_items);
}

}  // namespace dadam
