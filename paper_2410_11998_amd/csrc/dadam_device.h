// gfx950 kernels of the decentralized (accumulated) Adam step (device code, included by every kernel
// translation unit; the launchers are in dadam_kernels.hip).
//
//
// The work is streaming and elementwise over the packed parameter vector; neighbour mixing couples
// replicas, never elements.  The kernels:
//
//   k_tile    one workgroup owns a tile of elements for ALL rows: every source buffer's slice of the
//             tile is read from HBM once and parked in LDS, then the wavefronts of the group deal the
//             rows among themselves and update each from LDS.  Lane l of every wavefront works on
//             the same elements for all rows, so LDS is a per-lane indexable store - no lane ever
//             reads what another lane wrote, one barrier separates staging from use.  All sources
//             of the tile are read before anything is written, so updating in place is legal.
//   k_direct  one wavefront updates one vector per lane of one row and streams the row's sources from global
//             memory: a node's own parameters plus receive buffers, and rows that share sources where the
//             caches serve the second reader better than the staged tile does.
//   k_loop    one workgroup owns a piece of one loop: rows that list the same sources with the same weights share
//             one neighbour sum.
//   k_mix_rows, k_rows  large launches of what k_direct does for rows that share sources, whole items by four wavefronts.
//   k_acc     accumulate / fold only (Algorithm 3 lines 9-13).
//
// Every access of a full tile is a 128-bit (float32) or 64-bit (bfloat16) load or store per lane,
// laid out so that each instruction of a wavefront covers whole lines: one contiguous run of memory, or in kernels that
// stream two or four of them (see lane_start).  Tiles that a segment's edge cuts load whole groups of four and store single elements
// at the edge, or load element by element too (see Clip).  Neighbour lists are read once per
// row as one coalesced load (one entry per lane) and handed out with readlane, so the inner loop
// has no dependent scalar memory traffic - which also means that no lane may leave a wavefront
// before the last readlane (see direct_body).
#ifndef DADAM_DEVICE_H_
#define DADAM_DEVICE_H_

#include <hip/hip_runtime.h>

#include <type_traits>

#include "dadam_internal.h"

namespace dadam {
namespace {


// Distances in elements between the two groups of four that an 8-element lane vector consists of, and between a lane's two
// vectors.  Streaming kernels: sixteen lanes work side by side (see lane_start), and two float32 vectors lie like the two
// groups of a bfloat16 one.  Otherwise all lanes of the wavefront work side by side.
template <bool STREAM>
constexpr int kGroupStep = STREAM ? kWave : 4 * kWave;
template <int VEC, bool STREAM>
constexpr uint32_t kVectorStep = VEC == 4 && STREAM ? kGroupStep<STREAM> : kWave * VEC;

typedef float f4 __attribute__((ext_vector_type(4)));
typedef uint32_t u4 __attribute__((ext_vector_type(4)));
typedef uint32_t u2 __attribute__((ext_vector_type(2)));

// Which work item a workgroup takes.  Consecutive workgroup ids are dispatched to the device's X dies in turn.
//
// Tile mode: the n work items are cut into blocks of B and the blocks go to the dies in turn, so that each die
// (and its L2) walks runs of B consecutive tiles while all dies stay in the same neighbourhood of every array.
// B == 0: one contiguous X-th of the items per die.  A bijection of [0, X * (n / X)); the part of a die's
// share that does not fill a block is taken contiguously, and the last n mod X workgroups keep their item.
__device__ __forceinline__ uint32_t die_block_order(uint32_t b, uint32_t n, uint32_t X, uint32_t B) {
  const uint32_t chunk = n / X;
  if (b >= chunk * X) return b;
  const uint32_t x = b % X, j = b / X;
  if (B == 0) return x * chunk + j;
  const uint32_t whole = chunk / B * B;  // die x's first `whole` workgroups take their blocks
  return j < whole ? ((j / B) * X + x) * B + j % B : whole * X + x * (chunk - whole) + (j - whole);
}

// Direct mode with a sharing order of the R rows: die x takes positions [x R / X, (x + 1) R / X) of the order,
// tile after tile; every die gets G = ceil(R / X) workgroups per tile, and where R / X is not whole the last
// workgroup of some dies has no row (returns false).  Over b in [0, T X G) every (tile < T, position < R)
// comes up exactly once.
__device__ __forceinline__ bool die_group_order(uint32_t b, uint32_t R, uint32_t X, uint32_t G, uint32_t& tile,
                                                uint32_t& position) {
  const uint32_t x = b % X, j = b / X;
  tile = j / G;
  const uint32_t q = j - tile * G;
  const uint32_t first = x * R / X, count = (x + 1) * R / X - first;
  position = q < count ? first + q : 0;
  return q < count;
}

// Direct mode in die blocks: all R rows of a piece run on one die, and the dies take runs of B pieces in turn, as in tile
// mode.  A die walks `run` of its pieces at a time, row after row in the sharing order (1: all rows of a piece, then the
// next piece).  The grid is rounded up to whole dies (X ceil(n / X) R workgroups for n pieces); a workgroup beyond the last
// piece has nothing to do (returns false).
__device__ __forceinline__ bool die_block_piece(uint32_t b, uint32_t R, uint32_t X, uint32_t n, uint32_t B, uint32_t& piece,
                                                uint32_t& position, uint32_t run = 1) {
  const uint32_t x = b % X, j = b / X;
  uint32_t at = j / R;  // piece of the die
  position = j - at * R;
  if (run > 1) {
    const uint32_t each = (n + X - 1) / X, first = at / run * run, w = j - first * R, length = each - first < run ? each - first : run;
    position = w / length;
    at = first + (w - position * length);
  }
  const uint32_t index = at * X + x;
  const bool active = index < n;
  piece = active ? die_block_order(index, n, X, B) : 0;
  return active;
}

// Where a lane's first group of four elements lies, for tile `index` of N = 64 VEC U elements of a launch over [lo, hi).
//
// In streaming kernels the two halves of a wavefront work 8192 or 16384 elements apart: the tiles of a block of twice that
// many elements take its two halves side by side.  Why that helps is not known (timings alone show that address bits seven apart,
// 8 and 15, 9 and 16, are to differ together within an instruction, as if such bits chose a channel of the memory and an open row
// served both places; no counter shows either).  Found by trying which address bits the sixteen-lane groups, the lane's vectors, the dies and time should have: two
// placements of a wavefront's four runs of 256 bytes stand out, {0, 256, 32 K, 32 K + 256} and {0, 512, 64 K, 64 K + 512}
// with the lane's second group between; all others lie with or below the contiguous kilobyte.  Fraction of 8 TB/s,
// contiguous / spread: 7 reads and 2 writes 0.79 / 0.85, 80 reads and 32 writes of a tile of 16 rows with two vectors a lane 0.67 / 0.82
// (one vector 0.69 / 0.70), bfloat16 parameters with float32 state, 8 rows 0.69 / 0.80, one row 0.76 / 0.82, copy 0.85 / 0.86.
// Blocks that [lo, hi) cuts keep their elements in order (lane_in_order: a lane's place in its tile then).
template <int VEC, int U, bool STREAM>
__device__ __forceinline__ uint32_t lane_in_order(uint32_t l) {
  return STREAM && VEC * U > 4 ? 4 * (l & 15) + 8 * (l & 16) + (l >> 5) * 256 : 4 * l;
}
template <int VEC, int U>
constexpr uint32_t spread_distance = kWave * VEC * U == 256 ? 8192 : 16384;  // elements between the halves
template <int VEC, int U, bool STREAM>
__device__ __forceinline__ uint64_t lane_start(uint64_t index, uint64_t lo, uint64_t hi, int lane) {
  constexpr uint32_t N = kWave * VEC * U;
  const uint64_t first = index * N;
  const uint32_t l = (uint32_t)lane;
  if constexpr (!STREAM) return first + 4 * l;
  constexpr uint32_t NEAR = N == 256 ? 128 : 256, FAR = spread_distance<VEC, U>, BLOCK = 2 * FAR;
  static_assert(N == 256 || N == 512 || N == 1024, "one or two vectors a lane");
  const uint64_t block = first & ~(uint64_t)(BLOCK - 1);
  const bool whole = block >= lo && block + BLOCK <= hi;
  const uint32_t j = (uint32_t)(first - block) / N;  // tile of the block
  const uint64_t base = whole ? block + (N == 1024 ? (j & 1) * NEAR + (j >> 1) * N : j * NEAR) : first;
  return base + ((N == 256 ? 4 * (l & 31) : 4 * (l & 15) + 8 * (l & 16)) + (l >> 5) * (whole ? FAR : NEAR));
}

// One step of the search of all lanes of a wavefront for the segment of work item `work` among [s, s + n): lane k looks at
// every step-th segment's first work item (begin, increasing), the ballot of the answers narrows the range.
__device__ __forceinline__ uint32_t search_step(uint32_t n) { return (n + kWave - 1) / kWave; }
__device__ __forceinline__ bool search_not_after(const uint32_t* begin, uint32_t s, uint32_t n, uint32_t step, uint32_t lane,
                                                 uint32_t work) {
  const uint32_t at = lane * step;
  return at < n && begin[s + (at < n ? at : 0)] <= work;
}
__device__ __forceinline__ void search_narrow(uint64_t ballot, uint32_t step, uint32_t& s, uint32_t& n) {
  const uint32_t last = (uint32_t)__builtin_popcountll(ballot) - 1;  // lane 0 is always among them
  s += last * step;
  n = step < n - last * step ? step : n - last * step;
}

// Element types, with the elements per lane and vector of a handle whose parameters have that type:
// float32 4 (one 128-bit access); bfloat16 8, held as two groups of four (two 64-bit accesses of x and
// g, two 128-bit accesses of each float32 state vector; see load_vals for where the groups lie).
struct TF32 {
  typedef float elem;
  static constexpr int bytes = 4;
  static constexpr int vec = 4;
};
struct TBF16 {
  typedef uint16_t elem;
  static constexpr int bytes = 2;
  static constexpr int vec = 8;
};

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }

// float32 -> bfloat16, round to nearest even; NaN stays a quiet NaN.
__device__ __forceinline__ uint32_t f32_to_bf16_bits(float f) {
  uint32_t u = __float_as_uint(f);
  uint32_t r = (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
  return (f != f) ? ((u >> 16) | 0x40u) : r;
}

template <typename T>
__device__ __forceinline__ float load_elem(const void* base, uint64_t e) {
  if constexpr (T::bytes == 4) {
    return reinterpret_cast<const float*>(base)[e];
  } else {
    return bf16_bits_to_f32(reinterpret_cast<const uint16_t*>(base)[e]);
  }
}

template <typename T>
__device__ __forceinline__ void store_elem(void* base, uint64_t e, float v) {
  if constexpr (T::bytes == 4) {
    reinterpret_cast<float*>(base)[e] = v;
  } else {
    reinterpret_cast<uint16_t*>(base)[e] = (uint16_t)f32_to_bf16_bits(v);
  }
}

// Element e of type T (float or uint16_t).  An index of 32 bits counts from the tile's first element (see from): the distance in
// bytes then is 32 bits beside a uniform address.
template <typename T>
__device__ __forceinline__ const T* at(const void* base, uint64_t e) { return reinterpret_cast<const T*>(base) + e; }
template <typename T>
__device__ __forceinline__ T* at(void* base, uint64_t e) { return reinterpret_cast<T*>(base) + e; }
template <typename T>
__device__ __forceinline__ const T* at(const void* base, uint32_t e) {
  return reinterpret_cast<const T*>(static_cast<const char*>(base) + e * (uint32_t)sizeof(T));
}
template <typename T>
__device__ __forceinline__ T* at(void* base, uint32_t e) {
  return reinterpret_cast<T*>(static_cast<char*>(base) + e * (uint32_t)sizeof(T));
}

// The VEC elements of one lane and vector, of type T, widened to float.  VEC = 4: elements
// [e, e + 4).  VEC = 8: two groups of four, [e, e + 4) and [e + H, e + H + 4), where H is four times
// the number of lanes that work side by side (a wavefront): every access instruction of the group then covers one contiguous run of memory, 16
// bytes per lane for float32 and 8 for bfloat16, and every 128-byte line it touches is touched
// whole.  (Giving a lane 8 consecutive elements instead makes each float32 state access two
// instructions that each touch half of every line: measured 5-13 % slower once stores are involved.)
// e is a multiple of 4, so every group is 16-byte (float32) or 8-byte (bfloat16) aligned.
// Clipped tiles (CLIP) store only elements inside [lo, hi).  Their loads: kElements touches nothing else, and the rest reads
// as zero; one load an element, each waited for before the next group's can be issued.  kGroups loads whole groups, from
// the nearest group that holds an element of the range, so that all of a row's loads are in flight at once; what lies
// outside the range is loaded with it or repeated, and never used.  kGroupsZeroed does the same for sources and clears what lies
// outside (the consensus error counts on that).  Both need whole groups to end within the buffer (clip_of).  us, elements / groups:
// 8 replicas of 300 odd-sized tensors, bfloat16, four steps 68.6 / 59.8, one row of 700 such tensors 32.3 / 28.1 (bfloat16 37.5 /
// 33.8), ring of 12 x 20 tensors 26.2 / 22.0, 100 rows of seven sources x 400 tensors, bfloat16 1285 / 957.
// Streaming accesses: every global datum of a step is touched exactly once, so full-group
// accesses may carry the non-temporal hint (NT) and leave the caches to nobody in particular.
// Which classes of access carry the hint when a handle streams (all eight combinations measured:
// the hints on the stream loads and on the stores carry the gain, the one on source loads is neutral):
constexpr bool kNtSource = true;  // parameter (source) loads
constexpr bool kNtStream = true;  // gradient / moment / accumulator loads
constexpr bool kNtStore = true;   // all stores

template <bool NT, typename V>
__device__ __forceinline__ V vload(const V* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}
template <bool NT, typename V>
__device__ __forceinline__ void vstore(V* p, V v) {
  if constexpr (NT) __builtin_nontemporal_store(v, p);
  else *p = v;
}

enum Clip : int { kWhole = 0, kElements = 1, kGroups = 2, kGroupsZeroed = 3, kMapped = 4 };  // kMapped: all tiles of a layout with a map
template <typename E>
__device__ __forceinline__ E nearest_group(E e, E lo, E hi) {
  const E first = lo & ~(E)3, last = (hi - 1) & ~(E)3;
  const E up = e > first ? e : first;
  return up < last ? up : last;
}

template <typename T, int VEC, int H, int CLIP, bool NT, typename E>
__device__ __forceinline__ void load_vals(const void* base, E e, E lo, E hi, float (&out)[VEC]) {
  static_assert(VEC == 4 || (VEC == 8 && H >= 4), "a lane holds one or two groups of four elements");
  static_assert(CLIP != kGroupsZeroed, "only sources are cleared outside the range");
#pragma unroll
  for (int h = 0; h < VEC / 4; ++h) {
    const E group = e + (E)h * H, eh = CLIP >= kGroups ? nearest_group(group, lo, hi) : group;
    if (CLIP != kElements || (eh >= lo && eh + 4 <= hi)) {
      if constexpr (T::bytes == 4) {
        f4 v = vload<NT && kNtStream>(reinterpret_cast<const f4*>(at<float>(base, eh)));
        out[4 * h + 0] = v.x; out[4 * h + 1] = v.y; out[4 * h + 2] = v.z; out[4 * h + 3] = v.w;
      } else {
        u2 v = vload<NT && kNtStream>(reinterpret_cast<const u2*>(at<uint16_t>(base, eh)));
        out[4 * h + 0] = __uint_as_float(v.x << 16); out[4 * h + 1] = __uint_as_float(v.x & 0xFFFF0000u);
        out[4 * h + 2] = __uint_as_float(v.y << 16); out[4 * h + 3] = __uint_as_float(v.y & 0xFFFF0000u);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const E ej = eh + j;
        out[4 * h + j] = (ej >= lo && ej < hi) ? load_elem<T>(base, ej) : 0.0f;
      }
    }
  }
}

template <typename T, int VEC, int H, int CLIP, bool NT, typename E>
__device__ __forceinline__ void store_vals(void* base, E e, E lo, E hi, const float (&in)[VEC]) {
  static_assert(VEC == 4 || (VEC == 8 && H >= 4), "a lane holds one or two groups of four elements");
#pragma unroll
  for (int h = 0; h < VEC / 4; ++h) {
    const E eh = e + (E)h * H;
    if (CLIP == kWhole || (eh >= lo && eh + 4 <= hi)) {
      if constexpr (T::bytes == 4) {
        f4 v;
        v.x = in[4 * h + 0]; v.y = in[4 * h + 1]; v.z = in[4 * h + 2]; v.w = in[4 * h + 3];
        vstore<NT && kNtStore>(reinterpret_cast<f4*>(at<float>(base, eh)), v);
      } else {
        u2 v;
        v.x = f32_to_bf16_bits(in[4 * h + 0]) | (f32_to_bf16_bits(in[4 * h + 1]) << 16);
        v.y = f32_to_bf16_bits(in[4 * h + 2]) | (f32_to_bf16_bits(in[4 * h + 3]) << 16);
        vstore<NT && kNtStore>(reinterpret_cast<u2*>(at<uint16_t>(base, eh)), v);
      }
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const E ej = eh + j;
        if (ej >= lo && ej < hi) {
          if constexpr (sizeof(E) == 8) store_elem<T>(base, ej, in[4 * h + j]);
          else store_elem<T>(at<typename T::elem>(base, eh), j, in[4 * h + j]);
        }
      }
    }
  }
}

// What a launch may do to the elements of a lane's vector where the layout has a map: for group h, in bits 8 h to 8 h + 3, which
// elements it stores, and in bit 8 h + 4 whether they decay.
constexpr uint32_t kStoreBits = 0x0F, kDecayBit = 0x10;
template <typename E>
__device__ __forceinline__ uint32_t bits_inside(E group, E lo, E hi) {
  const uint32_t before = lo > group ? (lo - group < 4 ? (uint32_t)(lo - group) : 4u) : 0u;
  const uint32_t end = hi > group ? (hi - group < 4 ? (uint32_t)(hi - group) : 4u) : 0u;
  return (kStoreBits << before) & ((1u << end) - 1u);
}
template <typename T, int VEC, int H, bool NT, typename E>
__device__ __forceinline__ void store_bits(void* base, E e, uint32_t bits, const float (&in)[VEC]) {
#pragma unroll
  for (int h = 0; h < VEC / 4; ++h) {
    const E eh = e + (E)h * H;
    const uint32_t b = (bits >> (8 * h)) & kStoreBits;
    const float group[4] = {in[4 * h], in[4 * h + 1], in[4 * h + 2], in[4 * h + 3]};
    if (b == kStoreBits) {
      store_vals<T, 4, H, kWhole, NT>(base, eh, (E)0, (E)0, group);
    } else {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (b >> j & 1) store_elem<T>(at<typename T::elem>(base, eh), j, group[j]);
    }
  }
}

// The stores of a row's UT vectors.  With one vector per lane there must be no loop around the store: a loop
// that runs once has a loop-invariant address, the compiler's loop-invariant code motion then "promotes" the
// location to a register and re-creates the store behind the loop - without the non-temporal hint (seen with
// the bfloat16 one-vector tile kernels: 1.2 % slower on the ring of 8; the compile test counts the hints).
// Where the layout has a map they follow `bits`.
template <typename T, int VEC, int H, int CLIP, bool NT, int UT, typename E>
__device__ __forceinline__ void store_vectors(void* base, const E (&e)[UT], E lo, E hi, const uint32_t (&bits)[UT],
                                              const float (&in)[UT][VEC]) {
  if constexpr (CLIP == kMapped) {
#pragma unroll
    for (int u = 0; u < UT; ++u) store_bits<T, VEC, H, NT>(base, e[u], bits[u], in[u]);
  } else if constexpr (UT == 1) {
    store_vals<T, VEC, H, CLIP, NT>(base, e[0], lo, hi, in[0]);
  } else {
#pragma unroll
    for (int u = 0; u < UT; ++u) store_vals<T, VEC, H, CLIP, NT>(base, e[u], lo, hi, in[u]);
  }
}

// The 16 raw bytes of a lane's parameter vector (4 float32, or 2 x 4 bfloat16 in the two groups
// described above), as they are parked in LDS.
template <typename XT, int H, int CLIP, bool NT, typename E>
__device__ __forceinline__ u4 load_raw(const void* base, E e, E lo, E hi) {
  if constexpr (XT::bytes == 4) {
    if (CLIP != kElements || (e >= lo && e + 4 <= hi)) {
      const E eh = CLIP >= kGroups ? nearest_group(e, lo, hi) : e;
      u4 v = vload<NT && kNtSource>(reinterpret_cast<const u4*>(at<float>(base, eh)));
      if constexpr (CLIP == kGroupsZeroed) {
        v.x = e + 0 >= lo && e + 0 < hi ? v.x : 0u;
        v.y = e + 1 >= lo && e + 1 < hi ? v.y : 0u;
        v.z = e + 2 >= lo && e + 2 < hi ? v.z : 0u;
        v.w = e + 3 >= lo && e + 3 < hi ? v.w : 0u;
      }
      return v;
    }
    u4 r = {0u, 0u, 0u, 0u};
    const uint32_t* p = reinterpret_cast<const uint32_t*>(base);
    if (e + 0 >= lo && e + 0 < hi) r.x = p[e + 0];
    if (e + 1 >= lo && e + 1 < hi) r.y = p[e + 1];
    if (e + 2 >= lo && e + 2 < hi) r.z = p[e + 2];
    if (e + 3 >= lo && e + 3 < hi) r.w = p[e + 3];
    return r;
  } else {
    static_assert(XT::bytes == 4 || H >= 4, "bfloat16 vectors come in two groups");
    const uint16_t* p = reinterpret_cast<const uint16_t*>(base);
    u2 half[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const E group = e + (E)h * H, eh = CLIP >= kGroups ? nearest_group(group, lo, hi) : group;
      if (CLIP != kElements || (eh >= lo && eh + 4 <= hi)) {
        half[h] = vload<NT && kNtSource>(reinterpret_cast<const u2*>(at<uint16_t>(base, eh)));
        if constexpr (CLIP == kGroupsZeroed) {
          half[h].x &= (group + 0 >= lo && group + 0 < hi ? 0xFFFFu : 0u) | (group + 1 >= lo && group + 1 < hi ? 0xFFFF0000u : 0u);
          half[h].y &= (group + 2 >= lo && group + 2 < hi ? 0xFFFFu : 0u) | (group + 3 >= lo && group + 3 < hi ? 0xFFFF0000u : 0u);
        }
      } else {
        uint32_t q[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) q[j] = (eh + j >= lo && eh + j < hi) ? (uint32_t)p[eh + j] : 0u;
        half[h].x = q[0] | (q[1] << 16);
        half[h].y = q[2] | (q[3] << 16);
      }
    }
    u4 r = {half[0].x, half[0].y, half[1].x, half[1].y};
    return r;
  }
}

// What is computed from an index of a cut tile (clamped, scaled for each element type) is computed again after this, and held
// in no register from row to row or from a row's loads to its stores.
template <typename E>
__device__ __forceinline__ E afresh(E e) {
  if constexpr (sizeof(E) == 4) asm volatile("" : "+v"(e));
  return e;
}
// Clears the elements of a vector that the map leaves out (group: its bytes of the vector's groups, see load_map).
template <typename XT>
__device__ __forceinline__ u4 cleared(u4 r, const uint32_t (&group)[XT::vec / 4]) {
  if constexpr (XT::bytes == 4) {
    r.x = group[0] & 1 ? r.x : 0u;
    r.y = group[0] & 2 ? r.y : 0u;
    r.z = group[0] & 4 ? r.z : 0u;
    r.w = group[0] & 8 ? r.w : 0u;
  } else {
    auto halves = [](uint32_t b) { return (b & 1 ? 0xFFFFu : 0u) | (b & 2 ? 0xFFFF0000u : 0u); };
    const uint32_t g0 = afresh(group[0]), g1 = afresh(group[1]);
    r.x &= halves(g0);
    r.y &= halves(g0 >> 2);
    r.z &= halves(g1);
    r.w &= halves(g1 >> 2);
  }
  return r;
}

template <typename XT>
__device__ __forceinline__ void unpack_raw(u4 r, float (&out)[XT::vec]) {
  if constexpr (XT::bytes == 4) {
    out[0] = __uint_as_float(r.x); out[1] = __uint_as_float(r.y);
    out[2] = __uint_as_float(r.z); out[3] = __uint_as_float(r.w);
  } else {
    out[0] = __uint_as_float(r.x << 16); out[1] = __uint_as_float(r.x & 0xFFFF0000u);
    out[2] = __uint_as_float(r.y << 16); out[3] = __uint_as_float(r.y & 0xFFFF0000u);
    out[4] = __uint_as_float(r.z << 16); out[5] = __uint_as_float(r.z & 0xFFFF0000u);
    out[6] = __uint_as_float(r.w << 16); out[7] = __uint_as_float(r.w & 0xFFFF0000u);
  }
}

// ---------------------------------------------------------------------------------------------
// Algorithm 3, lines 6-13, for one element.  mix is the finished neighbour sum of line 8.
// Returns x^(t); updates mh, vh, b in registers according to the phase.
// ---------------------------------------------------------------------------------------------
// decay = lambda * x_own (0 where there is no weight decay): the AdamW-style part of the direction.
template <int PHASE>
__device__ __forceinline__ float element_step(const Scalars& s, float mix, float g, float& mh,
                                              float& vh, float& b, float decay) {
  if constexpr (PHASE == kMixOnly || PHASE == kMixConsensus) return mix;
  // lines 6-7: temporary moments from the persistent ones and the fresh gradient
  float m = fmaf(s.beta1, mh, s.omb1 * g);
  float v = fmaf(s.beta2, vh, s.omb2 * (g * g));
  // line 8: bias correction with exponent t_hat, epsilon outside the root
  float denom = sqrtf(v * s.inv_c2) + s.eps;
  float u = (m * s.inv_c1) / denom + decay;
  float x = fmaf(-s.lr, u, mix);
  // line 9
  if constexpr (PHASE == kPlain || PHASE == kFold) b = fmaf(g, s.inv_s, b);
  if constexpr (PHASE == kLoopStart || PHASE == kAlg1) b = g * s.inv_s;
  // lines 10-13
  if constexpr (PHASE == kFold || PHASE == kAlg1) {
    mh = fmaf(s.beta1, mh, s.omb1 * b);
    vh = fmaf(s.betav, vh, s.ombv * (b * b));
    b = 0.0f;
  }
  return x;
}

template <int PHASE>
struct Needs {
  static constexpr bool mixing_only = PHASE == kMixOnly || PHASE == kMixConsensus;
  static constexpr bool grad = !mixing_only;
  static constexpr bool moments_in = !mixing_only;
  static constexpr bool acc_in = PHASE == kPlain || PHASE == kFold;
  static constexpr bool acc_out = PHASE == kPlain || PHASE == kLoopStart || PHASE == kFold;
  static constexpr bool moments_out = PHASE == kFold || PHASE == kAlg1;
};

// The place of a launch's n tiles that comes up when the order says b.  Streaming kernels of large handles (LAST_FIRST) begin with the last tile:
// they load cut tiles element by element (see tile_entry), which is long, 6 or 12 rows to a wavefront one after the other, and at a layout's ragged end
// it was the launch's tail.  us of four steps, one cut tile, last / first: 96 rows of one loop, 3e7 elements 683 / 603, bfloat16 663 / 517 (mixing of 1e8 184 / 149),
// exponential graph on 96 rows 688 / 646, seven rounds of 96 bfloat16 pairs with the error 363 / 315.
template <bool LAST_FIRST>
__device__ __forceinline__ uint32_t begin_with_last(uint32_t b, uint32_t n) {
  return !LAST_FIRST ? b : b == 0 ? n - 1 : b - 1;
}

// Which segment does work item `work` belong to, and which tile of the launch's grid is it?  Every lane of the
// wavefront is active here.  In small launches, whose time is a chain of trips to memory, all lanes search the
// segments' first work items at once, 64 to a step: one trip for up to 64 segments, two for up to 4096, where a binary
// search takes one for each halving (8 replicas of 300 odd-sized tensors 74 -> 68 us a loop of four steps).  In large ones
// the binary search is served by the scalar cache and leaves the vector memory path alone.
// (Fields are read one by one through the pointer: copying the struct would put it in scratch.  The cast names global
// memory: the compiler would otherwise merge a read of a segment with the same read of the argument block into one
// through a generic pointer.)
template <bool MAP = false, typename A>
__device__ __forceinline__ void locate(const A& a, uint32_t work, uint64_t& tile_index,
                                       uint64_t& lo, uint64_t& hi, float& weight_decay) {
  if (MAP || a.n_seg == 1) {  // the launch's range lies inside the only segment, or the layout has a map
    tile_index = a.first_tile + work;
    lo = a.clip_lo;
    hi = a.clip_hi;
    weight_decay = a.weight_decay;
  } else {
    typedef const Segment __attribute__((address_space(4))) * GlobalSegments;  // constant memory: scalar loads
    typedef const uint32_t __attribute__((address_space(4))) * GlobalWork;
    const GlobalSegments seg = (GlobalSegments)a.seg;
    const uint32_t grid = a.grid;
    const GlobalWork work0 = (GlobalWork)(a.seg_work + (uint64_t)grid * a.n_seg);
    uint32_t s = 0, n = a.n_seg;  // the segment is one of [s, s + n)
    if (a.wide_search) {
      const uint32_t lane = threadIdx.x & (kWave - 1);
      const uint32_t* begin = a.seg_work + (uint64_t)grid * a.n_seg;  // first work item of each segment, increasing
      while (n > 1) {
        const uint32_t step = search_step(n);
        search_narrow(__ballot(search_not_after(begin, s, n, step, lane, work)), step, s, n);
      }
      s = __builtin_amdgcn_readfirstlane((int)s);
    } else {
      while (n > 1) {
        const uint32_t half = n >> 1;
        const bool right = work0[s + half] <= work;
        s = right ? s + half : s;
        n = right ? n - half : half;
      }
    }
    tile_index = seg[s].first_tile[grid] + (work - work0[s]);
    const uint64_t slo = seg[s].lo, shi = seg[s].hi;
    lo = slo > a.clip_lo ? slo : a.clip_lo;
    hi = shi < a.clip_hi ? shi : a.clip_hi;
    weight_decay = seg[s].weight_decay;
  }
}

// How the loads of a tile that [lo, hi) cuts are done.
template <typename A>
__device__ __forceinline__ int clip_of(const A& a, bool full, uint64_t hi) {
  return full ? kWhole : hi + 3 <= (a.d | 3) ? kGroups : kElements;
}

// The same lane and range as elements of a tile that [lo, hi) cuts (the block it lies in is cut as well, so lanes keep their order).
struct Cut {
  uint32_t e, lo, hi;
};
template <int VEC, int U, bool STREAM>
__device__ __forceinline__ Cut cut_of(uint64_t tbase, uint64_t lo, uint64_t hi, int lane) {
  constexpr uint32_t N = kWave * VEC * U;
  Cut c;
  c.e = lane_in_order<VEC, U, STREAM>((uint32_t)lane);
  c.lo = lo > tbase ? (uint32_t)(lo - tbase) : 0;
  c.hi = hi - tbase < N ? (uint32_t)(hi - tbase) : N;
  return c;
}

// Layouts with a map (many short tensors side by side): one dense grid of tiles over the whole vector.  A lane loads whole groups
// of four as if the vector were one tensor, padding included, and the map's byte for each group, in flight beside the data, says which
// elements it stores and whether they decay.  So no work item waits for a search (two trips to memory before the first load), a tile that
// several tensors cross is launched once instead of once for each, lanes are spread and tiles as wide as in layouts of one segment.
// Bound as those are, by HBM or by the launch; the map is a byte for every four elements of ONE row.  us, by segments / by the map, tensors of 1100 elements on
// average: 8 replicas of 300 tensors, bfloat16, decay, four steps 63.3 / 53.8; one row of 3000 tensors, bfloat16, four steps 104 / 77 (float32 103 / 90); 16
// replicas of 3000, four steps 1209 / 1005; 48 in pairs of 3000 1132 / 707; 96 in loops of 1000 2631 / 1988; mixing of 70 by threes of 1940, bfloat16
// 566 / 302; accumulation apart, 100 rows of 1000 4386 / 2623; the consensus error of 100 rows of 400 282 / 226.  In kernels of their own (_map): as a
// fourth body of the others it took a wavefront per SIMD from some and 0.5 to 3 % from mixing of layouts without a map.
// A tile of such a layout: its elements counted from `origin`, its first one or that of its block where lanes are spread.
struct MapTile {
  uint64_t origin;
  uint32_t e, lo, hi;
};
template <int VEC, int U, bool STREAM>
__device__ __forceinline__ MapTile map_tile(uint64_t tbase, uint64_t lo, uint64_t hi, int lane) {
  constexpr uint64_t BLOCK = 2 * spread_distance<VEC, U>;
  const uint64_t block = tbase & ~(BLOCK - 1);
  MapTile t;
  t.origin = STREAM && block >= lo && block + BLOCK <= hi ? block : tbase;
  t.e = (uint32_t)(lane_start<VEC, U, STREAM>(tbase / (kWave * VEC * U), lo, hi, lane) - t.origin);
  t.lo = lo > t.origin ? (uint32_t)(lo - t.origin) : 0;
  t.hi = hi - t.origin < BLOCK ? (uint32_t)(hi - t.origin) : (uint32_t)BLOCK;
  return t;
}

// What the map has for a lane's vectors at e (counted from origin): loaded before the data and first looked at behind it.
template <int VEC, int U>
struct MapBytes {
  uint32_t group[U][VEC / 4];
};
template <int VEC, int U, int H, typename A, typename E>
__device__ __forceinline__ MapBytes<VEC, U> load_map(const A& a, uint64_t origin, const E (&e)[U]) {
  const uint8_t* map = a.map + (origin >> 2);
  MapBytes<VEC, U> m;
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int h = 0; h < VEC / 4; ++h) m.group[u][h] = *at<uint8_t>(map, (E)((e[u] + h * H) >> 2));
  return m;
}
// What the launch may do to them: what lies in [lo, hi) (full: all of the tile), and of that what the map has.
template <int VEC, int U, int H, typename E>
__device__ __forceinline__ void group_bits(const MapBytes<VEC, U>& m, bool full, const E (&e)[U], E lo, E hi, uint32_t (&bits)[U]) {
  uint32_t inside[U];
#pragma unroll
  for (int u = 0; u < U; ++u) inside[u] = ~0u;
  if (!full) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      inside[u] = 0;
#pragma unroll
      for (int h = 0; h < VEC / 4; ++h) inside[u] |= (bits_inside<E>(e[u] + h * H, lo, hi) | kDecayBit) << (8 * h);
    }
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    bits[u] = m.group[u][0];
    if constexpr (VEC == 8) bits[u] |= m.group[u][1] << 8;
    bits[u] &= inside[u];
  }
}

// Pointers of the bound buffers.  EXT = false: from the argument block (at most kInlineRows rows and
// sources).  EXT = true: from the device-resident tables of a larger handle.  EXT is a parameter of the
// kernels themselves and the launcher picks: the small case is exactly the code it was before large handles
// existed, registers included (choosing per pointer inside the kernel cost 2.5 % with 64 rows, and a choice
// between two reads of the same type even forced the whole argument block into scratch; one branch around
// two bodies in one kernel gave the small case the large one's register count: bfloat16 plain phase 63 -> 71
// vector registers, 8 -> 7 wavefronts per SIMD, 1.2 % slower on the ring of 8).  The tables hold addresses as
// integers; the cast names global memory, or every access through the pointer would become a flat one
// (slower, and counted with the LDS operations the row loop waits for).
enum TableOf : int { kSrc = 0, kDst = 1, kMHat = 2, kVHat = 3, kAcc = 4 };  // order of BoundTables' members
static_assert(sizeof(BoundTables) == 5 * kMaxRows * sizeof(uint64_t), "BoundTables is five arrays of addresses");
template <typename P>
__device__ __forceinline__ P table_entry(const BoundTables* ext, TableOf which, int index) {
  const uint64_t v = reinterpret_cast<const uint64_t*>(ext)[which * kMaxRows + index];
  typedef typename std::remove_pointer<P>::type __attribute__((address_space(1))) * Global;
  return (P)(Global)v;
}
template <bool EXT, typename A>
__device__ __forceinline__ const void* src_of(const A& a, int c) {
  if constexpr (EXT) return table_entry<const void*>(a.ext, kSrc, c);
  else return a.x_src[c];
}
template <bool EXT, typename A>
__device__ __forceinline__ void* dst_of(const A& a, int i) {
  if constexpr (EXT) return table_entry<void*>(a.ext, kDst, i);
  else return a.x_dst[i];
}
template <bool EXT, typename A>
__device__ __forceinline__ float* m_hat_of(const A& a, int i) {
  if constexpr (EXT) return table_entry<float*>(a.ext, kMHat, i);
  else return a.m_hat[i];
}
template <bool EXT, typename A>
__device__ __forceinline__ float* v_hat_of(const A& a, int i) {
  if constexpr (EXT) return table_entry<float*>(a.ext, kVHat, i);
  else return a.v_hat[i];
}
template <bool EXT, typename A>
__device__ __forceinline__ float* acc_of(const A& a, int i) {
  if constexpr (EXT) return table_entry<float*>(a.ext, kAcc, i);
  else return a.acc[i];
}

// Up to 64 entries of row i's neighbour list, one per lane (a row with more entries is walked in chunks
// of 64), the row's length and where its list starts, as wave-uniform values.
struct RowList {
  int32_t col_v;
  float w_v;
  int deg;  // entries of the whole row
  int k0;   // index of the row's first entry in col / w
};

// Entries [k0 + first, k0 + first + 64) of a row of `deg` entries, one per lane.
template <typename A>
__device__ __forceinline__ void load_list_chunk(const A& a, RowList& r, int first, int lane) {
  const int left = r.deg - first;  // >= 1
  const int idx = r.k0 + first + (lane < left ? lane : 0);
  r.col_v = a.col[idx];
  r.w_v = a.w[idx];
}

// First chunk of the list of the row at `position` of a direct launch.  The lists lie at a fixed distance, so that
// nothing has to be known about the row before its list can be loaded (padding lists source 0).
template <typename A>
__device__ __forceinline__ RowList load_position_list(const A& a, int position, int lane) {
  RowList r;
  r.k0 = position * (int)a.list_stride;
  const int idx = r.k0 + (lane < (int)a.list_stride ? lane : 0);
  r.col_v = a.col[idx];
  r.w_v = a.w[idx];
  r.deg = __builtin_amdgcn_readfirstlane(a.row_len[position]);  // host guarantees 1 <= deg <= n_cols
  return r;
}

// All of row_ptr in registers (lane l of pair j holds row_ptr[64 j + l] and row_ptr[64 j + l + 1]; one
// pair covers 64 rows, three the 160 rows a large handle may have), so that a wavefront that walks
// several rows finds each row's bounds with two lane reads instead of a load it would have to wait for
// behind its own earlier stores.
template <bool EXT>
struct RowPtrs {
  static constexpr int pairs = EXT ? (kMaxRows + kWave - 1) / kWave : 1;
  int32_t lo[pairs], hi[pairs];
};

template <bool EXT, typename A>
__device__ __forceinline__ RowPtrs<EXT> load_row_ptrs(const A& a, int lane) {
  RowPtrs<EXT> p;
#pragma unroll
  for (int j = 0; j < RowPtrs<EXT>::pairs; ++j) {
    const int r = j * kWave + lane < (int)a.n_rows ? j * kWave + lane : 0;
    p.lo[j] = a.row_ptr[r];
    p.hi[j] = a.row_ptr[r + 1];
  }
  return p;
}

// First chunk of row `row`'s list (row is wave-uniform).
template <bool EXT, typename A>
__device__ __forceinline__ RowList load_row_list(const A& a, const RowPtrs<EXT>& p, int row, int lane) {
  int k0 = 0, k1 = 0;
  if constexpr (!EXT) {
    k0 = __builtin_amdgcn_readlane(p.lo[0], row);
    k1 = __builtin_amdgcn_readlane(p.hi[0], row);
  } else {
#pragma unroll
    for (int j = 0; j < RowPtrs<EXT>::pairs; ++j)
      if (row >= j * kWave && row < (j + 1) * kWave) {  // wave-uniform: one of the pairs
        k0 = __builtin_amdgcn_readlane(p.lo[j], row - j * kWave);
        k1 = __builtin_amdgcn_readlane(p.hi[j], row - j * kWave);
      }
  }
  RowList r;
  r.deg = k1 - k0;  // host guarantees 1 <= deg <= n_cols
  r.k0 = k0;
  load_list_chunk(a, r, 0, lane);
  return r;
}

// Entry k (0 <= k < 64) of the chunk the list currently holds.
__device__ __forceinline__ int list_col(const RowList& r, int k) {
  return __builtin_amdgcn_readlane(r.col_v, k);
}
__device__ __forceinline__ float list_w(const RowList& r, int k) {
  return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(r.w_v), k));
}

// ---------------------------------------------------------------------------------------------
// tile mode
// ---------------------------------------------------------------------------------------------
// Where a body works: elements of the buffers (origin 0), or, in tiles whose loads go by groups, elements of the tile from
// `origin` on.  A kernel's registers are those of its largest body: with clamped 64-bit indexes the body for such tiles took 4 to
// 20 more than that for whole ones, and a wavefront per SIMD from 119 kernels.  us, without that body / 64 / 32 bits: bfloat16 steps that
// do not stream 145.0 / 146.5 / 144.4 (16 replicas), 76.9 / 77.5 / 76.6 (96 replicas); 25 MB buckets of a bfloat16 row 2252 / 2246 / 2177;
// 8 replicas of 300 odd-sized tensors 68.8 / 60.0 / 58.8; mixing of 16 x 19 million elements 1464 / 1468 / 1452.  Mixing by tiles that
// do not stream, direct mixing, mixing of loops and accumulation have registers to spare and keep 64: tiles of 12 bfloat16 replicas of
// odd-sized tensors 32.0 / 33.8, direct mixing of 48 rows of 250 thousand elements 102 / 115, accumulation of 16 rows 1843 / 2134.
// Steps of bfloat16 rows with float32 gradients by tiles that do not stream keep 64 too, but for the fold (74 registers, 71 with 32):
// 8 replicas of 1 million elements in 200 odd-sized tensors 43.2 / 44.9, 5 replicas of 530 thousand 75.2 / 78.3, 16 replicas of 10 million
// 166.4 / 166.7.  With bfloat16 gradients the same layouts give 42.4 / 44.1 and 147.8 / 146.1 (69 registers, 63 with 32).
template <int BYTES, typename P>
__device__ __forceinline__ P* from(P* base, uint64_t origin) {
  typedef typename std::conditional<std::is_const<P>::value, const char, char>::type Byte;
  return reinterpret_cast<P*>(reinterpret_cast<Byte*>(base) + origin * BYTES);
}

template <int STEP, int U, typename E>
__device__ __forceinline__ void vector_indexes(E start, E (&e)[U]) {
#pragma unroll
  for (int u = 0; u < U; ++u) e[u] = start + u * STEP;
}

// Weight decay of element j of a vector: where the layout has a map only if the bits say so.
template <int CLIP>
__device__ __forceinline__ float decay_of(uint32_t bits, int j, float wd, float x) {
  return CLIP != kMapped || (bits & (kDecayBit << (8 * (j / 4)))) ? wd * x : 0.0f;
}

// The stream inputs of one row of a tile: gradient, moments, accumulator (whatever the phase needs).
template <typename GT, int PHASE, int VEC, int UT, int CLIP, bool NT, bool EXT, typename A, typename E>
__device__ __forceinline__ void load_row_inputs(const A& a, int i, uint64_t origin, const E (&e)[UT], E lo,
                                                E hi, float (&g)[UT][VEC], float (&mh)[UT][VEC],
                                                float (&vh)[UT][VEC], float (&b)[UT][VEC]) {
  if constexpr (Needs<PHASE>::grad) {
    const void* gp = from<GT::bytes>(a.grad[i], origin);
#pragma unroll
    for (int u = 0; u < UT; ++u) load_vals<GT, VEC, kGroupStep<NT>, CLIP, NT>(gp, e[u], lo, hi, g[u]);
  }
  if constexpr (Needs<PHASE>::moments_in) {
    const float* mp = from<4>(m_hat_of<EXT>(a, i), origin);
    const float* vp = from<4>(v_hat_of<EXT>(a, i), origin);
#pragma unroll
    for (int u = 0; u < UT; ++u) load_vals<TF32, VEC, kGroupStep<NT>, CLIP, NT>(mp, e[u], lo, hi, mh[u]);
#pragma unroll
    for (int u = 0; u < UT; ++u) load_vals<TF32, VEC, kGroupStep<NT>, CLIP, NT>(vp, e[u], lo, hi, vh[u]);
  }
  if constexpr (Needs<PHASE>::acc_in) {
    const float* bp = from<4>(acc_of<EXT>(a, i), origin);
#pragma unroll
    for (int u = 0; u < UT; ++u) load_vals<TF32, VEC, kGroupStep<NT>, CLIP, NT>(bp, e[u], lo, hi, b[u]);
  }
}

// Mixing from LDS, the update of Algorithm 3 and the stores of one row of a tile.
template <typename XT, int PHASE, int VEC, int UT, int CLIP, bool NT, bool EXT, typename A, typename E>
__device__ __forceinline__ void finish_row(const A& a, const u4* lds, int i, RowList rl,
                                           uint64_t origin, E start, E lo, E hi, const uint32_t (&bits)[UT], float wd, int lane,
                                           float (&g)[UT][VEC], float (&mh)[UT][VEC], float (&vh)[UT][VEC],
                                           float (&b)[UT][VEC]) {
  // neighbour sum in the order the row lists its entries: first a product, then fused
  // multiply-adds
  float mix[UT][VEC];
  {
    const int c0 = list_col(rl, 0);
    const float w0 = list_w(rl, 0);
#pragma unroll
    for (int u = 0; u < UT; ++u) {
      float xs[VEC];
      unpack_raw<XT>(lds[(c0 * UT + u) * kWave + lane], xs);
#pragma unroll
      for (int j = 0; j < VEC; ++j) mix[u][j] = w0 * xs[j];
    }
  }
  for (int k = 1, first = 0; k < rl.deg; ++k) {
    if constexpr (EXT) {
      if (k - first == kWave) {  // a row of more than 64 entries: the next 64 of them
        first = k;
        load_list_chunk(a, rl, first, lane);
      }
    }
    const int c = list_col(rl, k - first);
    const float wk = list_w(rl, k - first);
#pragma unroll
    for (int u = 0; u < UT; ++u) {
      float xs[VEC];
      unpack_raw<XT>(lds[(c * UT + u) * kWave + lane], xs);
#pragma unroll
      for (int j = 0; j < VEC; ++j) mix[u][j] = fmaf(wk, xs[j], mix[u][j]);
    }
  }

  // decoupled weight decay acts on the row's own previous parameters: source buffer i
  float decay[UT][VEC];
#pragma unroll
  for (int u = 0; u < UT; ++u)
#pragma unroll
    for (int j = 0; j < VEC; ++j) decay[u][j] = 0.0f;
  if (!Needs<PHASE>::mixing_only && wd != 0.0f) {
#pragma unroll
    for (int u = 0; u < UT; ++u) {
      float xs[VEC];
      unpack_raw<XT>(lds[(i * UT + u) * kWave + lane], xs);
#pragma unroll
      for (int j = 0; j < VEC; ++j) decay[u][j] = decay_of<CLIP>(bits[u], j, wd, xs[j]);
    }
  }

  float xo[UT][VEC];
#pragma unroll
  for (int u = 0; u < UT; ++u)
#pragma unroll
    for (int j = 0; j < VEC; ++j)
      xo[u][j] = element_step<PHASE>(a.s, mix[u][j], g[u][j], mh[u][j], vh[u][j], b[u][j], decay[u][j]);

  E e[UT];
  vector_indexes<kVectorStep<VEC, NT>>(VEC * UT > 4 ? afresh(start) : start, e);
  store_vectors<XT, VEC, kGroupStep<NT>, CLIP, NT>(from<XT::bytes>(dst_of<EXT>(a, i), origin), e, lo, hi, bits, xo);
  if constexpr (Needs<PHASE>::acc_out) store_vectors<TF32, VEC, kGroupStep<NT>, CLIP, NT>(from<4>(acc_of<EXT>(a, i), origin), e, lo, hi, bits, b);
  if constexpr (Needs<PHASE>::moments_out) {
    store_vectors<TF32, VEC, kGroupStep<NT>, CLIP, NT>(from<4>(m_hat_of<EXT>(a, i), origin), e, lo, hi, bits, mh);
    store_vectors<TF32, VEC, kGroupStep<NT>, CLIP, NT>(from<4>(v_hat_of<EXT>(a, i), origin), e, lo, hi, bits, vh);
  }
}

template <typename XT, typename GT, int PHASE, int W, int UT, int CLIP, bool NT, bool EXT, typename A, typename E>
__device__ __forceinline__ void tile_body(const A& a, u4* lds, uint64_t origin, E start, E lo, E hi, bool full, float wd, uint32_t tile_id,
                                          int lane, int wave) {
  constexpr int VEC = XT::vec;
  E e[UT];
  vector_indexes<kVectorStep<VEC, NT>>(start, e);
  MapBytes<VEC, UT> map;
  if constexpr (CLIP == kMapped) map = load_map<VEC, UT, kGroupStep<NT>>(a, origin, e);
  uint32_t bits[UT];
  // the consensus error counts on zeros outside the tensors
  constexpr bool CLEAR = CLIP == kMapped && PHASE == kMixConsensus;

  const int n_rows = (int)a.n_rows;
  const RowPtrs<EXT> rp = load_row_ptrs<EXT>(a, lane);

  // stage every source buffer's slice of the tile: HBM -> registers -> LDS, once.  With more than
  // two sources per wavefront, a wavefront issues the loads of up to KB of them before it parks
  // the first, so that their latencies overlap (+3 % with 64 sources); with one or two, taking
  // them in turn is faster (3 % in the bfloat16 ring of 8), so both forms are here.
  const int n_cols = (int)a.n_cols;
  if (n_cols > 2 * W) {
    constexpr int KB = 8 / UT;
    for (int c0 = wave; c0 < n_cols; c0 += KB * W) {
      u4 r[KB][UT];
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int c = c0 + k * W;
        if (c < n_cols) {
          const void* src = from<XT::bytes>(src_of<EXT>(a, c), origin);
#pragma unroll
          for (int u = 0; u < UT; ++u) r[k][u] = load_raw<XT, kGroupStep<NT>, CLIP, NT>(src, e[u], lo, hi);
        }
      }
#pragma unroll
      for (int k = 0; k < KB; ++k) {
        const int c = c0 + k * W;
        if (c < n_cols) {
#pragma unroll
          for (int u = 0; u < UT; ++u) lds[(c * UT + u) * kWave + lane] = CLEAR ? cleared<XT>(r[k][u], map.group[u]) : r[k][u];
        }
      }
    }
  } else {
    for (int c = wave; c < n_cols; c += W) {
      const void* src = from<XT::bytes>(src_of<EXT>(a, c), origin);
      u4 r[UT];
#pragma unroll
      for (int u = 0; u < UT; ++u) r[u] = load_raw<XT, kGroupStep<NT>, CLIP, NT>(src, e[u], lo, hi);
#pragma unroll
      for (int u = 0; u < UT; ++u) lds[(c * UT + u) * kWave + lane] = CLEAR ? cleared<XT>(r[u], map.group[u]) : r[u];
    }
  }
  // the first row's neighbour list travels while the group meets at the barrier
  RowList rl_next = load_row_list(a, rp, wave < n_rows ? wave : 0, lane);
  __syncthreads();
  if constexpr (CLIP == kMapped) group_bits<VEC, UT, kGroupStep<NT>>(map, full, e, lo, hi, bits);

  if constexpr (PHASE == kMixConsensus) {
    // Consensus error of the sources, sum_c (x_c - mean)^2 per element, as a by-product: the whole
    // tile is in LDS anyway.  One pass on values shifted by source 0, y_c = x_c - x_0, so that
    // sum y^2 - (sum y)^2 / C does not cancel.  The work is dealt evenly: each wavefront takes
    // PER of the tile's 16-byte slots, and its G = 64 / PER lane groups take every G-th source;
    // the groups' sums of y meet through lane exchanges before they are squared.
    // Elements outside the segment were staged as zeros in every source and add nothing.
    constexpr int PER = UT * kWave / W;
    constexpr int G = kWave / PER;
    static_assert(PER >= 1 && PER * W == UT * kWave && G * PER == kWave, "tile does not divide");
    const int q = wave * PER + (lane % PER);
    const int grp = lane / PER;
    float ref[VEC], s1[VEC], s2[VEC];
    unpack_raw<XT>(lds[q], ref);
#pragma unroll
    for (int j = 0; j < VEC; ++j) { s1[j] = 0.0f; s2[j] = 0.0f; }
    for (int c = 1 + grp; c < n_cols; c += G) {
      float xs[VEC];
      unpack_raw<XT>(lds[c * (UT * kWave) + q], xs);
#pragma unroll
      for (int j = 0; j < VEC; ++j) {
        const float y = xs[j] - ref[j];
        s1[j] += y;
        s2[j] = fmaf(y, y, s2[j]);
      }
    }
#pragma unroll
    for (int off = PER; off < kWave; off <<= 1)
#pragma unroll
      for (int j = 0; j < VEC; ++j) s1[j] += __shfl_xor(s1[j], off);
    const float inv_c = grp == 0 ? 1.0f / (float)n_cols : 0.0f;
    float acc = 0.0f;
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc += s2[j] - s1[j] * s1[j] * inv_c;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0)
      atomicAdd(a.partials + ((tile_id * (uint32_t)W + (uint32_t)wave) % kConsensusPartials), (double)acc);
  }

  // Each row's list is fetched one row ahead, so that no row waits for a load issued behind the
  // previous row's stores (memory operations of a wavefront retire in order).
  // (Issuing the next row's gradient and state loads early as well was measured and changes
  // nothing: with 8-32 wavefronts per CU in flight the memory system, not latency, is the limit.)
  for (int i = wave; i < n_rows; i += W) {
    const RowList rl = rl_next;
    rl_next = load_row_list(a, rp, i + W < n_rows ? i + W : i, lane);
    float g[UT][VEC], mh[UT][VEC], vh[UT][VEC], b[UT][VEC];
    if (VEC * UT > 4) start = afresh(start);
    vector_indexes<kVectorStep<VEC, NT>>(start, e);
    load_row_inputs<GT, PHASE, VEC, UT, CLIP, NT, EXT>(a, i, origin, e, lo, hi, g, mh, vh, b);
    finish_row<XT, PHASE, VEC, UT, CLIP, NT, EXT>(a, lds, i, rl, origin, start, lo, hi, bits, wd, lane, g, mh, vh, b);
  }
}

template <typename XT, typename GT, int PHASE, int W, int UT, bool NT, bool EXT, bool MAP, typename A>
__device__ __forceinline__ void tile_entry(const A& a) {
  constexpr int VEC = XT::vec;
  constexpr uint64_t TILE = (uint64_t)kWave * VEC * UT;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_bytes[];
  u4* lds = reinterpret_cast<u4*>(lds_bytes);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // Consecutive workgroup ids are dispatched to the device's X dies (XCDs, 8 on an MI355X) in turn.
  // Left alone, every die would touch every X-th tile of every array.  Instead the tiles are cut into blocks
  // of B = 32 and the blocks go to the dies in turn, so that each die (and its L2) reads and writes runs of
  // 32 consecutive tiles while all dies stay in the same neighbourhood of every array.  Measured on the
  // placed layout, against tile-by-tile round robin: one contiguous X-th of the tiles per die +2.5 %; blocks
  // of 32 tiles another +0.4 % (float32, 16 replicas) to +1.5 % (bfloat16 ring of 8); blocks of 16 ... 1024
  // all lie within 0.5 % of that, powers of two ahead of their neighbours.  With the lanes spread (lane_start) blocks of 32 to
  // 256 lie within 1 % for steps, and of 8 up to 8 % behind; streaming mixing takes 256 (kDieBlockMix: bfloat16 ring of 8 0.787 against
  // 0.794, 16 sources with the consensus error 0.76 against 0.78, the same without the error).
  const uint32_t b = die_block_order(blockIdx.x, gridDim.x, a.n_xcd, a.xcd_block);
  uint64_t tile_index, lo, hi;
  float wd;
  locate<MAP>(a, a.work_begin + begin_with_last<NT && EXT && !MAP>(b, gridDim.x), tile_index, lo, hi, wd);
  const uint64_t tbase = tile_index * TILE;
  const bool full = tbase >= lo && tbase + TILE <= hi;
  if constexpr (MAP) {
    const MapTile t = map_tile<VEC, UT, NT>(tbase, lo, hi, lane);
    tile_body<XT, GT, PHASE, W, UT, kMapped, NT, EXT>(a, lds, t.origin, t.e, t.lo, t.hi, full, wd, b, lane, wave);
  } else {
    const uint64_t start = lane_start<VEC, UT, NT>(tile_index, lo, hi, lane);
    const Cut cut = cut_of<VEC, UT, NT>(tbase, lo, hi, lane);
    // streaming launches of large handles have few cut tiles: a third body with its look-ups in the tables is not worth its size
    constexpr int CUT = NT && EXT ? kElements : PHASE == kMixConsensus ? kGroupsZeroed : kGroups;
    // see `from`; bfloat16 rows with float32 gradients keep their wavefronts with 64 bits where nothing is folded
    constexpr bool NARROW = NT || (Needs<PHASE>::grad && (XT::bytes == 4 || GT::bytes == 2 || PHASE == kFold));
    const int clip = clip_of(a, full, hi);
    if (clip == kWhole) tile_body<XT, GT, PHASE, W, UT, kWhole, NT, EXT>(a, lds, 0, start, lo, hi, full, wd, b, lane, wave);
    else if (CUT != kElements && clip == kGroups && NARROW) tile_body<XT, GT, PHASE, W, UT, CUT, NT, EXT>(a, lds, tbase, cut.e, cut.lo, cut.hi, full, wd, b, lane, wave);
    else if (CUT != kElements && clip == kGroups) tile_body<XT, GT, PHASE, W, UT, CUT, NT, EXT>(a, lds, 0, start, lo, hi, full, wd, b, lane, wave);
    else tile_body<XT, GT, PHASE, W, UT, kElements, NT, EXT>(a, lds, 0, start, lo, hi, full, wd, b, lane, wave);
  }
}

// ---------------------------------------------------------------------------------------------
// direct mode
// ---------------------------------------------------------------------------------------------
// A work item is kDirectItem parameter vectors of 16 bytes per lane of a wavefront (2048 float32 or 4096
// bfloat16 elements of one row); kPieces workgroups of ONE wavefront take it, one vector per lane each.
// The kernel is bound by HBM.  Why one small workgroup per vector: what the memory sustains depends on how
// much of a stream one workgroup covers, because consecutive workgroups go to the eight dies in turn.  7 reads
// and 2 writes of 1.4 GB arrays in place (one node's share), fraction of 8 TB/s by bytes of a stream per workgroup
// (ordinary allocations): 8 KB 0.73 (256 threads, two vectors: what this kernel used to be), 4 KB 0.74, 2 KB 0.78,
// 1 KB 0.795; the same with the hints off 0.68.  On the step itself: one row with three sources 0.72 -> 0.76.  The wavefront's
// two halves lie apart since (lane_start): 64 replicas in pairs 0.655 -> 0.778 on the same buffers, one row 0.81 -> 0.82.
constexpr int kPieces = kDirectItem;

// Where workgroup `b` of a launch over one-wavefront pieces works: `tile` counts pieces of the launch.
struct PieceAt {
  uint64_t index, lo, hi;  // which piece of the layout
  float wd;
  bool any, full;  // some / all elements of the piece lie in [lo, hi)
};
template <int VEC, bool MAP, typename A>
__device__ __forceinline__ PieceAt locate_piece(const A& a, uint32_t tile) {
  constexpr uint64_t PIECE = (uint64_t)kWave * VEC;
  PieceAt p;
  uint64_t tile_index;
  locate<MAP>(a, a.work_begin + tile / kPieces, tile_index, p.lo, p.hi, p.wd);
  p.index = tile_index * kPieces + tile % kPieces;
  const uint64_t tbase = p.index * PIECE;
  p.any = tbase < p.hi && tbase + PIECE > p.lo;
  p.full = tbase >= p.lo && tbase + PIECE <= p.hi;
  return p;
}

// N entries of the neighbour sum, from entry k of the list's chunk on, with all loads issued before the first
// use.  FIRST: the sum starts with a product, everything after that is a fused multiply-add.  Where the list
// names source own.col, its values are kept in own.x.
template <int VEC>
struct OwnSource {
  int col;  // wave-uniform; -1: not wanted
  bool found = false;
  float x[VEC];
};
template <typename XT, int N, bool FIRST, int U, int H, int CLIP, bool NT, bool EXT, typename A, typename E>  // NT: hint on the source loads
__device__ __forceinline__ void mix_entries(const A& a, const RowList& rl, int k, uint64_t origin, const E (&e)[U], E lo,
                                            E hi, float (&mix)[U][XT::vec], OwnSource<XT::vec>& own) {
  constexpr int VEC = XT::vec;
  u4 r[N][U];
  float wk[N];
  E f[U];
#pragma unroll
  for (int u = 0; u < U; ++u) f[u] = afresh(e[u]);
#pragma unroll
  for (int q = 0; q < N; ++q) {
    const void* src = from<XT::bytes>(src_of<EXT>(a, list_col(rl, k + q)), origin);
    wk[q] = list_w(rl, k + q);
#pragma unroll
    for (int u = 0; u < U; ++u) r[q][u] = load_raw<XT, H, CLIP, NT>(src, f[u], lo, hi);
  }
#pragma unroll
  for (int q = 0; q < N; ++q)
#pragma unroll
    for (int u = 0; u < U; ++u) {
      float xs[VEC];
      unpack_raw<XT>(r[q][u], xs);
      if constexpr (U == 1)
        if (list_col(rl, k + q) == own.col) {
          own.found = true;
#pragma unroll
          for (int j = 0; j < VEC; ++j) own.x[j] = xs[j];
        }
#pragma unroll
      for (int j = 0; j < VEC; ++j) mix[u][j] = (FIRST && q == 0) ? wk[0] * xs[j] : fmaf(wk[q], xs[j], mix[u][j]);
    }
}

// Neighbour sum of one row, in the order the row lists its entries, for U vectors per lane.  Batches of sources in flight:
// with two bfloat16 vectors a lane (16 sums live) they are two sources after the first four: four more cost 76 registers
// and with them the seventh wavefront (mixing in pairs, 24 to 64 rows, 0.96-0.98 -> 1.00-1.02 of the rate of workgroups of
// 67 registers, 96 rows of three 1.07 -> 1.13, rows of seven the same).
template <typename XT, int U, int H, int CLIP, bool NT, bool EXT, typename A, typename E>
__device__ __forceinline__ void mix_direct(const A& a, RowList rl, int lane, uint64_t origin, const E (&e)[U], E lo,
                                           E hi, float (&mix)[U][XT::vec], OwnSource<XT::vec>& own) {
#define DADAM_MIX(N, FIRST, K) mix_entries<XT, N, FIRST, U, H, CLIP, NT, EXT>(a, rl, K, origin, e, lo, hi, mix, own)
  constexpr int FIRST_BATCH = U == 1 ? 8 : 4;
  if (rl.deg < FIRST_BATCH) {
    switch (rl.deg) {
      case 1: DADAM_MIX(1, true, 0); break;
      case 2: DADAM_MIX(2, true, 0); break;
      case 3: DADAM_MIX(3, true, 0); break;
      default:
        if constexpr (FIRST_BATCH > 4) switch (rl.deg) {
          case 4: DADAM_MIX(4, true, 0); break;
          case 5: DADAM_MIX(5, true, 0); break;
          case 6: DADAM_MIX(6, true, 0); break;
          default: DADAM_MIX(7, true, 0); break;
        }
    }
  } else {
    DADAM_MIX(FIRST_BATCH, true, 0);
    constexpr int BATCH = U == 2 && XT::vec == 8 ? 2 : 4;
    int k = FIRST_BATCH, first = 0;
    for (; k + BATCH <= rl.deg; k += BATCH) {
      if constexpr (EXT) {
        if (k - first == kWave) {  // a row of more than 64 entries: the next 64 of them (64 is 4 or 8 and batches)
          first = k;
          load_list_chunk(a, rl, first, lane);
        }
      }
      DADAM_MIX(BATCH, false, k - first);
    }
    if (k < rl.deg) {
      if constexpr (EXT) {
        if (k - first == kWave) {
          first = k;
          load_list_chunk(a, rl, first, lane);
        }
      }
      if constexpr (BATCH > 2)
        if ((rl.deg - k) & 2) DADAM_MIX(2, false, k - first);
      if ((rl.deg - k) & 1) DADAM_MIX(1, false, k - first + ((rl.deg - k) & 2));
    }
  }
#undef DADAM_MIX
}

// HINT: 0 no streaming hints, 1 on every vector access, 2 on all but the loads of sources (rows share
// sources: the second reader must find them in the cache, while gradients, state and all stores still stream).
template <typename XT, typename GT, int PHASE, int U, int CLIP, int HINT, bool EXT, typename A, typename E>
__device__ __forceinline__ void direct_body(const A& a, int position, int row, uint64_t origin, const E (&e)[U], E lo,
                                            E hi, bool full, float wd, int lane) {
  constexpr bool NT = HINT != 0, NTSRC = HINT == 1;
  constexpr int VEC = XT::vec, H = kGroupStep<NT>;
  // The neighbour list sits one entry per lane and is handed out with readlane, which must find a
  // loaded value in whichever lane it asks.  So no lane may leave before the last readlane: a
  // thread of a cut tile whose vectors all lie outside the range runs through the body with its stores (and loads, where
  // they go by elements) masked off instead of returning early.  (With an early return the compiler is
  // free to sink the list's load below it, into the lanes that stay - and a row whose leading
  // lanes lie before the segment then reads its neighbours' indices from lanes that never loaded.)
  RowList rl = load_position_list(a, position, lane);
  MapBytes<VEC, U> map;
  if constexpr (CLIP == kMapped) map = load_map<VEC, U, H>(a, origin, e);
  float g[U][VEC], mh[U][VEC], vh[U][VEC], b[U][VEC];
  load_row_inputs<GT, PHASE, VEC, U, CLIP, NT, EXT>(a, row, origin, e, lo, hi, g, mh, vh, b);
  // Decoupled weight decay acts on the row's own previous parameters, source buffer `row`: kept from the mixing
  // sum where the row lists itself (loading them again would be a second trip to memory after the first).
  const bool decays = !Needs<PHASE>::mixing_only && wd != 0.0f;
  OwnSource<VEC> own;
  own.col = decays ? row : -1;
  float mix[U][VEC];
  mix_direct<XT, U, H, CLIP, NTSRC, EXT>(a, rl, lane, origin, e, lo, hi, mix, own);
  E f[U];
#pragma unroll
  for (int u = 0; u < U; ++u) f[u] = afresh(e[u]);
  uint32_t bits[U];
  if constexpr (CLIP == kMapped) group_bits<VEC, U, H>(map, full, f, lo, hi, bits);
  float xo[U][VEC];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    float decay[VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) decay[j] = 0.0f;
    if (decays) {
      if (!own.found) unpack_raw<XT>(load_raw<XT, H, CLIP, false>(from<XT::bytes>(src_of<EXT>(a, row), origin), f[u], lo, hi), own.x);
#pragma unroll
      for (int j = 0; j < VEC; ++j) decay[j] = decay_of<CLIP>(bits[u], j, wd, own.x[j]);
    }
#pragma unroll
    for (int j = 0; j < VEC; ++j)
      xo[u][j] = element_step<PHASE>(a.s, mix[u][j], g[u][j], mh[u][j], vh[u][j], b[u][j], decay[j]);
  }
  store_vectors<XT, VEC, H, CLIP, NT>(from<XT::bytes>(dst_of<EXT>(a, row), origin), f, lo, hi, bits, xo);
  if constexpr (Needs<PHASE>::acc_out) store_vectors<TF32, VEC, H, CLIP, NT>(from<4>(acc_of<EXT>(a, row), origin), f, lo, hi, bits, b);
  if constexpr (Needs<PHASE>::moments_out) {
    store_vectors<TF32, VEC, H, CLIP, NT>(from<4>(m_hat_of<EXT>(a, row), origin), f, lo, hi, bits, mh);
    store_vectors<TF32, VEC, H, CLIP, NT>(from<4>(v_hat_of<EXT>(a, row), origin), f, lo, hi, bits, vh);
  }
}

// Which piece and row a workgroup takes is the launch's order (see rows_stay_on_one_die).
template <typename XT, typename GT, int PHASE, int HINT, bool EXT, bool MAP, typename A>
__device__ __forceinline__ void direct_entry(const A& a) {
  const int lane = threadIdx.x;
  const uint32_t n_rows = a.n_rows;
  uint32_t t, position;
  bool active = true;
  if (a.order == kOrderDieBlocks) {
    // Rows share sources: a source comes from memory once and from the die's L2 for its other readers, whose turn
    // comes at once or a run of pieces later.
    active = die_block_piece(blockIdx.x, n_rows, a.n_xcd, a.n_pieces, a.xcd_block, t, position, a.die_run);
  } else if (a.order == kOrderDieGroups) {
    // Rows share sources.  Consecutive workgroup ids go to the device's X dies in turn; die x takes the
    // rows at positions [x R / X, (x + 1) R / X) of the sharing order (R = n_rows), tile after tile: the
    // rows that read a source run on one die at about the same time, and the second reader finds the
    // source in that die's L2.  Every die gets G = ceil(R / X) workgroups per tile; where R / X is not whole,
    // the last workgroup of some dies has no row and does nothing (the whole workgroup, so no lane leaves
    // a wavefront early).
    active = die_group_order(blockIdx.x, n_rows, a.n_xcd, a.order_group, t, position);
  } else {
    // Nothing is shared: workgroups in launch order.  (Tile mode's orders were measured here too, on one row with
    // three sources: runs of 2, 4, 8 pieces per die 0.79, 0.77, 0.77 against 0.795, one contiguous X-th of the
    // pieces per die 0.73.)
    t = blockIdx.x / n_rows;
    position = blockIdx.x - t * n_rows;
  }
  const int row = __builtin_amdgcn_readfirstlane(a.row_order[position]);
  const PieceAt p = locate_piece<XT::vec, MAP>(a, t);
  if constexpr (MAP) {
    if (active && p.any) {  // uniform over the workgroup
      const MapTile m = map_tile<XT::vec, 1, HINT != 0>(p.index * (kWave * XT::vec), p.lo, p.hi, lane);
      const uint32_t c[1] = {m.e};
      direct_body<XT, GT, PHASE, 1, kMapped, HINT, EXT>(a, (int)position, row, m.origin, c, m.lo, m.hi, p.full, p.wd, lane);
    }
  } else {
    const uint64_t e[1] = {lane_start<XT::vec, 1, HINT != 0>(p.index, p.lo, p.hi, lane)};
    if (active && p.any) {  // uniform over the workgroup
      constexpr int CUT = HINT == 1 && EXT ? kElements : kGroups;  // see tile_entry
      const int clip = clip_of(a, p.full, p.hi);
      const uint64_t tbase = p.index * (kWave * XT::vec);
      const Cut cut = cut_of<XT::vec, 1, HINT != 0>(tbase, p.lo, p.hi, lane);
      const uint32_t c[1] = {cut.e};
      if (clip == kWhole) direct_body<XT, GT, PHASE, 1, kWhole, HINT, EXT>(a, (int)position, row, 0, e, p.lo, p.hi, p.full, p.wd, lane);
      else if (CUT == kGroups && clip == kGroups && Needs<PHASE>::grad) direct_body<XT, GT, PHASE, 1, CUT, HINT, EXT>(a, (int)position, row, tbase, c, cut.lo, cut.hi, p.full, p.wd, lane);
      else if (CUT == kGroups && clip == kGroups) direct_body<XT, GT, PHASE, 1, CUT, HINT, EXT>(a, (int)position, row, 0, e, p.lo, p.hi, p.full, p.wd, lane);
      else direct_body<XT, GT, PHASE, 1, kElements, HINT, EXT>(a, (int)position, row, 0, e, p.lo, p.hi, p.full, p.wd, lane);
    }
  }
}

// Mixing only, of rows that share sources: a wavefront has little to do for one vector (two or three loads, one store),
// and what bounds the launch is how fast the chip starts workgroups (about 1.7 a nanosecond).  So a workgroup of four
// wavefronts takes a whole work item, two vectors a lane.  With pairs it is then bound by HBM (72 rows, 3e8 elements: 1.33 GB
// read, 1.20 written in 449 us); longer rows fetch a source once for every die that has a reader, and those bytes bound them
// (96 rows of seven sources: 4.84 GB read for 1.20 of sources, 897 us, 6.7 TB/s).  us, two rounds, one-wavefront pieces / this: 72 rows
// in pairs 631 / 465, 96 rows of three sources 608 / 500, 96 replicas of a one-peer graph, one round of each hop, 2030 / 1640.
// Cut items load element by element, here and in k_rows and k_acc_rows: only large launches come here, and those over short
// segments, where cut items are many, mix by the tile (see staging_is_faster).
constexpr int kWideWaves = kDirectItem / 2;
template <typename XT, int HINT, bool EXT>
__global__ __launch_bounds__(kWave* kWideWaves) void k_mix_rows(const StepArgs a) {
  constexpr int VEC = XT::vec;
  constexpr uint64_t PIECE = (uint64_t)kWave * VEC, ITEM = PIECE * kDirectItem;
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t item, position;
  const bool active = die_group_order(blockIdx.x, a.n_rows, a.n_xcd, a.order_group, item, position);
  const int row = __builtin_amdgcn_readfirstlane(a.row_order[position]);
  uint64_t tile_index, lo, hi;
  float wd;
  locate(a, a.work_begin + item, tile_index, lo, hi, wd);
  const uint64_t tbase = tile_index * ITEM;
  if (active) {  // uniform over the workgroup
    const RowList rl = load_position_list(a, (int)position, lane);
    const uint64_t e0 = lane_start<VEC, 2, HINT != 0>(tile_index * kWideWaves + wave, lo, hi, lane);
    const uint64_t e[2] = {e0, e0 + kVectorStep<VEC, HINT != 0>};
    OwnSource<VEC> none;
    none.col = -1;
    float mix[2][VEC];
    void* to = dst_of<EXT>(a, row);
    const uint32_t bits[2] = {};  // of layouts with a map only
    if (tbase >= lo && tbase + ITEM <= hi) {
      mix_direct<XT, 2, kGroupStep<HINT != 0>, kWhole, HINT == 1, EXT>(a, rl, lane, 0, e, lo, hi, mix, none);
      store_vectors<XT, VEC, kGroupStep<HINT != 0>, kWhole, HINT != 0>(to, e, lo, hi, bits, mix);
    } else {
      mix_direct<XT, 2, kGroupStep<HINT != 0>, kElements, HINT == 1, EXT>(a, rl, lane, 0, e, lo, hi, mix, none);
      store_vectors<XT, VEC, kGroupStep<HINT != 0>, kElements, HINT != 0>(to, e, lo, hi, bits, mix);
    }
  }
}

template <typename XT, int HINT, bool EXT>
__global__ __launch_bounds__(kWave* kWideWaves) void k_mix_rows_map(const StepArgs a) {
  constexpr int VEC = XT::vec, H = kGroupStep<HINT != 0>;
  constexpr uint64_t TILE = (uint64_t)kWave * VEC * 2;
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t item, position;
  const bool active = die_group_order(blockIdx.x, a.n_rows, a.n_xcd, a.order_group, item, position);
  const int row = __builtin_amdgcn_readfirstlane(a.row_order[position]);
  uint64_t tile_index, lo, hi;
  float wd;
  locate<true>(a, a.work_begin + item, tile_index, lo, hi, wd);
  const uint64_t tbase = (tile_index * kWideWaves + wave) * TILE;
  if (active && tbase < hi && tbase + TILE > lo) {  // uniform over the wavefront
    const RowList rl = load_position_list(a, (int)position, lane);
    const MapTile t = map_tile<VEC, 2, HINT != 0>(tbase, lo, hi, lane);
    const uint32_t e[2] = {t.e, t.e + kVectorStep<VEC, HINT != 0>};
    const MapBytes<VEC, 2> map = load_map<VEC, 2, H>(a, t.origin, e);
    OwnSource<VEC> none;
    none.col = -1;
    float mix[2][VEC];
    mix_direct<XT, 2, H, kMapped, HINT == 1, EXT>(a, rl, lane, t.origin, e, t.lo, t.hi, mix, none);
    const uint32_t f[2] = {afresh(e[0]), afresh(e[1])};
    uint32_t bits[2];
    group_bits<VEC, 2, H>(map, tbase >= lo && tbase + TILE <= hi, f, t.lo, t.hi, bits);
    store_vectors<XT, VEC, H, kMapped, HINT != 0>(from<XT::bytes>(dst_of<EXT>(a, row), t.origin), f, t.lo, t.hi, bits, mix);
  }
}

// Steps in the same geometry (33 to 63 float32 rows, see whole_items).
template <typename XT, typename GT, int PHASE, int HINT, bool EXT>
__global__ __launch_bounds__(kWave* kWideWaves) void k_rows(const StepArgs a) {
  constexpr int VEC = XT::vec;
  constexpr uint64_t PIECE = (uint64_t)kWave * VEC, ITEM = PIECE * kDirectItem;
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t item, position;
  const bool active = die_group_order(blockIdx.x, a.n_rows, a.n_xcd, a.order_group, item, position);
  const int row = __builtin_amdgcn_readfirstlane(a.row_order[position]);
  uint64_t tile_index, lo, hi;
  float wd;
  locate(a, a.work_begin + item, tile_index, lo, hi, wd);
  const uint64_t tbase = tile_index * ITEM;
  const uint64_t e0 = lane_start<VEC, 2, HINT != 0>(tile_index * kWideWaves + wave, lo, hi, lane);
  const uint64_t e[2] = {e0, e0 + kVectorStep<VEC, HINT != 0>};
  if (active) {  // uniform over the workgroup
    if (tbase >= lo && tbase + ITEM <= hi) direct_body<XT, GT, PHASE, 2, kWhole, HINT, EXT>(a, (int)position, row, 0, e, lo, hi, true, wd, lane);
    else direct_body<XT, GT, PHASE, 2, kElements, HINT, EXT>(a, (int)position, row, 0, e, lo, hi, true, wd, lane);
  }
}

// ---------------------------------------------------------------------------------------------
// loops: groups of rows that list the same sources with the same weights
// ---------------------------------------------------------------------------------------------
// The rows of an All-Reduce loop (the complete graph; the loops of the alternating exponential ring) share one
// neighbour sum.  A workgroup takes one piece of one loop: its wavefronts share out the loop's sources, three or more
// each, each sums its own straight from memory, the partial sums (one vector per lane and wavefront) meet in LDS, and after one
// barrier the wavefronts deal the loop's rows among themselves.  Every source is read once and summed once, where
// the tile kernel sums it once per row from a staged copy.  What that costs there: 64 rows of 64 sources read 64 x
// the tile from LDS, and beyond 80 sources a CU holds one workgroup of the tile, whose phases nothing overlaps.
// Where loops have many rows, a.loop_shares workgroups take the rows of one tile between them (see loop_shares): each sums the sources
// for itself, in the same order, and in streaming launches the loads of sources carry no hint, so that the second finds them in its die's L2.
// All sources of the loop are read before the barrier and its rows written after it.  Bound by HBM: the bytes moved are
// those needed (96 rows in loops of 48 and 24, 2e8 elements: 4.0 GB read and 1.6 written in 1062 us, 5.3 TB/s); measured against the other kernels in loop_kernel_waves (mixing 64 sources 0.19 -> 0.69 of 8 TB/s, 96 in loops
// of 48 and 24 0.14 -> 0.69, the step on those 0.34 -> 0.71).
template <typename XT, typename GT, int PHASE, int CLIP, int HINT, bool EXT, typename A, typename E>
__device__ __forceinline__ void loop_body(const A& a, f4* lds, int loop, int share, uint64_t origin, E start, E lo, E hi, bool full, float wd, int lane,
                                          int wave, int waves) {
  constexpr bool NT = HINT != 0;
  constexpr int VEC = XT::vec, H = kGroupStep<NT>;
  const E e[1] = {start};
  MapBytes<VEC, 1> map;
  if constexpr (CLIP == kMapped) map = load_map<VEC, 1, H>(a, origin, e);
  const Loop l = a.loops[loop];
  // This wavefront's rows, every `row_step`-th of the loop's, and sources, every `parts`-th, one per lane (at most 160 / 8 of
  // each).  A wavefront that sums has at least three sources, so that the sum is never less accurate than the listed
  // order: a partial sum starts with a rounded product and is added with a rounded sum, where the chain of fused
  // multiply-adds rounds once.  Mean error against 64 bits, relative to that chain, 3 / 9 / 13 / 20 sources of
  // independent values and unequal weights: one wavefront a source 1.39 / 1.13 / 1.09 / 1.02, as it is 1 / 0.89 / 0.82 / 0.76.
  const int parts = l.n_entries < 6 ? 1 : l.n_entries / 3 < waves ? l.n_entries / 3 : waves;
  RowList rl;
  rl.k0 = 0;
  rl.deg = wave < parts ? (l.n_entries - wave + parts - 1) / parts : 0;
  const int first_row = share * waves + wave, row_step = (int)a.loop_shares * waves;
  const int my_rows = first_row < l.n_rows ? (l.n_rows - first_row + row_step - 1) / row_step : 0;
  const int entry = l.first_entry + (lane < rl.deg ? wave + lane * parts : 0);
  rl.col_v = a.col[entry];
  rl.w_v = a.w[entry];
  const int row_v = a.row_order[l.first_row + (lane < my_rows ? first_row + lane * row_step : 0)];
  float g[1][VEC], mh[1][VEC], vh[1][VEC], b[1][VEC];
  int row = __builtin_amdgcn_readlane(row_v, 0);
  if (my_rows > 0) load_row_inputs<GT, PHASE, VEC, 1, CLIP, NT, EXT>(a, row, origin, e, lo, hi, g, mh, vh, b);
  if (rl.deg > 0) {
    float part[1][VEC];
    OwnSource<VEC> none;
    none.col = -1;
    mix_direct<XT, 1, H, CLIP, HINT == 1, EXT>(a, rl, lane, origin, e, lo, hi, part, none);
#pragma unroll
    for (int h = 0; h < VEC / 4; ++h) {
      f4 v = {part[0][4 * h], part[0][4 * h + 1], part[0][4 * h + 2], part[0][4 * h + 3]};
      lds[(wave * (VEC / 4) + h) * kWave + lane] = v;
    }
  }
  __syncthreads();
  uint32_t bits[1];
  if constexpr (CLIP == kMapped) group_bits<VEC, 1, H>(map, full, e, lo, hi, bits);
  float mix[VEC];
  for (int p = 0; p < parts; ++p)
#pragma unroll
    for (int h = 0; h < VEC / 4; ++h) {
      const f4 v = lds[(p * (VEC / 4) + h) * kWave + lane];
#pragma unroll
      for (int j = 0; j < 4; ++j) mix[4 * h + j] = p == 0 ? v[j] : mix[4 * h + j] + v[j];
    }
  for (int r = 0; r < my_rows; ++r) {
    float decay[VEC], xo[1][VEC];
#pragma unroll
    for (int j = 0; j < VEC; ++j) decay[j] = 0.0f;
    if (!Needs<PHASE>::mixing_only && wd != 0.0f) {
      float own[VEC];
      unpack_raw<XT>(load_raw<XT, H, CLIP, false>(from<XT::bytes>(src_of<EXT>(a, row), origin), e[0], lo, hi), own);
#pragma unroll
      for (int j = 0; j < VEC; ++j) decay[j] = decay_of<CLIP>(bits[0], j, wd, own[j]);
    }
#pragma unroll
    for (int j = 0; j < VEC; ++j) xo[0][j] = element_step<PHASE>(a.s, mix[j], g[0][j], mh[0][j], vh[0][j], b[0][j], decay[j]);
    store_vectors<XT, VEC, H, CLIP, NT>(from<XT::bytes>(dst_of<EXT>(a, row), origin), e, lo, hi, bits, xo);
    if constexpr (Needs<PHASE>::acc_out) store_vectors<TF32, VEC, H, CLIP, NT>(from<4>(acc_of<EXT>(a, row), origin), e, lo, hi, bits, b);
    if constexpr (Needs<PHASE>::moments_out) {
      store_vectors<TF32, VEC, H, CLIP, NT>(from<4>(m_hat_of<EXT>(a, row), origin), e, lo, hi, bits, mh);
      store_vectors<TF32, VEC, H, CLIP, NT>(from<4>(v_hat_of<EXT>(a, row), origin), e, lo, hi, bits, vh);
    }
    if (r + 1 < my_rows) {
      row = __builtin_amdgcn_readlane(row_v, r + 1);
      load_row_inputs<GT, PHASE, VEC, 1, CLIP, NT, EXT>(a, row, origin, e, lo, hi, g, mh, vh, b);
    }
  }
}

// Workgroup b of a loop launch.  A launch is a chain of trips to memory, so a division that only shared tiles need is made for those alone (mixing
// of 32 to 64 rows, 300 tiles, 6.6 to 9.5 us, took 0.2 to 0.3 more with it).
struct LoopUnit {
  uint32_t tile;
  int share, loop;
};
__device__ __forceinline__ LoopUnit loop_unit(uint32_t b, uint32_t n_loops, uint32_t shares) {
  const uint32_t part = b / n_loops;
  LoopUnit u = {part, 0, (int)(b - part * n_loops)};
  if (shares > 1) {
    u.tile = part / shares;
    u.share = (int)(part - u.tile * shares);
  }
  return u;
}
template <typename XT, typename GT, int PHASE, int HINT, bool EXT>
__global__ __launch_bounds__(kWave* kMaxLoopWaves) void k_loop(const StepArgs a) {
  constexpr uint64_t TILE = (uint64_t)kWave * XT::vec;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_bytes[];
  f4* lds = reinterpret_cast<f4*>(lds_bytes);
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  // the dies take runs of tiles in turn, all shares and loops of a tile one after the other (see k_tile).  Streaming launches: runs of two
  // tiles (kDieBlockLoops), because every tile of several loops is many streams: 96 rows in loops of 48 and 24, runs of
  // 1, 2, 4, 8, 32, 256 tiles 0.80, 0.81, 0.80, 0.80, 0.76, 0.76 of 8 TB/s; one loop of 64 rows the same with all of them.
  const uint32_t units = a.n_loops * a.loop_shares, b = die_block_order(blockIdx.x, gridDim.x, a.n_xcd, a.xcd_block * units);
  const auto [tile, share, loop] = loop_unit(b, a.n_loops, a.loop_shares);
  uint64_t tile_index, lo, hi;
  float wd;
  locate(a, a.work_begin + begin_with_last<HINT != 0 && EXT>(tile, gridDim.x / units), tile_index, lo, hi, wd);
  const uint64_t tbase = tile_index * TILE;
  const bool full = tbase >= lo && tbase + TILE <= hi;
  const int waves = (int)(blockDim.x / kWave);
  const uint64_t start = lane_start<XT::vec, 1, HINT != 0>(tile_index, lo, hi, lane);
  constexpr int CUT = HINT != 0 && EXT ? kElements : kGroups;  // see tile_entry
  const int clip = clip_of(a, full, hi);
  const Cut cut = cut_of<XT::vec, 1, HINT != 0>(tbase, lo, hi, lane);
  if (clip == kWhole) loop_body<XT, GT, PHASE, kWhole, HINT, EXT>(a, lds, loop, share, 0, start, lo, hi, full, wd, lane, wave, waves);
  else if (CUT == kGroups && clip == kGroups && Needs<PHASE>::grad) loop_body<XT, GT, PHASE, CUT, HINT, EXT>(a, lds, loop, share, tbase, cut.e, cut.lo, cut.hi, full, wd, lane, wave, waves);
  else if (CUT == kGroups && clip == kGroups) loop_body<XT, GT, PHASE, CUT, HINT, EXT>(a, lds, loop, share, 0, start, lo, hi, full, wd, lane, wave, waves);
  else loop_body<XT, GT, PHASE, kElements, HINT, EXT>(a, lds, loop, share, 0, start, lo, hi, full, wd, lane, wave, waves);
}
template <typename XT, typename GT, int PHASE, int HINT, bool EXT>
__global__ __launch_bounds__(kWave* kMaxLoopWaves) void k_loop_map(const StepArgs a) {
  constexpr uint64_t TILE = (uint64_t)kWave * XT::vec;
  extern __shared__ __attribute__((aligned(16))) unsigned char lds_bytes[];
  const int lane = threadIdx.x & (kWave - 1);
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t units = a.n_loops * a.loop_shares, b = die_block_order(blockIdx.x, gridDim.x, a.n_xcd, a.xcd_block * units);
  const auto [tile, share, loop] = loop_unit(b, a.n_loops, a.loop_shares);
  uint64_t tile_index, lo, hi;
  float wd;
  locate<true>(a, a.work_begin + tile, tile_index, lo, hi, wd);
  const uint64_t tbase = tile_index * TILE;
  const bool full = tbase >= lo && tbase + TILE <= hi;
  const MapTile t = map_tile<XT::vec, 1, HINT != 0>(tbase, lo, hi, lane);
  loop_body<XT, GT, PHASE, kMapped, HINT, EXT>(a, reinterpret_cast<f4*>(lds_bytes), loop, share, t.origin, t.e, t.lo, t.hi,
                                               full, wd, lane, wave, (int)(blockDim.x / kWave));
}

// ---------------------------------------------------------------------------------------------
// accumulate / fold only (Algorithm 3 lines 9-13).  Walks the direct kernel's grid in the same pieces, so a lane
// vector has as many elements as a parameter vector of the handle (4 or 8).
// ---------------------------------------------------------------------------------------------
template <int PHASE>
__device__ __forceinline__ void acc_step(const Scalars& s, float g, float& mh, float& vh, float& b) {
  if constexpr (PHASE == kPlain || PHASE == kFold) b = fmaf(g, s.inv_s, b);
  if constexpr (PHASE == kLoopStart || PHASE == kAlg1) b = g * s.inv_s;
  if constexpr (PHASE == kFold || PHASE == kAlg1) {
    mh = fmaf(s.beta1, mh, s.omb1 * b);
    vh = fmaf(s.betav, vh, s.ombv * (b * b));
    b = 0.0f;
  }
}

template <typename GT, int VEC, int PHASE, int U, int CLIP, bool NT, bool EXT, typename A>
__device__ __forceinline__ void acc_body(const A& a, int row, const uint64_t (&e)[U], uint64_t lo, uint64_t hi, bool full) {
  constexpr int H = kGroupStep<NT>;
  MapBytes<VEC, U> map;
  if constexpr (CLIP == kMapped) map = load_map<VEC, U, H>(a, 0, e);
  float g[U][VEC], mh[U][VEC], vh[U][VEC], b[U][VEC];
#pragma unroll
  for (int u = 0; u < U; ++u) load_vals<GT, VEC, H, CLIP, NT>(a.grad[row], e[u], lo, hi, g[u]);
  if constexpr (Needs<PHASE>::moments_out) {
#pragma unroll
    for (int u = 0; u < U; ++u) load_vals<TF32, VEC, H, CLIP, NT>(m_hat_of<EXT>(a, row), e[u], lo, hi, mh[u]);
#pragma unroll
    for (int u = 0; u < U; ++u) load_vals<TF32, VEC, H, CLIP, NT>(v_hat_of<EXT>(a, row), e[u], lo, hi, vh[u]);
  }
  if constexpr (Needs<PHASE>::acc_in) {
#pragma unroll
    for (int u = 0; u < U; ++u) load_vals<TF32, VEC, H, CLIP, NT>(acc_of<EXT>(a, row), e[u], lo, hi, b[u]);
  }
#pragma unroll
  for (int u = 0; u < U; ++u)
#pragma unroll
    for (int j = 0; j < VEC; ++j) acc_step<PHASE>(a.s, g[u][j], mh[u][j], vh[u][j], b[u][j]);
  uint32_t bits[U];
  if constexpr (CLIP == kMapped) group_bits<VEC, U, H>(map, full, e, lo, hi, bits);
  if constexpr (Needs<PHASE>::acc_out) store_vectors<TF32, VEC, H, CLIP, NT>(acc_of<EXT>(a, row), e, lo, hi, bits, b);
  if constexpr (Needs<PHASE>::moments_out) {
    store_vectors<TF32, VEC, H, CLIP, NT>(m_hat_of<EXT>(a, row), e, lo, hi, bits, mh);
    store_vectors<TF32, VEC, H, CLIP, NT>(v_hat_of<EXT>(a, row), e, lo, hi, bits, vh);
  }
}

// VEC is the element count of a parameter vector of this handle, so that the accumulate kernel walks the
// same grid as the direct kernel.
template <typename GT, int VEC, int PHASE, bool NT, bool EXT, bool MAP, typename A>
__device__ __forceinline__ void acc_entry(const A& a) {
  const uint32_t n_rows = a.n_rows;
  uint32_t t, row_at;
  bool active = true;
  if (a.order == kOrderDieBlocks) {
    active = die_block_piece(blockIdx.x, n_rows, a.n_xcd, a.n_pieces, a.xcd_block, t, row_at, a.die_run);
  } else {
    t = blockIdx.x / n_rows;
    row_at = blockIdx.x - t * n_rows;
  }
  const int row = (int)row_at;
  const PieceAt p = locate_piece<VEC, MAP>(a, t);
  const uint64_t e[1] = {lane_start<VEC, 1, NT>(p.index, p.lo, p.hi, (int)threadIdx.x)};
  if (active && p.any) {
    constexpr int CUT = NT && EXT ? kElements : kGroups;  // see tile_entry
    const int clip = clip_of(a, p.full, p.hi);
    if constexpr (MAP) acc_body<GT, VEC, PHASE, 1, kMapped, NT, EXT>(a, row, e, p.lo, p.hi, p.full);
    else if (clip == kWhole) acc_body<GT, VEC, PHASE, 1, kWhole, NT, EXT>(a, row, e, p.lo, p.hi, p.full);
    else if (CUT == kGroups && clip == kGroups) acc_body<GT, VEC, PHASE, 1, CUT, NT, EXT>(a, row, e, p.lo, p.hi, p.full);
    else acc_body<GT, VEC, PHASE, 1, kElements, NT, EXT>(a, row, e, p.lo, p.hi, p.full);
  }
}

// The same, whole items by four wavefronts, two vectors a lane (see accumulate_whole_items).
template <typename GT, int VEC, int PHASE, bool NT, bool EXT>
__global__ __launch_bounds__(kWave* kWideWaves) void k_acc_rows(const StepArgs a) {
  constexpr uint64_t PIECE = (uint64_t)kWave * VEC, ITEM = PIECE * kDirectItem;
  const int lane = threadIdx.x & (kWave - 1);
  const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t item, row_at;
  bool active = true;
  if (a.order == kOrderDieBlocks) {
    active = die_block_piece(blockIdx.x, a.n_rows, a.n_xcd, a.n_pieces, a.xcd_block, item, row_at, a.die_run);
  } else {
    item = blockIdx.x / a.n_rows;
    row_at = blockIdx.x - item * a.n_rows;
  }
  const int row = (int)row_at;
  uint64_t tile_index, lo, hi;
  float wd;
  locate(a, a.work_begin + item, tile_index, lo, hi, wd);
  const uint64_t tbase = tile_index * ITEM;
  const uint64_t e0 = lane_start<VEC, 2, NT>(tile_index * kWideWaves + wave, lo, hi, lane);
  const uint64_t e[2] = {e0, e0 + kVectorStep<VEC, NT>};
  if (active) {  // uniform over the workgroup
    if (tbase >= lo && tbase + ITEM <= hi) acc_body<GT, VEC, PHASE, 2, kWhole, NT, EXT>(a, row, e, lo, hi, true);
    else acc_body<GT, VEC, PHASE, 2, kElements, NT, EXT>(a, row, e, lo, hi, true);
  }
}

// ---------------------------------------------------------------------------------------------
// the kernels
// ---------------------------------------------------------------------------------------------
// Of each a second one, _map, for layouts with a map (see StepArgsFor::map): one body instead of three.
template <typename XT, typename GT, int PHASE, int W, int UT, bool NT, bool EXT>
__global__ __launch_bounds__(kWave* W) void k_tile(const StepArgs a) {
  tile_entry<XT, GT, PHASE, W, UT, NT, EXT, false>(a);
}
template <typename XT, typename GT, int PHASE, int W, int UT, bool NT, bool EXT>
__global__ __launch_bounds__(kWave* W) void k_tile_map(const StepArgs a) {
  tile_entry<XT, GT, PHASE, W, UT, NT, EXT, true>(a);
}
template <typename XT, typename GT, int PHASE, int HINT, bool EXT>
__global__ __launch_bounds__(kWave) void k_direct(const StepArgs a) {
  direct_entry<XT, GT, PHASE, HINT, EXT, false>(a);
}
template <typename XT, typename GT, int PHASE, int HINT, bool EXT>
__global__ __launch_bounds__(kWave) void k_direct_map(const StepArgs a) {
  direct_entry<XT, GT, PHASE, HINT, EXT, true>(a);
}
template <typename GT, int VEC, int PHASE, bool NT, bool EXT>
__global__ __launch_bounds__(kWave) void k_acc(const StepArgs a) {
  acc_entry<GT, VEC, PHASE, NT, EXT, false>(a);
}
template <typename GT, int VEC, int PHASE, bool NT, bool EXT>
__global__ __launch_bounds__(kWave) void k_acc_map(const StepArgs a) {
  acc_entry<GT, VEC, PHASE, NT, EXT, true>(a);
}
// The same on the short argument block (small handles: no streaming hints, tables in the block).
template <typename XT, typename GT, int PHASE, int W, int UT>
__global__ __launch_bounds__(kWave* W) void k_tile_few(const StepArgsFew a) {
  tile_entry<XT, GT, PHASE, W, UT, false, false, false>(a);
}
template <typename XT, typename GT, int PHASE, int W, int UT>
__global__ __launch_bounds__(kWave* W) void k_tile_few_map(const StepArgsFew a) {
  tile_entry<XT, GT, PHASE, W, UT, false, false, true>(a);
}
template <typename XT, typename GT, int PHASE>
__global__ __launch_bounds__(kWave) void k_direct_few(const StepArgsFew a) {
  direct_entry<XT, GT, PHASE, 0, false, false>(a);
}
template <typename XT, typename GT, int PHASE>
__global__ __launch_bounds__(kWave) void k_direct_few_map(const StepArgsFew a) {
  direct_entry<XT, GT, PHASE, 0, false, true>(a);
}
template <typename GT, int VEC, int PHASE>
__global__ __launch_bounds__(kWave) void k_acc_few(const StepArgsFew a) {
  acc_entry<GT, VEC, PHASE, false, false, false>(a);
}
template <typename GT, int VEC, int PHASE>
__global__ __launch_bounds__(kWave) void k_acc_few_map(const StepArgsFew a) {
  acc_entry<GT, VEC, PHASE, false, false, true>(a);
}

// ---------------------------------------------------------------------------------------------
// dispatch tables
// ---------------------------------------------------------------------------------------------

template <typename XT, typename GT, int W, int UT, bool NT, bool EXT>
KernelFn tile_kernel_for_phase(int phase, bool map) {
  switch (phase) {
    case kMixOnly: return map ? (KernelFn)k_tile_map<XT, GT, kMixOnly, W, UT, NT, EXT> : (KernelFn)k_tile<XT, GT, kMixOnly, W, UT, NT, EXT>;
    case kMixConsensus: return map ? (KernelFn)k_tile_map<XT, GT, kMixConsensus, W, UT, NT, EXT> : (KernelFn)k_tile<XT, GT, kMixConsensus, W, UT, NT, EXT>;
    case kUpdateOnly: return map ? (KernelFn)k_tile_map<XT, GT, kUpdateOnly, W, UT, NT, EXT> : (KernelFn)k_tile<XT, GT, kUpdateOnly, W, UT, NT, EXT>;
    case kPlain: return map ? (KernelFn)k_tile_map<XT, GT, kPlain, W, UT, NT, EXT> : (KernelFn)k_tile<XT, GT, kPlain, W, UT, NT, EXT>;
    case kLoopStart: return map ? (KernelFn)k_tile_map<XT, GT, kLoopStart, W, UT, NT, EXT> : (KernelFn)k_tile<XT, GT, kLoopStart, W, UT, NT, EXT>;
    case kFold: return map ? (KernelFn)k_tile_map<XT, GT, kFold, W, UT, NT, EXT> : (KernelFn)k_tile<XT, GT, kFold, W, UT, NT, EXT>;
    case kAlg1: return map ? (KernelFn)k_tile_map<XT, GT, kAlg1, W, UT, NT, EXT> : (KernelFn)k_tile<XT, GT, kAlg1, W, UT, NT, EXT>;
  }
  return nullptr;
}

template <typename XT, typename GT, int W, int UT>
KernelFn few_tile_kernel_for_phase(int phase, bool map) {
  switch (phase) {
    case kMixOnly: return map ? (KernelFn)k_tile_few_map<XT, GT, kMixOnly, W, UT> : (KernelFn)k_tile_few<XT, GT, kMixOnly, W, UT>;
    case kMixConsensus: return map ? (KernelFn)k_tile_few_map<XT, GT, kMixConsensus, W, UT> : (KernelFn)k_tile_few<XT, GT, kMixConsensus, W, UT>;
    case kUpdateOnly: return map ? (KernelFn)k_tile_few_map<XT, GT, kUpdateOnly, W, UT> : (KernelFn)k_tile_few<XT, GT, kUpdateOnly, W, UT>;
    case kPlain: return map ? (KernelFn)k_tile_few_map<XT, GT, kPlain, W, UT> : (KernelFn)k_tile_few<XT, GT, kPlain, W, UT>;
    case kLoopStart: return map ? (KernelFn)k_tile_few_map<XT, GT, kLoopStart, W, UT> : (KernelFn)k_tile_few<XT, GT, kLoopStart, W, UT>;
    case kFold: return map ? (KernelFn)k_tile_few_map<XT, GT, kFold, W, UT> : (KernelFn)k_tile_few<XT, GT, kFold, W, UT>;
    case kAlg1: return map ? (KernelFn)k_tile_few_map<XT, GT, kAlg1, W, UT> : (KernelFn)k_tile_few<XT, GT, kAlg1, W, UT>;
  }
  return nullptr;
}
template <typename XT, typename GT>
KernelFn few_tile_kernel(int phase, TileShape s, bool map) {
  if (s.waves == 4 && s.ut == 1) return few_tile_kernel_for_phase<XT, GT, 4, 1>(phase, map);
  if (s.waves == 4 && s.ut == 2) return few_tile_kernel_for_phase<XT, GT, 4, 2>(phase, map);
  if (s.waves == 8 && s.ut == 1) return few_tile_kernel_for_phase<XT, GT, 8, 1>(phase, map);
  return nullptr;  // no handle of few rows has another shape
}
template <typename XT, typename GT>
KernelFn few_direct_kernel(int phase, bool map) {
  switch (phase) {
    case kMixOnly: return map ? (KernelFn)k_direct_few_map<XT, GT, kMixOnly> : (KernelFn)k_direct_few<XT, GT, kMixOnly>;
    case kUpdateOnly: return map ? (KernelFn)k_direct_few_map<XT, GT, kUpdateOnly> : (KernelFn)k_direct_few<XT, GT, kUpdateOnly>;
    case kPlain: return map ? (KernelFn)k_direct_few_map<XT, GT, kPlain> : (KernelFn)k_direct_few<XT, GT, kPlain>;
    case kLoopStart: return map ? (KernelFn)k_direct_few_map<XT, GT, kLoopStart> : (KernelFn)k_direct_few<XT, GT, kLoopStart>;
    case kFold: return map ? (KernelFn)k_direct_few_map<XT, GT, kFold> : (KernelFn)k_direct_few<XT, GT, kFold>;
    case kAlg1: return map ? (KernelFn)k_direct_few_map<XT, GT, kAlg1> : (KernelFn)k_direct_few<XT, GT, kAlg1>;
  }
  return nullptr;
}

template <typename XT, typename GT, bool NT, bool EXT>
KernelFn tile_kernel_for_shape_nt(int phase, TileShape s, bool map) {
  if (s.waves == 4 && s.ut == 1) return tile_kernel_for_phase<XT, GT, 4, 1, NT, EXT>(phase, map);
  if (s.waves == 4 && s.ut == 2) return tile_kernel_for_phase<XT, GT, 4, 2, NT, EXT>(phase, map);
  if (s.waves == 8 && s.ut == 1) return tile_kernel_for_phase<XT, GT, 8, 1, NT, EXT>(phase, map);
  if constexpr (NT && XT::vec == 4) {
    if (s.waves == 8 && s.ut == 2) return tile_kernel_for_phase<XT, GT, 8, 2, NT, EXT>(phase, map);
    if (s.waves == 16 && s.ut == 2) return tile_kernel_for_phase<XT, GT, 16, 2, NT, EXT>(phase, map);
  }
  if constexpr (EXT)
    if (s.waves == 16 && s.ut == 1) return tile_kernel_for_phase<XT, GT, 16, 1, NT, EXT>(phase, map);
  return nullptr;
}
template <typename XT, typename GT, int HINT, bool EXT>
KernelFn loop_kernel_for_phase(int phase, bool map) {
  if constexpr (HINT != 2)  // streaming mixing has no shares: loop_shares gives it one workgroup a tile
    if (phase == kMixOnly) return map ? (KernelFn)k_loop_map<XT, GT, kMixOnly, HINT, EXT> : (KernelFn)k_loop<XT, GT, kMixOnly, HINT, EXT>;
  switch (phase) {
    case kUpdateOnly: return map ? (KernelFn)k_loop_map<XT, GT, kUpdateOnly, HINT, EXT> : (KernelFn)k_loop<XT, GT, kUpdateOnly, HINT, EXT>;
    case kPlain: return map ? (KernelFn)k_loop_map<XT, GT, kPlain, HINT, EXT> : (KernelFn)k_loop<XT, GT, kPlain, HINT, EXT>;
    case kLoopStart: return map ? (KernelFn)k_loop_map<XT, GT, kLoopStart, HINT, EXT> : (KernelFn)k_loop<XT, GT, kLoopStart, HINT, EXT>;
    case kFold: return map ? (KernelFn)k_loop_map<XT, GT, kFold, HINT, EXT> : (KernelFn)k_loop<XT, GT, kFold, HINT, EXT>;
    case kAlg1: return map ? (KernelFn)k_loop_map<XT, GT, kAlg1, HINT, EXT> : (KernelFn)k_loop<XT, GT, kAlg1, HINT, EXT>;
  }
  return nullptr;
}
template <typename XT, typename GT, int HINT, bool EXT>
KernelFn direct_kernel_for_phase(int phase, bool map) {
  switch (phase) {
    case kMixOnly: return map ? (KernelFn)k_direct_map<XT, GT, kMixOnly, HINT, EXT> : (KernelFn)k_direct<XT, GT, kMixOnly, HINT, EXT>;
    case kUpdateOnly: return map ? (KernelFn)k_direct_map<XT, GT, kUpdateOnly, HINT, EXT> : (KernelFn)k_direct<XT, GT, kUpdateOnly, HINT, EXT>;
    case kPlain: return map ? (KernelFn)k_direct_map<XT, GT, kPlain, HINT, EXT> : (KernelFn)k_direct<XT, GT, kPlain, HINT, EXT>;
    case kLoopStart: return map ? (KernelFn)k_direct_map<XT, GT, kLoopStart, HINT, EXT> : (KernelFn)k_direct<XT, GT, kLoopStart, HINT, EXT>;
    case kFold: return map ? (KernelFn)k_direct_map<XT, GT, kFold, HINT, EXT> : (KernelFn)k_direct<XT, GT, kFold, HINT, EXT>;
    case kAlg1: return map ? (KernelFn)k_direct_map<XT, GT, kAlg1, HINT, EXT> : (KernelFn)k_direct<XT, GT, kAlg1, HINT, EXT>;
  }
  return nullptr;
}
// Whole items by four wavefronts: mixing (no gradient: built once per parameter type), and the large float32 steps that
// the host gives it (streaming, tables in the argument block).
template <typename XT, typename GT, int HINT, bool EXT>
KernelFn rows_kernel_for_phase(int phase, bool map) {
  if constexpr (XT::bytes == GT::bytes)
    if (phase == kMixOnly) return map ? (KernelFn)k_mix_rows_map<XT, HINT, EXT> : (KernelFn)k_mix_rows<XT, HINT, EXT>;
  if constexpr (XT::bytes == 4 && HINT == 2 && !EXT) switch (phase) {
    case kUpdateOnly: return (KernelFn)k_rows<XT, GT, kUpdateOnly, HINT, EXT>;
    case kPlain: return (KernelFn)k_rows<XT, GT, kPlain, HINT, EXT>;
    case kLoopStart: return (KernelFn)k_rows<XT, GT, kLoopStart, HINT, EXT>;
    case kFold: return (KernelFn)k_rows<XT, GT, kFold, HINT, EXT>;
    case kAlg1: return (KernelFn)k_rows<XT, GT, kAlg1, HINT, EXT>;
  }
  return nullptr;
}

}  // namespace
}  // namespace dadam

#endif  // DADAM_DEVICE_H_
