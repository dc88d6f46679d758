// The map of layouts of short segments and what the kernels make of it, compiled for the host from the sources' own text under
// the address sanitizer: which layouts get one (can_map), and that over the tiles of a launch every element of the range that
// belongs to a tensor is stored once, with the tensor's decay, everything else never, by loads that stay inside the buffer.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <random>
#include <vector>
#define __device__
#define __forceinline__ inline
static inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
constexpr int kWave = 64;
constexpr uint32_t kLongSegment = 65536, kWidestGap = 7;
constexpr uint64_t kMostMapped = 1ull << 28;
struct Segment { uint64_t lo, hi; float weight_decay; };
struct dadam_handle {
  struct { uint64_t d; } cfg;
  std::vector<Segment> segs;
  bool short_segments = true;
};
namespace emu {
#include "helpers.inc"
#include "clip.inc"
#include "host.inc"
}
using namespace emu;
struct Args { uint64_t d; const uint8_t* map; };
static long bad = 0, spread = 0, partial = 0;

template <int VEC, int U, bool STREAM>
void tiles(const dadam_handle& h, const std::vector<uint8_t>& map, const std::vector<int>& want, uint64_t lo, uint64_t hi) {
  constexpr uint64_t N = (uint64_t)kWave * VEC * U;
  constexpr int H = kGroupStep<STREAM>;
  const Args a{h.cfg.d, map.data()};
  std::vector<int> got(h.cfg.d, 0);
  const std::vector<float> data(h.cfg.d, 1.0f);
  for (uint64_t t = lo / N; t <= (hi - 1) / N; ++t) {
    const bool full = t * N >= lo && t * N + N <= hi;
    for (int lane = 0; lane < kWave; ++lane) {
      const uint64_t start = lane_start<VEC, U, STREAM>(t, lo, hi, lane);
      const MapTile c = map_tile<VEC, U, STREAM>(t * N, lo, hi, lane);
      spread += c.origin != t * N;
      uint32_t e[U], bits[U];
      uint64_t f[U];
      uint32_t wide[U];
      for (int u = 0; u < U; ++u) { e[u] = c.e + u * kVectorStep<VEC, STREAM>; f[u] = start + u * kVectorStep<VEC, STREAM>; }
      const MapBytes<VEC, U> bytes = load_map<VEC, U, H>(a, c.origin, e);
      group_bits<VEC, U, H>(bytes, full, e, c.lo, c.hi, bits);
      group_bits<VEC, U, H>(load_map<VEC, U, H>(a, 0, f), full, f, lo, hi, wide);
      for (int u = 0; u < U; ++u) {
        bad += bits[u] != wide[u];  // indexes of the buffer and of the tile agree
        float v[VEC];
        load_vals<TF32, VEC, H, kMapped, true>(data.data() + c.origin, e[u], c.lo, c.hi, v);
        for (int j = 0; j < VEC; ++j) {
          const uint32_t b = bits[u] >> (8 * (j / 4));
          const uint64_t at = f[u] + (uint64_t)(j / 4) * H + j % 4;
          partial += j % 4 == 0 && (b & kStoreBits) != 0 && (b & kStoreBits) != kStoreBits;
          if (b >> (j % 4) & 1) {
            if (at >= h.cfg.d) { ++bad; continue; }
            got[at] += b & kDecayBit ? 2 : 1;
            bad += got[at] > 2 || v[j] != 1.0f;
          }
        }
      }
    }
  }
  for (uint64_t i = 0; i < h.cfg.d; ++i) bad += got[i] != (i >= lo && i < hi ? want[i] : 0);
}

static bool mapped(std::vector<Segment> segs, uint64_t d, bool short_segments = true) {
  dadam_handle h;
  h.cfg.d = d;
  h.segs = std::move(segs);
  h.short_segments = short_segments;
  float decay;
  return can_map(&h, &decay);
}

int main() {
  std::mt19937 rng(7);
  auto below = [&](uint32_t n) { return (uint32_t)(rng() % n); };
  for (int trial = 0; trial < 60; ++trial) {
    dadam_handle h;
    std::vector<uint64_t> edges;
    const bool packed = trial % 3 == 0;  // to multiples of 8, or gaps of 0 to 7 anywhere
    uint64_t at = trial % 4 == 1 ? below(90) : 0;
    const uint64_t most = trial % 5 == 4 ? 80000 : 4000;
    while (at < most) {
      const bool decays = trial % 2 && below(2);
      const uint64_t n = 1 + below(trial % 7 == 3 ? 9 : 1500);
      h.segs.push_back({at, at + n, decays ? 0.1f : 0.0f});
      edges.push_back(at);
      edges.push_back(at + n);
      at += n;
      at = packed ? (at + 7) / 8 * 8 : at + below(8);
      // a group of four has one decay
      if (!packed && trial % 2) at = std::max(at, (h.segs.back().hi + 3) / 4 * 4);
    }
    h.cfg.d = (at + 3) / 4 * 4 + 4 * below(40);
    float decay = -1.f;
    if (!can_map(&h, &decay)) { ++bad; continue; }
    const std::vector<uint8_t> map = build_map(&h);
    std::vector<int> want(h.cfg.d, 0);
    for (const Segment& s : h.segs) for (uint64_t i = s.lo; i < s.hi; ++i) want[i] = s.weight_decay != 0.f ? 2 : 1;
    for (int range = 0; range < 4; ++range) {
      uint64_t lo = h.segs.front().lo, hi = h.segs.back().hi;
      if (range) {
        const size_t k = below((uint32_t)h.segs.size()), l = k + below((uint32_t)(h.segs.size() - k));
        lo = h.segs[k].lo;
        hi = h.segs[l].hi;
      }
      tiles<4, 1, false>(h, map, want, lo, hi);
      tiles<4, 1, true>(h, map, want, lo, hi);
      tiles<4, 2, true>(h, map, want, lo, hi);
      tiles<8, 1, false>(h, map, want, lo, hi);
      tiles<8, 1, true>(h, map, want, lo, hi);
      tiles<8, 2, true>(h, map, want, lo, hi);
    }
  }
  printf("bad %ld, spread %s, partial groups %s\n", bad, spread ? "some" : "none", partial ? "some" : "none");
  printf("packed %d one %d gap7 %d gap8 %d d%d two decays %d decay inside a group %d long %d\n",
         mapped({{0, 10, 0.f}, {16, 20, 0.1f}}, 24), mapped({{0, 10, 0.f}}, 24), mapped({{0, 9, 0.f}, {16, 20, 0.f}}, 24),
         mapped({{0, 8, 0.f}, {16, 20, 0.f}}, 24), mapped({{0, 10, 0.f}, {16, 20, 0.f}}, 22), mapped({{0, 8, 0.2f}, {8, 20, 0.1f}}, 24),
         mapped({{0, 10, 0.f}, {10, 20, 0.1f}}, 24), mapped({{0, 10, 0.f}, {16, 20, 0.f}}, 24, false));
}
