// Where the lanes of a wavefront lie over a tile (lane_start and the distances between a lane's groups and vectors), compiled
// for the host from the kernel source's own text: over the tiles of a launch every element of the range comes up once,
// groups of four are whole, tiles that are full touch nothing outside the range, and whole blocks are spread.  And the order
// in which a die walks runs of pieces row after row: every piece of every row once, and rows outside, pieces inside a run.
#include <cstdint>
#include <cstdio>
#include <vector>
#define __device__
#define __forceinline__ inline
constexpr int kWave = 64;
namespace emu {
#include "layout.inc"
}
using namespace emu;

static void runs() {
  long bad = 0;
  for (uint32_t X : {1u, 2u, 8u})
    for (uint32_t R : {1u, 2u, 18u, 64u, 160u})
      for (uint32_t n : {1u, 7u, 8u, 9u, 255u, 2047u, 2048u, 2049u, 5000u})
        for (uint32_t run : {1u, 3u, 32u, 256u})
          for (uint32_t B : {32u, 256u}) {
            std::vector<int> seen((size_t)n * R, 0);
            const uint32_t grid = (n + X - 1) / X * X * R;
            uint32_t last = 0;
            for (uint32_t b = 0; b < grid; ++b) {
              uint32_t piece = n, position = R;
              const bool active = die_block_piece(b, R, X, n, B, piece, position, run);
              if (piece >= n || position >= R) { ++bad; continue; }
              if (active) ++seen[(size_t)piece * R + position];
              if (b % X == 0) {  // the first die: its positions rise within a run and start again with the next
                bad += position < last && position != 0;
                last = position;
              }
            }
            for (int c : seen) bad += c != 1;
          }
  printf("runs: %s\n", bad ? "FAIL" : "right");
}

template <int VEC, int U, bool STREAM>
long run(uint64_t lo, uint64_t hi) {
  constexpr uint64_t N = kWave * VEC * U;
  const uint64_t first = lo / N, last = (hi - 1) / N, base = first * N;
  std::vector<int> seen((last + 1) * N - base, 0);
  long bad = 0;
  for (uint64_t t = first; t <= last; ++t) {
    const bool full = t * N >= lo && t * N + N <= hi;
    bool spread = false;
    for (int lane = 0; lane < kWave; ++lane) {
      const uint64_t start = lane_start<VEC, U, STREAM>(t, lo, hi, lane);
      for (int u = 0; u < U; ++u)
        for (int h = 0; h < VEC / 4; ++h)
          for (int j = 0; j < 4; ++j) {
            const uint64_t e = start + u * kVectorStep<VEC, STREAM> + h * kGroupStep<STREAM> + j;
            if (e < base || e - base >= seen.size()) { ++bad; continue; }
            if (full && (e < lo || e >= hi)) ++bad;
            if (e / N != t) spread = true;
            ++seen[e - base];
          }
      bad += start % 4 != 0;
    }
    const uint64_t block = N == 256 ? 16384 : 32768, b0 = t * N / block * block;
    bad += spread != (STREAM && b0 >= lo && b0 + block <= hi);
  }
  for (int c : seen) bad += c != 1;
  return bad;
}

template <int VEC, int U, bool STREAM>
void sweep() {
  long bad = 0;
  for (uint64_t lo : {0ull, 4ull, 16384ull, 32767ull, 32768ull, 32769ull, 49152ull, 70000ull})
    for (uint64_t n : {1ull, 300ull, 16383ull, 16384ull, 32768ull, 32769ull, 65536ull, 98304ull + 5, 131072ull}) bad += run<VEC, U, STREAM>(lo, lo + n);
  printf("%d elements, %d vectors, %s: %s\n", VEC, U, STREAM ? "streaming" : "ordinary", bad ? "FAIL" : "right");
}

int main() {
  runs();
  sweep<4, 1, false>();
  sweep<4, 2, false>();
  sweep<8, 1, false>();
  sweep<8, 2, false>();
  sweep<4, 1, true>();
  sweep<4, 2, true>();
  sweep<8, 1, true>();
  sweep<8, 2, true>();
}
