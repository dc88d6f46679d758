// Loads of whole groups of four at the edges of a range, compiled for the host from the kernel source's own text under the
// address sanitizer (buffers are exactly as long as the data): elements of the range arrive, sources are cleared outside it
// where the error needs that, stores keep to the range, and clip_of takes groups only where they end within the buffer.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>
#define __device__
#define __forceinline__ inline
static inline float __uint_as_float(uint32_t u) { float f; memcpy(&f, &u, 4); return f; }
static inline uint32_t __float_as_uint(float f) { uint32_t u; memcpy(&u, &f, 4); return u; }
constexpr int kWave = 64;
namespace emu {
#include "helpers.inc"
#include "clip.inc"
}
using namespace emu;
struct Args { uint64_t d; };
static long bad = 0, groups = 0, elements = 0;

template <typename XT, typename ST>
void run(uint64_t d, uint64_t lo, uint64_t hi) {
  constexpr int VEC = XT::vec, H = 4 * kWave;
  const uint64_t N = (uint64_t)kWave * VEC;
  std::vector<uint8_t> x(d * XT::bytes), st(d * ST::bytes), xo(d * XT::bytes, 0xEE), so(d * ST::bytes, 0xEE);
  for (uint64_t i = 0; i < d; ++i) { store_elem<XT>(x.data(), i, (float)(i % 251) + 1.0f); store_elem<ST>(st.data(), i, (float)(i % 241) + 2.0f); }
  const Args a{d};
  for (uint64_t t = lo / N; t <= (hi - 1) / N; ++t) {
    const bool full = t * N >= lo && t * N + N <= hi;
    const int clip = clip_of(a, full, hi);
    if ((clip == kWhole) != full) ++bad;
    if (clip != kGroups) { elements += clip == kElements; if (clip == kElements && d % 4 == 0) ++bad; }
    if (clip != kGroups) continue;
    ++groups;
    for (uint32_t lane = 0; lane < (uint32_t)kWave; ++lane) {
      const uint64_t e = t * N + 4 * lane;
      float xv[VEC], sv[VEC], zero[VEC];
      unpack_raw<XT>(load_raw<XT, H, kGroups, true>(x.data(), e, lo, hi), xv);
      unpack_raw<XT>(load_raw<XT, H, kGroupsZeroed, true>(x.data(), e, lo, hi), zero);
      load_vals<ST, VEC, H, kGroups, true>(st.data(), e, lo, hi, sv);
      store_vals<XT, VEC, H, kGroups, true>(xo.data(), e, lo, hi, xv);
      store_vals<ST, VEC, H, kGroups, true>(so.data(), e, lo, hi, sv);
      for (int j = 0; j < VEC; ++j) {
        const uint64_t at = e + (j / 4) * H + j % 4;
        const bool inside = at >= lo && at < hi;
        if (inside && (xv[j] != load_elem<XT>(x.data(), at) || sv[j] != load_elem<ST>(st.data(), at))) ++bad;
        if (zero[j] != (inside ? load_elem<XT>(x.data(), at) : 0.0f)) ++bad;
      }
    }
    for (uint64_t i = 0; i < d; ++i) {
      const bool inside = i >= lo && i < hi && i >= t * N && i < t * N + N;
      for (int k = 0; k < XT::bytes; ++k) if (xo[i * XT::bytes + k] != (inside ? x[i * XT::bytes + k] : 0xEE)) ++bad;
      for (int k = 0; k < ST::bytes; ++k) if (so[i * ST::bytes + k] != (inside ? st[i * ST::bytes + k] : 0xEE)) ++bad;
    }
    std::fill(xo.begin(), xo.end(), 0xEE);
    std::fill(so.begin(), so.end(), 0xEE);
  }
}

int main() {
  for (uint64_t d : {512ull, 1032ull, 1030ull, 1029ull, 2051ull})
    for (uint64_t lo : {0ull, 1ull, 3ull, 4ull, 255ull, 258ull, 509ull})
      for (uint64_t n : {(uint64_t)1, (uint64_t)2, (uint64_t)3, (uint64_t)5, (uint64_t)250, (uint64_t)515, d})
        if (lo < d) {
          const uint64_t hi = lo + n < d ? lo + n : d;
          run<TF32, TF32>(d, lo, hi);
          run<TF32, TBF16>(d, lo, hi);
          run<TBF16, TF32>(d, lo, hi);
          run<TBF16, TBF16>(d, lo, hi);
        }
  printf("bad %ld, tiles by groups %s, by elements %s\n", bad, groups > 1000 ? "many" : "few", elements > 0 ? "some" : "none");
}
