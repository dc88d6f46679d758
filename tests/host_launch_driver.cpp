// What a failed launch leaves behind, without a GPU: the built library on a modelled HIP runtime (this program defines the
// calls, so the library's references resolve here), whose launches fail when told to and then, like the real ones, leave
// the error for whoever asks next.  tests/test_host_abi.py builds and runs it.
#include "dadam.h"
#include <hip/hip_runtime_api.h>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

static hipError_t pending = hipSuccess;
static int launches = 0, fail_at = 0;  // the fail_at-th launch from now fails
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t a, int) {
  *v = a == hipDeviceAttributeNumberOfXccs ? 8 : 160 * 1024;
  return hipSuccess;
}
hipError_t hipMalloc(void** p, size_t n) { *p = calloc(1, n); return hipSuccess; }
hipError_t hipFree(void* p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void*) { static double array[1024]; *p = array; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipGetLastError() { const hipError_t e = pending; pending = hipSuccess; return e; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) {
  ++launches;
  if (fail_at && --fail_at == 0) return pending = hipErrorLaunchOutOfResources;
  return hipSuccess;
}
}

int main() {
  const uint32_t R = 4;
  const dadam_tensor_desc t = {0, 3000, 0.f, 0};
  dadam_config cfg{};
  cfg.abi_version = DADAM_ABI_VERSION; cfg.n_rows = cfg.n_cols = R; cfg.d = t.numel; cfg.n_tensors = 1; cfg.tensors = &t;
  cfg.lr = 1e-3f; cfg.beta1 = 0.9f; cfg.beta2 = 0.999f; cfg.eps = 1e-8f; cfg.accum_s = 2; cfg.beta_vhat = -1.f; cfg.device = 0;
  dadam_handle* h = nullptr;
  if (dadam_init(&cfg, &h) != DADAM_OK) { printf("init failed: %s\n", dadam_last_error(nullptr)); return 1; }
  const int32_t ptr[] = {0, 2, 4, 6, 8}, col[] = {0, 1, 1, 2, 2, 3, 3, 0};
  const std::vector<float> w(8, 0.5f);
  if (dadam_set_topology(h, 0, ptr, col, w.data(), nullptr) != DADAM_OK) return 1;
  std::vector<void*> at;
  for (uint32_t k = 0; k < 6 * R; ++k) at.push_back((void*)(uintptr_t)((1u << 30) + 16384 * k));
  dadam_buffers b{(const void* const*)&at[0], &at[R], (float* const*)&at[2 * R], (float* const*)&at[3 * R], (float* const*)&at[4 * R]};
  if (dadam_bind(h, &b) != DADAM_OK) return 1;
  const void* const* g = (const void* const*)&at[5 * R];
  double out = 0.0;
  struct { const char* name; int n_launches; int (*call)(dadam_handle*, const void* const*, double*); } calls[] = {
      {"step", 1, [](dadam_handle* hh, const void* const* gg, double*) { return dadam_gossip_step(hh, 0, gg, 1, DADAM_FUSE_ACCUM, nullptr); }},
      {"direct", 1, [](dadam_handle* hh, const void* const* gg, double*) { return dadam_gossip_step(hh, 0, gg, 1, DADAM_FORCE_DIRECT, nullptr); }},
      {"accumulate", 1, [](dadam_handle* hh, const void* const* gg, double*) { return dadam_accumulate(hh, gg, 1, nullptr); }},
      {"mix", 1, [](dadam_handle* hh, const void* const*, double*) { return dadam_mix(hh, 0, 0, nullptr); }},
      {"consensus", 2, [](dadam_handle* hh, const void* const*, double* o) { return dadam_mix_consensus(hh, 0, 0, o, nullptr); }},
      {"static", 3, [](dadam_handle* hh, const void* const*, double* o) { return dadam_mix_consensus_static(hh, 0, 0, o, nullptr); }}};
  for (const auto& c : calls) {
    for (int k = 1; k <= c.n_launches; ++k) {  // the k-th launch fails: reported once, by the call
      fail_at = k;
      const int rc = c.call(h, g, &out);
      printf("%s, launch %d fails: rc %d pending %d\n", c.name, k, rc, (int)hipGetLastError());
      fail_at = 0;
      (void)c.call(h, g, &out);  // a whole pass again
    }
    pending = hipErrorNotReady;  // somebody else's error is theirs, and no reason to call this launch failed
    launches = 0;
    const int rc = c.call(h, g, &out);
    printf("%s, another's error pending: rc %d launches %d pending %d\n", c.name, rc, launches, (int)hipGetLastError());
  }
  dadam_destroy(h);
  return 0;
}
