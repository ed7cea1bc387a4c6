// The permutation search with the HIP runtime's part played by this file: copies are under way until the stream is waited for,
// and the n-th check of a launch fails.  Whatever n is, no copy from or to the caller's arrays may be left when the search returns.
// Built by tests/test_host_sanitizers.py from the host pass of csrc/vnm_permsearch.hip and vnm_lsa.hip.
#include <hip/hip_runtime.h>
#include <cstdio>
#include <cstring>
#include <vector>
#include "vnm_internal.h"

static int g_pending = 0, g_checks = 0, g_fail_at = -1;
extern "C" {
hipError_t hipMemcpyAsync(void* dst, const void*, size_t n, hipMemcpyKind kind, hipStream_t) {
  ++g_pending;
  if (kind == hipMemcpyDeviceToHost) memset(dst, 0, n);          // (gains of zero: any assignment is optimal)
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { g_pending = 0; return hipSuccess; }
hipError_t hipGetLastError() { return g_checks++ == g_fail_at ? hipErrorLaunchFailure : hipSuccess; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, dim3*, dim3*, int*) {}
const char* hipGetErrorString(hipError_t) { return ""; }
}
namespace vnm {
void set_hip_error(hipError_t, const char*) {}
int allow_big_lds(const void*, const char*) { return VNM_OK; }
}

int main() {
  const int64_t out = 64, in = 20;
  std::vector<float> S((size_t)(out * in), 1.f);
  std::vector<int> po((size_t)out), pi((size_t)in);
  int64_t bytes = 0, history[3];
  if (vnm_permutation_search_workspace_bytes(out, in, 16, 2, 5, &bytes)) return 1;
  void* ws = (void*)256;                                          // never touched: nothing is launched
  int failed = 0;
  for (g_fail_at = 0;; ++g_fail_at) {
    g_pending = g_checks = 0;
    const int rc = vnm_permutation_search(S.data(), out, in, in, 16, 2, 5, 1.0, 1, po.data(), pi.data(), history, ws, bytes, nullptr);
    if (g_pending) { fprintf(stderr, "%d copies under way after failure %d\n", g_pending, g_fail_at); ++failed; }
    if (rc == VNM_OK) break;                                      // beyond the last check
    if (rc != VNM_ERR_HIP) return 2;
  }
  if (g_fail_at < 20 || failed) return 3;
  printf("search_errors ok\n");
  return 0;
}
