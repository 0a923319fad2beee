// Training set-up that fails at each of its runtime calls in turn, without a
// GPU: this program brings its own HIP and rocBLAS entry points (the library's
// references bind to the program first), which count the calls, hand out
// addresses that nobody reads and fail the call that they are told to.
//
// A set-up that failed must leave nothing behind: the next training call does
// all of it again, and what was allocated is given back.
//
// usage: host_train_setup; prints one line per fault, exit status 0 when all hold
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../include/msd.h"

namespace {
int calls = 0, fail_at = -1;  // runtime calls of the set-up so far; the one to fail
int mallocs = 0, live = 0, handles = 0;
bool next_fails() { return calls++ == fail_at; }
void* address() {
  static uintptr_t p = 1 << 20;
  return reinterpret_cast<void*>(p += 1 << 20);
}
}  // namespace

extern "C" {
struct dim3_ {
  uint32_t x, y, z;
};
int hipMalloc(void** p, size_t) {
  ++mallocs;
  if (next_fails()) return 2;
  ++live;
  *p = address();
  return 0;
}
int hipFree(void* p) {
  if (p) --live;
  return 0;
}
int hipHostMalloc(void** p, size_t n, unsigned) { return (*p = calloc(n, 1)) ? 0 : 2; }
int hipHostFree(void* p) {
  free(p);
  return 0;
}
int hipGetDevice(int* d) {
  *d = 0;
  return 0;
}
int hipGetSymbolAddress(void** p, const void*) {
  *p = address();
  return 0;
}
int hipMemcpyAsync(void*, const void*, size_t, int, void*) { return next_fails() ? 1 : 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipStreamSynchronize(void*) { return next_fails() ? 1 : 0; }
int hipGetLastError() { return 0; }
const char* hipGetErrorString(int) { return "told to fail"; }
int hipLaunchKernel(const void*, dim3_, dim3_, void**, size_t, void*) { return 0; }
int hipExtLaunchKernel(const void*, dim3_, dim3_, void**, size_t, void*, void*, void*, int) {
  return 0;
}
int __hipPushCallConfiguration(dim3_, dim3_, size_t, void*) { return 0; }
int __hipPopCallConfiguration(dim3_* g, dim3_* b, size_t* n, void** s) {
  *g = *b = dim3_{1, 1, 1};
  *n = 0;
  *s = nullptr;
  return 0;
}
int rocblas_create_handle(void** h) {
  if (next_fails()) return 1;
  ++handles;
  *h = address();
  return 0;
}
int rocblas_destroy_handle(void*) {
  --handles;
  return 0;
}
int rocblas_set_stream(void*, void*) { return next_fails() ? 1 : 0; }
int rocblas_set_workspace(void*, void*, size_t) { return next_fails() ? 1 : 0; }
}

int main() {
  const msd_model_desc m = {2, 128, 4, 2, 64, 256, 512, 1e4f, 1e-5f};
  const msd_limits lim = {1, 512, 16, 300};
  void* const a = address();
  const msd_layer_weights lw = {a, a, a, a, a, a, a, a, a};
  const msd_layer_weights layers[2] = {lw, lw};
  const msd_target_weights tw = {a, layers, a, a};
  const msd_draft_weights dw = {a, lw};
  const msd_buffers bufs = {a, a, a, a, a, a};
  const size_t qd = 256, kd = 128, d = 128, F = 256;
  const size_t np = 2 * d * d + (qd + 2 * kd) * d + d * qd + 3 * F * d + 2 * d;
  int bad = 0, total = 0, per_setup = 0;
  for (int k = -1; k < total || k < 0; ++k) {  // -1: no fault, to count the calls
    msd_ctx* c = nullptr;
    if (msd_create(&m, &lim, &tw, &dw, &bufs, nullptr, &c) != MSD_OK) {
      printf("msd_create: %s\n", msd_last_error(nullptr));
      return 1;
    }
    calls = mallocs = 0;
    fail_at = k;
    const int r1 = msd_train_read(c, 0, static_cast<float*>(a), np);
    fail_at = -1;
    if (k < 0) {
      total = calls - 1;  // the last one is the read's own wait
      per_setup = mallocs;
      if (r1 != MSD_OK || per_setup == 0) {
        printf("msd_train_read: %s\n", msd_last_error(c));
        return 1;
      }
    } else {
      const int left = live;
      mallocs = 0;
      const int r2 = msd_train_read(c, 0, static_cast<float*>(a), np);
      const bool ok = r1 == MSD_ERR_HIP && left == 0 && r2 == MSD_OK && mallocs == per_setup;
      printf("call %d of %d fails: error %d, %d buffers left; again: error %d, %d of %d buffers%s\n",
             k, total, r1, left, r2, mallocs, per_setup, ok ? "" : "  WRONG");
      bad += !ok;
    }
    msd_destroy(c);
    if (live != 0 || handles != 0) {
      printf("call %d: %d buffers and %d handles after msd_destroy\n", k, live, handles);
      ++bad;
      live = handles = 0;
    }
  }
  printf("%d faults, %d wrong\n", total, bad);
  return bad ? 1 : 0;
}
