// Test shim: the network's host code (csrc/mlp.hip) over stand-ins for the HIP runtime and the kernels, so
// that the CPU tests can let a chosen allocation fail.  The stand-ins keep a list of live allocations; a
// free of anything else and a kernel argument outside all of them are counted as faults.
#include <cstdlib>
#include <cstring>
#include <map>

#include "../paper_2608_14123_amd/csrc/mlp.hip"

namespace {
std::map<char*, size_t> live;
int faults = 0, fail_at = -1;

void check(const void* p, size_t bytes) {
  auto it = live.upper_bound((char*)p);
  if (it == live.begin()) { ++faults; return; }
  --it;
  if ((char*)p + bytes > it->first + it->second) ++faults;
}
}  // namespace

extern "C" {
hipError_t hipMalloc(void** p, size_t n) {
  if (fail_at >= 0 && fail_at-- == 0) return hipErrorOutOfMemory;
  *p = std::calloc(n, 1);
  live[(char*)*p] = n;
  return hipSuccess;
}
hipError_t hipFree(void* p) {
  if (!live.erase((char*)p)) { ++faults; return hipErrorInvalidValue; }
  std::free(p);
  return hipSuccess;
}
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) {
  if (k != hipMemcpyDeviceToHost) check(d, n);
  if (k != hipMemcpyHostToDevice) check(s, n);
  if (!faults) std::memmove(d, s, n);
  return hipSuccess;
}
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) {
  check(d, n);
  if (!faults) std::memset(d, v, n);
  return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }

int shim_faults() { return faults; }
int shim_live() { return (int)live.size(); }
void shim_fail_at(int k) { fail_at = k; }
void* shim_alloc(size_t n) { void* p = nullptr; return hipMalloc(&p, n) == hipSuccess ? p : nullptr; }
void shim_free(void* p) { hipFree(p); }
}

namespace dgfas {
const char* set_error(const std::string&) { return nullptr; }
void cast_bf16(int64_t n, const float* x, uint16_t* y, hipStream_t) { check(x, n * 4); check(y, n * 2); }
void gemm_bf16(int M, int N, int K, const uint16_t* A, int64_t sam, int64_t sak, const uint16_t* B, int64_t sbk,
               int64_t sbn, float* C, uint16_t* Cb, const float* bias, int, int, hipStream_t, float* ws, int64_t ws_cap,
               int ones, const float* gate) {
  check(A, 2 * ((M - ones - 1) * sam + (K - 1) * sak + 1));
  check(B, 2 * ((K - 1) * sbk + (N - 1) * sbn + 1));
  if (C) check(C, 4 * (size_t)M * N);
  if (Cb) check(Cb, 2 * (size_t)M * N);
  if (bias) check(bias, 4 * (size_t)N);
  if (gate) check(gate, 4 * (size_t)M * N);
  if (ws) check(ws, 4 * (size_t)ws_cap);
}
void mse_grad(int64_t n, int cols, int ldb, const float* Y, const float* T, float, uint16_t* dYb, double* part, int nb,
              hipStream_t) {
  check(Y, n * 4); check(T, n * 4); check(dYb, 2 * (n / cols * ldb)); check(part, nb * sizeof(double));
}
void pad_rows(int rows, int cols, int ldd, const uint16_t* s, uint16_t* d, hipStream_t) {
  check(s, 2 * (size_t)rows * cols); check(d, 2 * (size_t)rows * ldd);
}
void adam(int64_t n, float* w, const float* g, float* m, float* v, uint16_t* wb, float, float, float, float, float, float,
          hipStream_t) {
  check(w, n * 4); check(g, n * 4); check(m, n * 4); check(v, n * 4); check(wb, n * 2);
}
}  // namespace dgfas
