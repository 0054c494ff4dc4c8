// The tracker's short square roots and reciprocals beside the general
// operations, for tests/test_gpu_roots.py.
#include "tpc_device.h"

using namespace tpc;

namespace {

__device__ void note(unsigned long long* bad, uint32_t* example, int k, uint32_t bits) {
  if (atomicAdd(&bad[k], 1ull) == 0ull) example[k] = bits;
}

// every float with bits in [lo, lo + n)
__global__ void k_floats(uint32_t lo, uint32_t n, unsigned long long* bad, uint32_t* example) {
  const uint32_t stride = gridDim.x * blockDim.x;
  for (uint64_t i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) {
    const uint32_t bits = lo + (uint32_t)i;
    const float x = __uint_as_float(bits);
    const uint32_t root = __float_as_uint(sqrt_mid(x)), rcp = __float_as_uint(rcp_mid(x));
    if (root != __float_as_uint(sqrtf(x))) note(bad, example, 0, bits);
    if (rcp != __float_as_uint(1.0f / x)) note(bad, example, 1, bits);
    // in double and rounded once: correctly rounded for both
    if (root != __float_as_uint((float)sqrt((double)x))) note(bad, example, 2, bits);
    if (rcp != __float_as_uint((float)(1.0 / (double)x))) note(bad, example, 3, bits);
    // the determinant's reciprocal is the same for either sign
    if (__float_as_uint(rcp_det(-x)) != (rcp | 0x80000000u)) note(bad, example, 4, bits);
  }
}

__global__ void k_dets(const float* x, float* out, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] = rcp_det(x[i]);
}

__global__ void k_doubles(const double* x, double* root, double* rcp, int64_t n) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  root[i] = sqrt_mid(x[i]);
  rcp[i] = rcp_mid(x[i]);
}

int launched(int64_t n) { return n >= 0 && hipGetLastError() == hipSuccess ? 0 : -1; }

}  // namespace

extern "C" {

int roots_floats(uint32_t lo, uint32_t n, unsigned long long* bad, uint32_t* example, void* stream) {
  k_floats<<<4096, 256, 0, reinterpret_cast<hipStream_t>(stream)>>>(lo, n, bad, example);
  return launched(n);
}
int roots_dets(const float* x, float* out, int64_t n, void* stream) {
  if (n < 1) return -1;
  k_dets<<<(unsigned)((n + 255) / 256), 256, 0, reinterpret_cast<hipStream_t>(stream)>>>(x, out, n);
  return launched(n);
}
int roots_doubles(const double* x, double* root, double* rcp, int64_t n, void* stream) {
  if (n < 1) return -1;
  k_doubles<<<(unsigned)((n + 255) / 256), 256, 0, reinterpret_cast<hipStream_t>(stream)>>>(x, root, rcp, n);
  return launched(n);
}

}  // extern "C"
