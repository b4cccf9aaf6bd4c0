// Device helpers shared by the HIP kernels of the library.
#pragma once

#include <hip/hip_runtime.h>

namespace mdd {

__device__ __forceinline__ float2 cadd(float2 a, float2 b) { return make_float2(a.x + b.x, a.y + b.y); }
__device__ __forceinline__ float2 csub(float2 a, float2 b) { return make_float2(a.x - b.x, a.y - b.y); }
__device__ __forceinline__ float2 cscale(float2 a, float s) { return make_float2(a.x * s, a.y * s); }
__device__ __forceinline__ float2 cconj(float2 a) { return make_float2(a.x, -a.y); }
__device__ __forceinline__ float2 cmul(float2 a, float2 b) {
  return make_float2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x);
}

// Orders LDS traffic of one wavefront: every lane's earlier LDS writes are
// visible to every lane's later LDS reads (a wavefront executes in lockstep;
// the fences stop the compiler from moving accesses across this point).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_down(v, off, 64);
  return v;
}

// Global memory through buffer descriptors: a uniform base, a 32-bit byte offset per lane
// that does not change over a loop, and the hardware's bounds check, which reads zeros
// past the end and drops stores there.  That takes the address arithmetic, the clamping
// and the zeroing of partial chunks out of the vector unit.
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
constexpr unsigned PAST_END = 0xffffffffu;        // an offset that is out of bounds for every buffer
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_at(const void* base, unsigned bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00020000);
}
__device__ __forceinline__ float2 buffer_get2(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
__device__ __forceinline__ float4 buffer_get4(__amdgpu_buffer_rsrc_t r, unsigned off) {
  return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, 0));
}
// NT: a streaming store, for results that push reused data out of the caches.
template <bool NT = false>
__device__ __forceinline__ void buffer_put2(__amdgpu_buffer_rsrc_t r, unsigned off, float2 v) {
  __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(uintx2, v), r, off, 0, NT ? 2 : 0);
}

// Row of D_k for batch entry b whose source s is valid: s in the resident spectra,
// b in spectra staged for the batch.
template <class GemmArgsT>
__device__ __forceinline__ int drow_of(const GemmArgsT& a, int b, int s) {
  return a.dpos ? b : s;
}

// Offset of row (k, .) of U_k for batch entry b with source s: row s of the resident
// data spectra, or row b of data spectra staged for the batch.  Callers pass b < nb.
template <class GemmArgsT>
__device__ __forceinline__ long long urow_off(const GemmArgsT& a, int k, int b, int s) {
  return ((long long)k * a.uns + (a.upos ? b : s)) * a.nvsp;
}

// Sum of n doubles by one workgroup of NTH threads in a fixed order (four
// independent loads per thread per round, then a fixed tree): bitwise
// reproducible.  `red` is LDS of NTH / 64 doubles; the result is in thread 0.
template <int NTH>
__device__ __forceinline__ double block_fixed_sum(const double* p, int n, double* red) {
  double acc = 0.0;
  int i = threadIdx.x;
  for (; i + 3 * NTH < n; i += 4 * NTH) {
    const double x0 = p[i], x1 = p[i + NTH], x2 = p[i + 2 * NTH], x3 = p[i + 3 * NTH];
    acc += (x0 + x1) + (x2 + x3);
  }
  for (; i < n; i += NTH) acc += p[i];
  acc = wave_sum(acc);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) red[wave] = acc;
  __syncthreads();
  double s = 0.0;
  if (threadIdx.x == 0)
    for (int w = 0; w < NTH / 64; ++w) s += red[w];
  return s;
}

}  // namespace mdd
