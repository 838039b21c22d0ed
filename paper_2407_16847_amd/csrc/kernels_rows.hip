// kernels_rows.hip -- one wavefront per (batch*head, row) kernels.
//
// These walk each row's affine runs directly (the ACSR index map of section
// 5.1: the k-th value of run r sits at column start + stride * k) and serve
// every dtype and pattern: they are the fp32 path (fp32 FMA throughout, the
// library's accurate path) and run any request the matrix-core kernels do
// not take.  Lanes own output features.
#include <hip/hip_runtime.h>
#include <math.h>

#include "bounds.hpp"
#include "launch.hpp"

namespace splat {
namespace {

constexpr int kWave = 64;

__device__ __forceinline__ float to_f32(float x) { return x; }
__device__ __forceinline__ float to_f32(__bf16 x) { return (float)x; }
__device__ __forceinline__ void store(float* p, float v) { *p = v; }
__device__ __forceinline__ void store(__bf16* p, float v) { *p = (__bf16)v; }

// COL: P holds the head's values in column-major order, value (i, j) at
// col_pos(cols[j], i).
template <typename T, typename OutT, bool COL>
__global__ __launch_bounds__(kWave) void k_rspmm_rows(DevAcsr a, int d, const float* __restrict__ P,
                                                      const T* __restrict__ V,
                                                      OutT* __restrict__ O) {
  const int i = blockIdx.x, bh = blockIdx.y, lane = threadIdx.x;
  const size_t head = (size_t)bh * a.L * d;
  const float* p = P + (size_t)bh * a.nnz + (COL ? 0 : a.row_ptr[i]);
  const int64_t r0 = COL ? 0 : a.row_ptr[i];   // p's position in the head
  const RowRuns rr = a.runs[i];
  const bool two = d > kWave;
  float acc0 = 0.f, acc1 = 0.f;
#pragma unroll
  for (int r = 0; r < SPLAT_MAX_RUNS; ++r) {
    const Run q = rr.r[r];
#pragma unroll 4
    for (int k = 0; k < q.count; ++k) {
      const int j = dbg::idx(q.start + q.stride * k, a.L, dbg::kKey);
      const float pk = COL ? p[dbg::idx((int64_t)col_pos(a.cols[j], i), a.nnz, dbg::kColPos)]
                           : p[dbg::rel(q.prefix + k, r0, a.nnz, dbg::kValue)];
      const T* v = V + head + (size_t)j * d;
      acc0 = fmaf(pk, to_f32(v[lane]), acc0);
      if (two) acc1 = fmaf(pk, to_f32(v[lane + kWave]), acc1);
    }
  }
  OutT* o = O + head + (size_t)i * d;
  store(o + lane, acc0);
  if (two) store(o + lane + kWave, acc1);
}

#ifdef SPLAT_DEBUG_BOUNDS
// One index check on the device (the checked build's own test): out = the
// checked index.
__global__ void k_bounds_probe(int kind, int index, int n, int* out) {
  *out = dbg::idx(index, n, (dbg::Kind)kind);
}
#endif

}  // namespace

hipError_t bounds_collect_rows(uint32_t* bits, bool clear) { return dbg::collect(bits, clear); }

hipError_t bounds_probe(int kind, int index, int n, int* result) {
#ifndef SPLAT_DEBUG_BOUNDS
  (void)kind;
  (void)index;
  (void)n;
  (void)result;
  return hipErrorNotSupported;
#else
  int* d = nullptr;
  hipError_t e = hipMalloc(&d, sizeof(int));
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(k_bounds_probe, dim3(1), dim3(1), 0, 0, kind, index, n, d);
  e = hipGetLastError();
  if (e == hipSuccess) e = hipMemcpy(result, d, sizeof(int), hipMemcpyDeviceToHost);
  const hipError_t f = hipFree(d);
  return e != hipSuccess ? e : f;
#endif
}

template <typename T, bool COL>
static hipError_t rspmm_t(const DevAcsr& a, int BH, int d, const float* P, const void* V, void* O,
                          int out_dtype, hipStream_t st) {
  dim3 grid(a.L, BH);
  if (out_dtype == 0)
    hipLaunchKernelGGL((k_rspmm_rows<T, float, COL>), grid, dim3(kWave), 0, st, a, d, P,
                       (const T*)V, (float*)O);
  else
    hipLaunchKernelGGL((k_rspmm_rows<T, __bf16, COL>), grid, dim3(kWave), 0, st, a, d, P,
                       (const T*)V, (__bf16*)O);
  return hipGetLastError();
}

hipError_t launch_rspmm_rows(const DevAcsr& a, int dtype, int BH, int d, const float* P,
                             const void* V, void* O, int out_dtype, bool colmajor, hipStream_t st) {
  if (colmajor)
    return dtype == 0 ? rspmm_t<float, true>(a, BH, d, P, V, O, out_dtype, st)
                      : rspmm_t<__bf16, true>(a, BH, d, P, V, O, out_dtype, st);
  return dtype == 0 ? rspmm_t<float, false>(a, BH, d, P, V, O, out_dtype, st)
                    : rspmm_t<__bf16, false>(a, BH, d, P, V, O, out_dtype, st);
}

}  // namespace splat
