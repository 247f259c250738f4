// Element-wise glue between convolution layers (activation, residual add, channel concat and
// their gradients).  Not part of the paper's method; they exist so that a whole network can
// run on the library's own kernels.  All are bandwidth-bound streaming kernels over
// [rows][channels] tensors: a lane moves 16 bytes at a time (one element at a time they were bound by the
// number of memory instructions: gradient through a ReLU at the large levels of a 400k-voxel network 14.6 -> 9.3 us a
// call, concatenating copies 14.9 -> 7.8 us).
#include "common.h"

#include <algorithm>

namespace spc {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

enum EwOp { EW_RELU = 0, EW_ADD = 1, EW_ADD_RELU = 2, EW_RELU_BWD = 3 };

template <typename T, int OP> __device__ __forceinline__ T ew_one(T a, T b) {
  const float x = (float)a;
  const float y = (OP == EW_RELU) ? 0.f : (float)b;
  float r;
  if (OP == EW_RELU) r = x > 0.f ? x : 0.f;
  else if (OP == EW_ADD) r = x + y;
  else if (OP == EW_ADD_RELU) r = (x + y) > 0.f ? (x + y) : 0.f;
  else r = y > 0.f ? x : 0.f;
  return (T)r;
}

// out[i] = op(a[i], b[i]); RELU: max(a,0); ADD: a+b; ADD_RELU: max(a+b,0); RELU_BWD: b > 0 ? a : 0.
// (out may alias a or b: no __restrict__.)  Vectors [0, nv) of 16 bytes, one per thread, then the elements that
// fill no vector, or every element where a pointer is not 16-byte aligned (nv = 0).
template <typename T, int OP>
__global__ void __launch_bounds__(256) k_ew(const T* a, const T* b, T* out, long long nv, long long n) {
  constexpr int W = 16 / sizeof(T);
  typedef T vec __attribute__((ext_vector_type(W)));
  const long long stride = (long long)gridDim.x * blockDim.x;
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long long i = t; i < nv; i += stride) {
    const vec x = reinterpret_cast<const vec*>(a)[i];
    vec y = x, r;
    if (OP != EW_RELU) y = reinterpret_cast<const vec*>(b)[i];
#pragma unroll
    for (int j = 0; j < W; ++j) r[j] = ew_one<T, OP>(x[j], y[j]);
    reinterpret_cast<vec*>(out)[i] = r;
  }
  for (long long i = nv * W + t; i < n; i += stride) out[i] = ew_one<T, OP>(a[i], OP == EW_RELU ? a[i] : b[i]);
}

// dst[r][dst_off + c] = src[r][src_off + c] for c < cols (channel concat / split), in units of V: row lengths,
// offsets and column count are multiples of it.
template <typename V, typename I>
__global__ void __launch_bounds__(256) k_copy_cols(const V* __restrict__ src, int src_ld, int src_off, V* __restrict__ dst,
                                                   int dst_ld, int dst_off, int cols, I total) {
  const I stride = (I)gridDim.x * blockDim.x;
  for (I i = (I)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += stride) {
    const I r = i / (I)cols;
    const int c = (int)(i - r * (I)cols);
    dst[(long long)r * dst_ld + dst_off + c] = src[(long long)r * src_ld + src_off + c];
  }
}

template <typename T>
int launch_ew(int op, const void* a, const void* b, void* out, long long n, hipStream_t st) {
  constexpr long long W = 16 / sizeof(T);
  const bool aligned = (((size_t)a | (size_t)(op == EW_RELU ? a : b) | (size_t)out) & 15) == 0;
  const long long nv = aligned ? n / W : 0;
  const long long threads = nv > 0 ? std::max(nv, n - nv * W) : n;
  const unsigned blocks = (unsigned)std::min<long long>((threads + 255) / 256, 1 << 16);
  const T* pa = (const T*)a;
  const T* pb = (const T*)b;
  T* po = (T*)out;
  switch (op) {
    case EW_RELU: hipLaunchKernelGGL((k_ew<T, EW_RELU>), dim3(blocks), dim3(256), 0, st, pa, pb, po, nv, n); break;
    case EW_ADD: hipLaunchKernelGGL((k_ew<T, EW_ADD>), dim3(blocks), dim3(256), 0, st, pa, pb, po, nv, n); break;
    case EW_ADD_RELU: hipLaunchKernelGGL((k_ew<T, EW_ADD_RELU>), dim3(blocks), dim3(256), 0, st, pa, pb, po, nv, n); break;
    case EW_RELU_BWD: hipLaunchKernelGGL((k_ew<T, EW_RELU_BWD>), dim3(blocks), dim3(256), 0, st, pa, pb, po, nv, n); break;
    default: return SPCONV_EINVAL;
  }
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

template <typename V>
int launch_copy_cols(const void* src, int src_ld, int src_off, void* dst, int dst_ld, int dst_off, int cols, long long rows,
                     hipStream_t st) {
  const long long total = rows * cols;
  const unsigned blocks = (unsigned)std::min<long long>((total + 255) / 256, 1 << 16);
  if (total < (1ll << 31))  // (32-bit index arithmetic: the loop's step stays below 2^24)
    hipLaunchKernelGGL((k_copy_cols<V, unsigned>), dim3(blocks), dim3(256), 0, st, (const V*)src, src_ld, src_off, (V*)dst,
                       dst_ld, dst_off, cols, (unsigned)total);
  else
    hipLaunchKernelGGL((k_copy_cols<V, unsigned long long>), dim3(blocks), dim3(256), 0, st, (const V*)src, src_ld, src_off,
                       (V*)dst, dst_ld, dst_off, cols, (unsigned long long)total);
  SPC_LAUNCH_CHECK();
  return SPCONV_OK;
}

}  // namespace
}  // namespace spc

using namespace spc;

extern "C" {

SPCONV_API int spconv_ew(int op, const void* a, const void* b, void* out, int64_t n, spconv_dtype dtype, void* stream) {
  if (n < 0 || op < 0 || op > 3) return SPCONV_EINVAL;
  if (n == 0) return SPCONV_OK;
  if (!a || !out || (op != EW_RELU && !b)) return SPCONV_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  switch (dtype) {
    case SPCONV_F32: return launch_ew<float>(op, a, b, out, n, st);
    case SPCONV_F16: return launch_ew<_Float16>(op, a, b, out, n, st);
    case SPCONV_BF16: return launch_ew<__bf16>(op, a, b, out, n, st);
  }
  return SPCONV_EINVAL;
}

SPCONV_API int spconv_copy_cols(const void* src, int src_ld, int src_off, void* dst, int dst_ld, int dst_off, int cols,
                                int64_t rows, spconv_dtype dtype, void* stream) {
  if (rows < 0 || cols < 0 || src_off < 0 || dst_off < 0 || src_off + cols > src_ld || dst_off + cols > dst_ld)
    return SPCONV_EINVAL;
  if (rows == 0 || cols == 0) return SPCONV_OK;
  if (!src || !dst) return SPCONV_EINVAL;
  hipStream_t st = (hipStream_t)stream;
  if (dtype != SPCONV_F32 && dtype != SPCONV_F16 && dtype != SPCONV_BF16) return SPCONV_EINVAL;
  // the widest unit (16, 8, 4 or 2 bytes) that divides every length, offset and address
  const int e = dtype == SPCONV_F32 ? 4 : 2;
  const size_t all = (size_t)(src_ld * e) | (size_t)(src_off * e) | (size_t)(dst_ld * e) | (size_t)(dst_off * e) |
                     (size_t)(cols * e) | (size_t)src | (size_t)dst;
  const int u = (all & 15) == 0 ? 16 : (all & 7) == 0 ? 8 : (all & 3) == 0 ? 4 : 2;
  src_ld = src_ld * e / u, src_off = src_off * e / u, dst_ld = dst_ld * e / u, dst_off = dst_off * e / u, cols = cols * e / u;
  switch (u) {
    case 16: return launch_copy_cols<u32x4>(src, src_ld, src_off, dst, dst_ld, dst_off, cols, rows, st);
    case 8: return launch_copy_cols<unsigned long long>(src, src_ld, src_off, dst, dst_ld, dst_off, cols, rows, st);
    case 4: return launch_copy_cols<unsigned>(src, src_ld, src_off, dst, dst_ld, dst_off, cols, rows, st);
  }
  return launch_copy_cols<unsigned short>(src, src_ld, src_off, dst, dst_ld, dst_off, cols, rows, st);
}

}  // extern "C"
