// Elementwise and reduction kernels around the sweep: the column normalisation
// of W before the first sweep, BF16 operand casts, input checks, and the
// fixed-order FP64 reductions of the objective (Eq. 2 and the relative
// objective of Sec. 6.2).
#include <algorithm>

#include "internal.hpp"

namespace plnmf {
namespace {

__device__ __forceinline__ double block_sum_d(double v, double* sh) {
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if (lane == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  if (threadIdx.x == 0)
    for (int i = 0; i < (int)(blockDim.x >> 6); i++) t += sh[i];
  __syncthreads();
  return t;
}

// partial[b][k] = sum over rows r = b, b + nblk, ... of X[r,k]^2 (FP64)
__global__ void colsq_kernel(const float* __restrict__ X, int64_t rows, int K,
                              double* __restrict__ part) {
  const int b = blockIdx.x, nblk = gridDim.x;
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    double s = 0.0;
    for (int64_t r = b; r < rows; r += nblk) {
      const double x = X[r * K + k];
      s += x * x;
    }
    part[(int64_t)b * K + k] = s;
  }
}

// A column whose norm is zero (or overflows FP32) cannot be normalised: it is
// left unchanged and bit `bit` of *flag is set (every block sees the same
// norms; block 0 reports).
__global__ void colscale(float* __restrict__ X, int64_t rows, int K, const double* __restrict__ part,
                         int nblk, int32_t* flag, int bit) {
  __shared__ float norm[kMaxK];
  for (int k = threadIdx.x; k < K; k += blockDim.x) {
    double s = 0.0;
    for (int b = 0; b < nblk; b++) s += part[(int64_t)b * K + k];
    const float nk = (float)sqrt(s);
    const bool ok = nk > 0.0f && !isinf(nk);
    norm[k] = ok ? nk : 1.0f;
    if (!ok && blockIdx.x == 0) atomicOr(flag, bit);
  }
  __syncthreads();
  const int64_t n = rows * K;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int k = (int)(i % K);
    X[i] = X[i] / norm[k];
  }
}

__global__ void cast_kernel(const float* __restrict__ x, __bf16* __restrict__ y, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    y[i] = (__bf16)x[i];
}

// rows of the output ld apart
__global__ void cast_rows_kernel(const float* __restrict__ x, __bf16* __restrict__ y, int64_t rows,
                                 int64_t cols, int64_t ld) {
  const int64_t n = rows * cols;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t r = i / cols;
    y[r * ld + (i - r * cols)] = (__bf16)x[i];
  }
}

__global__ void cast_t_kernel(const float* __restrict__ x, __bf16* __restrict__ y, int64_t rows,
                              int64_t cols, int64_t ld) {
  __shared__ float tile[32][33];
  const int64_t r0 = (int64_t)blockIdx.y * 32, c0 = (int64_t)blockIdx.x * 32;
  const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;  // 256 threads: 8 rows per pass
  for (int i = ty; i < 32; i += 8) {
    const int64_t r = r0 + i, c = c0 + tx;
    tile[i][tx] = (r < rows && c < cols) ? x[r * cols + c] : 0.0f;
  }
  __syncthreads();
  for (int i = ty; i < 32; i += 8) {
    const int64_t c = c0 + i, r = r0 + tx;
    if (c < cols && r < rows) y[c * ld + r] = (__bf16)tile[tx][i];
  }
}

__global__ void finite_nonneg(const float* __restrict__ x, int64_t n, int32_t* flag, int bit) {
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const float v = x[i];
    if (!(v >= 0.0f) || isinf(v)) bad = true;
  }
  if (bad) atomicOr(flag, bit);
}

__global__ void sumsq_kernel(const float* __restrict__ x, int64_t n, double* __restrict__ part) {
  __shared__ double sh[16];
  double s = 0.0;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x) {
    const double v = x[i];
    s += v * v;
  }
  const double t = block_sum_d(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = t;
}

__global__ void finish_kernel(const double* __restrict__ part, int n, double* __restrict__ out) {
  __shared__ double sh[16];
  double s = 0.0;
  // fixed assignment of partials to threads, then a fixed tree
  for (int i = threadIdx.x; i < n; i += blockDim.x) s += part[i];
  const double t = block_sum_d(s, sh);
  if (threadIdx.x == 0) out[0] = t;
}

__device__ __forceinline__ void put_objective(double a2, double e2, double* out_half, double* out_rel) {
  if (e2 < 0.0) e2 = 0.0;
  out_half[0] = 0.5 * e2;
  out_rel[0] = sqrt(e2 / a2);
}

__global__ void combine_kernel(const double* a2, const double* e2, double* out_half, double* out_rel) {
  put_objective(a2[0], e2[0], out_half, out_rel);
}

// Two dot products over FP32 inputs, products and sums in FP64, and what is made
// of them, in one launch (five before: at a few hundred rows each took longer
// to start than to run: 17 -> 6 us at 256 x 100).  Blocks [0, nb1) take x y, the rest g q, a fixed
// share each; the last block to finish adds the partial sums in block order, so
// the result does not depend on which one that is.
__global__ __launch_bounds__(256) void objective_kernel(const double* __restrict__ a2,
                                                        const float* __restrict__ x,
                                                        const float* __restrict__ y, int64_t n1,
                                                        const float* __restrict__ g,
                                                        const float* __restrict__ q, int64_t n2, int nb1,
                                                        double* part, int32_t* count, double* out_half,
                                                        double* out_rel) {
  __shared__ double sh[16];
  __shared__ int last;
  const bool first = (int)blockIdx.x < nb1;
  const float* __restrict__ u = first ? x : g;
  const float* __restrict__ v = first ? y : q;
  const int64_t n = first ? n1 : n2;
  const int64_t b = first ? blockIdx.x : blockIdx.x - nb1, nb = first ? nb1 : gridDim.x - nb1;
  double s = 0.0;
  const int64_t st = nb * 256;
  int64_t i = b * 256 + threadIdx.x;
  for (; i + 3 * st < n; i += 4 * st) {  // four loads of each in flight
    const float u0 = u[i], u1 = u[i + st], u2 = u[i + 2 * st], u3 = u[i + 3 * st];
    const float v0 = v[i], v1 = v[i + st], v2 = v[i + 2 * st], v3 = v[i + 3 * st];
    s += (double)u0 * (double)v0;
    s += (double)u1 * (double)v1;
    s += (double)u2 * (double)v2;
    s += (double)u3 * (double)v3;
  }
  for (; i < n; i += st) s += (double)u[i] * (double)v[i];
  const double t = block_sum_d(s, sh);
  if (threadIdx.x == 0) {
    __hip_atomic_store(part + blockIdx.x, t, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    last = __hip_atomic_fetch_add(count, 1, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) ==
           (int)gridDim.x - 1;
  }
  __syncthreads();
  if (!last) return;
  double d1 = 0.0, d2 = 0.0;
  for (int k = threadIdx.x; k < (int)gridDim.x; k += 256) {
    const double p = __hip_atomic_load(part + k, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (k < nb1) d1 += p;
    else d2 += p;
  }
  d1 = block_sum_d(d1, sh);
  d2 = block_sum_d(d2, sh);
  if (threadIdx.x == 0) {
    put_objective(a2[0], a2[0] - 2.0 * d1 + d2, out_half, out_rel);
    *count = 0;
  }
}

}  // namespace

int reduce_blocks(int64_t n) {
  int64_t b = (n + 4095) / 4096;
  if (b > 1024) b = 1024;
  if (b < 1) b = 1;
  return (int)b;
}

hipError_t normalize_columns(float* X, int64_t rows, int K, double* part, int nblk_max,
                             int32_t* flag, int bit, hipStream_t s) {
  int nblk = (int)((rows + 63) / 64);
  if (nblk > nblk_max) nblk = nblk_max;
  if (nblk < 1) nblk = 1;
  colsq_kernel<<<nblk, 256, 0, s>>>(X, rows, K, part);
  int gb = (int)((rows * K + 255) / 256);
  if (gb > 2048) gb = 2048;
  if (gb < 1) gb = 1;
  colscale<<<gb, 256, 0, s>>>(X, rows, K, part, nblk, flag, bit);
  return hipGetLastError();
}

static int grid_for(int64_t n) {
  int64_t b = (n + 255) / 256;
  if (b > 4096) b = 4096;
  if (b < 1) b = 1;
  return (int)b;
}

hipError_t cast_bf16(const float* x, __bf16* y, int64_t n, hipStream_t s) {
  cast_kernel<<<grid_for(n), 256, 0, s>>>(x, y, n);
  return hipGetLastError();
}

hipError_t cast_bf16_rows(const float* x, __bf16* y, int64_t rows, int64_t cols, int64_t ld,
                          hipStream_t s) {
  cast_rows_kernel<<<grid_for(rows * cols), 256, 0, s>>>(x, y, rows, cols, ld);
  return hipGetLastError();
}

hipError_t cast_bf16_transpose(const float* x, __bf16* y, int64_t rows, int64_t cols, int64_t ld,
                               hipStream_t s) {
  dim3 grid((unsigned)((cols + 31) / 32), (unsigned)((rows + 31) / 32));
  cast_t_kernel<<<grid, 256, 0, s>>>(x, y, rows, cols, ld);
  return hipGetLastError();
}

__global__ void or_bits_kernel(int32_t* word, int32_t bits) { atomicOr(word, bits); }

hipError_t or_bits(int32_t* word, int32_t bits, hipStream_t s) {
  or_bits_kernel<<<1, 1, 0, s>>>(word, bits);
  return hipGetLastError();
}

hipError_t check_finite_nonneg(const float* x, int64_t n, int32_t* flag, int bit, hipStream_t s) {
  finite_nonneg<<<grid_for(n), 256, 0, s>>>(x, n, flag, bit);
  return hipGetLastError();
}

hipError_t sumsq_f64(const float* x, int64_t n, double* partial, int nblk, hipStream_t s) {
  sumsq_kernel<<<nblk, 256, 0, s>>>(x, n, partial);
  return hipGetLastError();
}

hipError_t finish_f64(const double* partial, int n, double* out, hipStream_t s) {
  finish_kernel<<<1, 256, 0, s>>>(partial, n, out);
  return hipGetLastError();
}

hipError_t combine_objective(const double* a2, const double* e2, double* out_half, double* out_rel,
                             hipStream_t s) {
  combine_kernel<<<1, 1, 0, s>>>(a2, e2, out_half, out_rel);
  return hipGetLastError();
}

hipError_t objective_identity(const double* a2, const float* x, const float* y, int64_t n1, const float* g,
                              const float* q, int64_t n2, double* part, int32_t* count, double* out_half,
                              double* out_rel, hipStream_t s) {
  // about 2,048 products per block
  const int nb1 = (int)std::max<int64_t>(1, std::min<int64_t>((n1 + 2047) / 2048, kObjParts - 128));
  const int nb2 = (int)std::max<int64_t>(1, std::min<int64_t>((n2 + 2047) / 2048, 128));
  objective_kernel<<<(unsigned)(nb1 + nb2), 256, 0, s>>>(a2, x, y, n1, g, q, n2, nb1, part, count, out_half,
                                                      out_rel);
  return hipGetLastError();
}

namespace {
__global__ void dense_rows_kernel(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                                  const float* __restrict__ val, const int32_t* __restrict__ rows,
                                  int64_t cols, float* __restrict__ out) {
  const int i = blockIdx.x;
  const int64_t r = rows[i];
  float* o = out + (int64_t)i * cols;
  for (int64_t j = rowptr[r] + threadIdx.x; j < rowptr[r + 1]; j += blockDim.x) o[col[j]] = val[j];
}

__global__ void scatter_rows_kernel(const float* __restrict__ src, const int32_t* __restrict__ rows,
                                    int K, float* __restrict__ dst) {
  const int i = blockIdx.x;
  const int64_t r = rows[i];
  for (int c = threadIdx.x; c < K; c += blockDim.x) dst[r * K + c] = src[(int64_t)i * K + c];
}
}  // namespace

hipError_t csr_dense_rows(const int32_t* rowptr, const int32_t* col, const float* val,
                          const int32_t* rows, int n, int64_t cols, float* out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipError_t e = hipMemsetAsync(out, 0, (size_t)n * cols * sizeof(float), s);
  if (e != hipSuccess) return e;
  dense_rows_kernel<<<(unsigned)n, 256, 0, s>>>(rowptr, col, val, rows, cols, out);
  return hipGetLastError();
}

hipError_t scatter_rows(const float* src, const int32_t* rows, int n, int K, float* dst,
                        hipStream_t s) {
  if (n <= 0) return hipSuccess;
  scatter_rows_kernel<<<(unsigned)n, 128, 0, s>>>(src, rows, K, dst);
  return hipGetLastError();
}

}  // namespace plnmf
