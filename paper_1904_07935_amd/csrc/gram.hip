// Gram matrices of the sweep, S = W^T W and Q = H H^T = Ht^T Ht (Alg. 1, the
// S and Q statements): C = X^T X for X [rows, K] row-major, K <= 512.
//
// The contraction (rows) is long and the output small, so the work is split
// by rows: one 512-thread workgroup per chunk of rows stages its chunk through
// LDS and accumulates the chunk's partial Gram on the matrix cores.  A second
// kernel adds the chunks' partials in chunk order and writes both triangles:
// the result is bitwise reproducible and independent of scheduling.
//
// Two kernels form the partials.
//  * gram_partial, on the FP32 matrix cores, up to 65,535 rows.  A chunk is one
//    chain of products in row order, whatever the tiling.
//  * gram_partial_split, from 65,536 rows on, where the FP32 matrix rate bounds
//    the first: BF16 matrix cores, every FP32 value split into three BF16 parts
//    (split8 in bf16x3.hpp), a column split once per stage for all its products.
//    LDS holds 16-byte chunks of eight consecutive rows of one column,
//    [part][row/8][column].  The high products have an accumulator of their own:
//    beside them the small ones (2^-8 of them and less) are below its rounding
//    after some hundred rows, and what falls away there is of one sign on the
//    diagonal.  Up to 256 columns the small ones' accumulator runs along; above,
//    for want of registers, it takes one stage's and is added.  Error against 64
//    bits, RMS relative, FP32 kernel / this one: 300,000 x 400 2.4e-7 / 7.8e-8
//    (one accumulator for both: 1.2e-6), 100,000 x 200 8.8e-8 / 6.6e-8, 65,536 x
//    40 6.9e-8 / 6.1e-8.  Fewer rows stay with the FP32 chain: there the
//    launch and the first load take most of the time (6,037 x 77: 8 us FP32;
//    26,000 x 200: 24 us FP32, 16 us split), and a sweep of a small sparse corpus, whose weak components
//    amplify the last bit of S and Q some hundredfold, keeps its trajectory.
//
// The split kernel cuts the output into units of 64 x 64 (2 x 2 matrix-core
// blocks) of the upper triangle.  Up to 256 columns (10 units) four waves take a
// unit each and the other four the same units on the other half of a stage's
// rows; for 64 columns (one unit) all eight waves split the rows.  Such shares
// are added in the LDS in a fixed order.  Wider Grams give each wave two units.
// Workgroups along y take different units of the same rows, so that a chunk's
// partial (4 K^2 bytes or so, against 4 K rows of input) stays small against its
// rows.  300,000 x 400: 688 -> 373 us, 100,000 x 400: 240 -> 130 us (FP32 before,
// split after); the matrix cores are busy about half of that.
#include <algorithm>

#include "bf16x3.hpp"
#include "internal.hpp"

namespace plnmf {
namespace {

constexpr int kThreads = 512;
constexpr int kWaves = kThreads / 64;

__host__ __device__ inline int nblk(int K) { return (K + 31) / 32; }
__host__ __device__ inline int upper_blocks(int K) { return nblk(K) * (nblk(K) + 1) / 2; }
__host__ __device__ inline int npair(int K) { return (K + 63) / 64; }
__host__ __device__ inline int upper_units(int K) { return npair(K) * (npair(K) + 1) / 2; }

// index u in the row-major upper triangle of n x n -> (i, j), i <= j
__device__ __forceinline__ void upper_of(int u, int n, int& i, int& j) {
  int r = 0, len = n;
  while (u >= len) {
    u -= len;
    r++;
    len--;
  }
  i = r;
  j = r + u;
}

// partial[chunk][u][32][32] for the upper blocks [8 BPW y, 8 BPW (y + 1)) on the
// FP32 matrix cores, BPW blocks per wave.  A stage is the rows that kPer float4
// (or 4 kPer floats, K % 4 != 0) per thread hold; the next one is in flight in
// registers and the LDS has two, so the first two stages' loads overlap.  What
// bounds it: the FP32 matrix rate at some 100 rows and 28 blocks per CU (26,000 x
// 200: 9.5 of 24 us, then the partials' 29 MB), else the launch and one memory
// round trip (1,000 x 16: 14 -> 5 us, 6,037 x 77: 17 -> 8 us, against stages of
// 32 rows and four blocks in every wave).
constexpr int kPer = 8;
inline int stage_rows(int K) {
  const int r = kPer * kThreads * 4 / (32 * nblk(K));
  return r < 64 ? r / 2 * 2 : 64;
}

template <int BPW, bool VEC>
__global__ __launch_bounds__(kThreads) void gram_partial(const float* __restrict__ X, int64_t rows,
                                                         int K, int64_t rows_per_chunk, int rs,
                                                         float* __restrict__ partial) {
  extern __shared__ float stage[];  // [2][rs][P], P = 32 * nblk(K)
  constexpr int NR = VEC ? kPer : 4 * kPer;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int nb = nblk(K), P = 32 * nb, nu = upper_blocks(K);
  const int64_t chunk = blockIdx.x, r0 = chunk * rows_per_chunk;
  const int64_t r1 = r0 + rows_per_chunk < rows ? r0 + rows_per_chunk : rows;
  const int ubase = blockIdx.y * kWaves * BPW;
  int bi[BPW], bj[BPW];
#pragma unroll
  for (int k = 0; k < BPW; k++) {
    const int u = ubase + k * kWaves + w;
    bi[k] = bj[k] = 0;  // a block past the last is computed like (0, 0), never stored
    if (u < nu) upper_of(u, nb, bi[k], bj[k]);
  }
  const bool idle = ubase + w >= nu;
  floatx16 acc[BPW];
#pragma unroll
  for (int k = 0; k < BPW; k++)
#pragma unroll
    for (int e = 0; e < 16; e++) acc[k][e] = 0.0f;

  // item i of a thread: a float4 (a float) of a staged row, column fastest
  const int per_row = VEC ? P / 4 : P, items = rs * per_row;
  uint32_t off[NR];
#pragma unroll
  for (int i = 0; i < NR; i++) {
    const int c = tid + kThreads * i, r = c / per_row, col = (c - r * per_row) * (VEC ? 4 : 1);
    off[i] = c < items && col < K ? (uint32_t)(r * K + col) * 4 : kOutside;
  }
  floatx4 v4[VEC ? NR : 1];
  float v1[VEC ? 1 : NR];
  auto fetch = [&](int64_t s0) {  // rows past the chunk read as zeros
    const __amdgpu_buffer_rsrc_t view = tile_view(X + s0 * K, (r1 - s0) * K * 4);
#pragma unroll
    for (int i = 0; i < NR; i++) {
      if constexpr (VEC) v4[i] = __builtin_bit_cast(floatx4, ld16(view, off[i]));
      else v1[i] = __uint_as_float(ld4(view, off[i]));
    }
  };
  auto put = [&](float* st) {
#pragma unroll
    for (int i = 0; i < NR; i++) {
      const int c = tid + kThreads * i;
      if (c >= items) continue;
      if constexpr (VEC) *(floatx4*)(st + 4 * c) = v4[i];
      else st[c] = v1[i];
    }
  };
  fetch(r0);
  const int h = lane >> 5, m = lane & 31;
  const int ns = (int)((r1 - r0 + rs - 1) / rs);
  put(stage);
  if (ns > 1) fetch(r0 + rs);
  __syncthreads();
#pragma unroll 1
  for (int t = 0; t < ns; t++) {
    const float* st = stage + (t & 1) * rs * P;
    const int64_t left = r1 - r0 - (int64_t)t * rs;
    const int n = left < rs ? (int)left : rs;
    if (!idle) {
      auto step = [&](int kk) {
        const float* row = st + (kk + h) * P;
        float av[BPW], bv[BPW];
#pragma unroll
        for (int k = 0; k < BPW; k++) {
          av[k] = row[32 * bi[k] + m];
          bv[k] = row[32 * bj[k] + m];
        }
#pragma unroll
        for (int k = 0; k < BPW; k++)
          acc[k] = __builtin_amdgcn_mfma_f32_32x32x2f32(av[k], bv[k], acc[k], 0, 0, 0);
      };
      int kk = 0;
      for (; kk + 16 <= n; kk += 16) {
#pragma unroll
        for (int q = 0; q < 16; q += 2) step(kk + q);
      }
      for (; kk < n; kk += 2) step(kk);
    }
    if (t + 1 < ns) {
      put(stage + ((t + 1) & 1) * rs * P);
      if (t + 2 < ns) fetch(r0 + (int64_t)(t + 2) * rs);
      __syncthreads();
    }
  }
  // lane holds C block row 8 j + 4 h + i, column lane % 32, in acc[4 j + i]
#pragma unroll
  for (int k = 0; k < BPW; k++) {
    const int u = ubase + k * kWaves + w;
    if (u >= nu) continue;
    float* dst = partial + (chunk * nu + u) * 1024;
#pragma unroll
    for (int e = 0; e < 16; e++) dst[(8 * (e >> 2) + 4 * h + (e & 3)) * 32 + m] = acc[k][e];
  }
}

// How a width is worked on by the split kernel: row shares per unit, units per wave, rows per stage
// and LDS stages.
template <int MODE>
struct Mode;
template <>
struct Mode<0> {  // K <= 64
  static constexpr int KS = 8, UPW = 1, BK = 128, BUFS = 1, COLS = 64;
};
template <>
struct Mode<1> {  // K <= 256
  static constexpr int KS = 2, UPW = 1, BK = 32, BUFS = 2, COLS = 256;
};
template <>
struct Mode<2> {  // K <= 512
  static constexpr int KS = 1, UPW = 2, BK = 16, BUFS = 2, COLS = 512;
};
inline int mode_of(int K) { return K <= 64 ? 0 : K <= 256 ? 1 : 2; }
// units a workgroup holds
template <int MODE>
__host__ __device__ constexpr int unit_slots() {
  return kWaves / Mode<MODE>::KS * Mode<MODE>::UPW;
}
template <int MODE>
size_t lds_bytes(int K) {
  using M = Mode<MODE>;
  const size_t stage = (size_t)M::BUFS * 3 * (M::BK / 8) * 64 * npair(K) * 16;
  const size_t shares = (size_t)(kWaves - kWaves / M::KS) * 4096 * 4;  // of the later row shares
  return stage > shares ? stage : shares;
}

// partial[chunk][u][32][32], u the upper 32 x 32 blocks; workgroup (chunk, y)
// computes the units [y upw, (y + 1) upw)
template <int MODE>
__global__ __launch_bounds__(kThreads) void gram_partial_split(const float* __restrict__ X, int64_t rows,
                                                         int K, int64_t rows_per_chunk, int upw,
                                                         float* __restrict__ partial) {
  using M = Mode<MODE>;
  constexpr int KS = M::KS, UPW = M::UPW, BK = M::BK, K8 = BK / 8, BUFS = M::BUFS;
  constexpr int UW = kWaves / KS;                             // waves over units
  constexpr bool KEEP = UPW == 1;  // the small products' sums fit beside the high ones'
  constexpr int NI = (M::COLS * K8 + kThreads - 1) / kThreads;  // items per thread, at most
  extern __shared__ __align__(16) unsigned char gram_lds[];
  uintx4* lds = (uintx4*)gram_lds;
  const int tid = threadIdx.x, lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int np = npair(K), n = nblk(K), NC = 64 * np, nu = upper_blocks(K);
  const int PLANE = K8 * NC, BUF = 3 * PLANE;
  const int64_t chunk = blockIdx.x, r0 = chunk * rows_per_chunk;
  const int64_t r1 = r0 + rows_per_chunk < rows ? r0 + rows_per_chunk : rows;
  const int u0 = blockIdx.y * upw;
  const int uend = min(u0 + upw, np * (np + 1) / 2);
  const int slice = w / UW;
  int pi[UPW], pj[UPW];
  bool has[UPW];
#pragma unroll
  for (int k = 0; k < UPW; k++) {
    const int u = u0 + w % UW + UW * k;
    has[k] = u < uend;
    pi[k] = pj[k] = 0;
    if (has[k]) upper_of(u, np, pi[k], pj[k]);
  }
  floatx16 acc[UPW][2][2];
#pragma unroll
  for (int k = 0; k < UPW; k++)
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int e = 0; e < 16; e++) acc[k][i][j][e] = 0.0f;
  floatx16 lo[KEEP ? 2 : 1][KEEP ? 2 : 1];
  if constexpr (KEEP) {
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int e = 0; e < 16; e++) lo[i][j][e] = 0.0f;
  }

  // item i of a thread: eight rows of one column (column fastest)
  unsigned v[NI][8];
  uint32_t off[NI];
  const uint32_t st = (uint32_t)K * 4;
#pragma unroll
  for (int i = 0; i < NI; i++) {
    const int c = tid + kThreads * i, col = c % NC, k8 = c / NC;
    off[i] = k8 < K8 && col < K ? (uint32_t)(8 * k8 * K + col) * 4 : kOutside;
  }
  auto fetch = [&](int64_t s0) {
    // a view of the chunk's rest: rows past it read as zeros
    const __amdgpu_buffer_rsrc_t view = tile_view(X + s0 * K, (r1 - s0) * K * 4);
    if (s0 + BK <= r1) {
#pragma unroll
      for (int i = 0; i < NI; i++)
#pragma unroll
        for (int q = 0; q < 8; q++)
          v[i][q] = __builtin_amdgcn_raw_buffer_load_b32(view, off[i], q * st, 0);
    } else {
#pragma unroll
      for (int i = 0; i < NI; i++)
#pragma unroll
        for (int q = 0; q < 8; q++)
          v[i][q] = __builtin_amdgcn_raw_buffer_load_b32(view, off[i] != kOutside ? off[i] + q * st : kOutside, 0, 0);
    }
  };
  auto put = [&](int b) {
#pragma unroll
    for (int i = 0; i < NI; i++) {
      const int c = tid + kThreads * i;
      if (c >= PLANE) continue;
      uintx4 h, m, l;
      split8(v[i], h, m, l);
      uintx4* d = lds + b * BUF + c;
      d[0] = h;
      d[PLANE] = m;
      d[2 * PLANE] = l;
    }
  };
  auto products = [&](int b) {
#pragma unroll
    for (int k = 0; k < UPW; k++) {
      if (!has[k]) continue;
#pragma unroll
      for (int ss = 0; ss < BK / 16 / KS; ss++) {
        const int s = KS > 1 ? slice : ss;
        const uintx4* base = lds + b * BUF + (2 * s + (lane >> 5)) * NC + (lane & 31);
        bf16x8 a[3][2], c[3][2];
#pragma unroll
        for (int p = 2; p >= 0; p--)
#pragma unroll
          for (int i = 0; i < 2; i++) {
            a[p][i] = __builtin_bit_cast(bf16x8, base[p * PLANE + 64 * pi[k] + 32 * i]);
            c[p][i] = __builtin_bit_cast(bf16x8, base[p * PLANE + 64 * pj[k] + 32 * i]);
          }
        auto mul = [&](int p, int q, int i, int j, floatx16& x) {
          x = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[p][i], c[q][j], x, 0, 0, 0);
        };
#pragma unroll
        for (int i = 0; i < 2; i++) {
          floatx16 t[2];
          if constexpr (!KEEP) {
#pragma unroll
            for (int j = 0; j < 2; j++)
#pragma unroll
              for (int e = 0; e < 16; e++) t[j][e] = 0.0f;
          }
#pragma unroll
          for (int j = 0; j < 2; j++) {
            floatx16& x = KEEP ? lo[KEEP ? i : 0][KEEP ? j : 0] : t[j];
            mul(2, 0, i, j, x);
            mul(0, 2, i, j, x);
            mul(1, 1, i, j, x);
            mul(1, 0, i, j, x);
            mul(0, 1, i, j, x);
            mul(0, 0, i, j, acc[k][i][j]);
          }
          if constexpr (!KEEP) {
#pragma unroll
            for (int j = 0; j < 2; j++) {
              acc[k][i][j] += t[j];
              asm volatile("" : "+v"(acc[k][i][j]));  // added here and now: registers
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      }
    }
  };

  const int ns = (int)((r1 - r0 + BK - 1) / BK);
  fetch(r0);
  put(0);
  if (ns > 1) fetch(r0 + BK);
  __syncthreads();
  // Stage t is computed while stage t + 1 goes from registers to the other LDS
  // buffer and stage t + 2 is loaded.  The waves of one half store first, those
  // of the other compute first, so that on every SIMD one wave's splitting runs
  // beside the other's matrix-core products.
#pragma unroll 1
  for (int t = 0; t < ns; t++) {
    if constexpr (BUFS == 2) {
      const int b = t & 1;
      if (w >= kWaves / 2) products(b);
      if (t + 1 < ns) {
        put(b ^ 1);
        if (t + 2 < ns) fetch(r0 + (int64_t)(t + 2) * BK);
      }
      if (w < kWaves / 2) products(b);
      __syncthreads();
    } else {
      products(0);
      __syncthreads();
      if (t + 1 < ns) {
        put(0);
        if (t + 2 < ns) fetch(r0 + (int64_t)(t + 2) * BK);
        __syncthreads();
      }
    }
  }

  if constexpr (KEEP) {
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++) acc[0][i][j] += lo[i][j];
  }
  // Rare: sums of the parts that are not finite (an infinite value's lower parts are
  // NaN) are formed again from the values, on the FP32 matrix cores.
#pragma unroll
  for (int k = 0; k < UPW; k++) {
    float z = 0.0f;
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++)
#pragma unroll
        for (int e = 0; e < 16; e++) z = fmaf(acc[k][i][j][e], 0.0f, z);
    if (!has[k] || !__any(z != z)) continue;
    const int half = lane >> 5, l = lane & 31;
    // the share's rows: 16 of every stage (all of it where a stage is one share's)
    constexpr int n = BK / KS;
#pragma unroll 1
    for (int i = 0; i < 2; i++)
#pragma unroll 1
      for (int j = 0; j < 2; j++) {
        floatx16 x;
#pragma unroll
        for (int e = 0; e < 16; e++) x[e] = 0.0f;
        const int ca = 64 * pi[k] + 32 * i + l, cb = 64 * pj[k] + 32 * j + l;
#pragma unroll 1
        for (int64_t s0 = r0 + n * slice; s0 < r1; s0 += BK) {
          float a[n / 2], b[n / 2];
#pragma unroll
          for (int q = 0; q < n / 2; q++) {
            const int64_t r = s0 + 2 * q + half;
            a[q] = r < r1 && ca < K ? X[r * K + ca] : 0.0f;
            b[q] = r < r1 && cb < K ? X[r * K + cb] : 0.0f;
          }
#pragma unroll
          for (int q = 0; q < n / 2; q++) x = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q], b[q], x, 0, 0, 0);
        }
#pragma unroll
        for (int ii = 0; ii < 2; ii++)
#pragma unroll
          for (int jj = 0; jj < 2; jj++)
#pragma unroll
            for (int e = 0; e < 16; e++)
              if (ii == i && jj == j && !isfinite(acc[k][ii][jj][e])) acc[k][ii][jj][e] = x[e];
      }
  }
  // lane holds C block row 8 jj + 4 h + ii, column lane % 32, in acc[4 jj + ii]
  const int h = lane >> 5, m = lane & 31;
  auto put_blocks = [&](int k, auto value) {
#pragma unroll
    for (int i = 0; i < 2; i++)
#pragma unroll
      for (int j = 0; j < 2; j++) {
        const int bi = 2 * pi[k] + i, bj = 2 * pj[k] + j;
        if (bi > bj || bj >= n) continue;
        const int u = bi * n - bi * (bi - 1) / 2 + (bj - bi);
        float* dst = partial + (chunk * nu + u) * 1024;
#pragma unroll
        for (int e = 0; e < 16; e++)
          dst[(8 * (e >> 2) + 4 * h + (e & 3)) * 32 + m] = value(i, j, e);
      }
  };
  if constexpr (KS == 1) {
#pragma unroll
    for (int k = 0; k < UPW; k++)
      if (has[k]) put_blocks(k, [&](int i, int j, int e) { return acc[k][i][j][e]; });
  } else {
    // the row shares of a unit, added in share order by the first share's wave
    float* sh = (float*)gram_lds + lane;
    if (slice > 0 && has[0]) {
#pragma unroll
      for (int i = 0; i < 2; i++)
#pragma unroll
        for (int j = 0; j < 2; j++)
#pragma unroll
          for (int e = 0; e < 16; e++) sh[(w - UW) * 4096 + ((2 * i + j) * 16 + e) * 64] = acc[0][i][j][e];
    }
    __syncthreads();
    if (slice == 0 && has[0])
      put_blocks(0, [&](int i, int j, int e) {
        float t = acc[0][i][j][e];
#pragma unroll
        for (int q = 1; q < KS; q++) t += sh[(w + (q - 1) * UW) * 4096 + ((2 * i + j) * 16 + e) * 64];
        return t;
      });
  }
}

// C[K][K] from the partials: workgroup (u, part) handles 32 float4 of block u;
// thread (f, sl) sums chunks sl, sl + 16, ... of float4 f, then slice 0 adds
// the 16 slice sums in slice order.
constexpr int kRedSlices = 16;
constexpr int kRedThreads = 32 * kRedSlices;

// Panel entry of C[l][col] for the tile products of the column updates (the B
// operand of the tile of col, contraction row l): 1 - C or 0 on the diagonal,
// 0 for l inside the tile and left of col, -C elsewhere.  Same layout as the
// update kernels read: panel[j][l][c] (l < kpad(K), c < 32), then gblk[j][t][c].
// The same entries in the H rows kernel's staging order, one block of
// NB * NT * 1024 + tile^2 floats per tile (NT = ceil(K / 32), NB = max(1,
// tile / 32)): entry (l, c) of the tile's panel at
// ((((c / 32) NT + l / 32) 4 + s / 4) 2 + l % 2) 32 + c % 32) 4 + s % 4 with
// s = (l % 32) / 2 -- lane (m, h) then reads rows 32 t + 2 (4 sq + i) + h of
// column m as one float4 -- then the G block split by column parity,
// [h][t][k] = G[t][2 k + h] where 2 k + h > t (zero elsewhere).
__device__ __forceinline__ void put_panel_rows(float* panel, int K, int diag_one, int tile, int l, int col,
                                               float v) {
  const int nt = (K + 31) / 32, nb = tile >= 32 ? tile / 32 : 1;
  const int64_t per_tile = (int64_t)nb * nt * 1024 + tile * tile;
  const int j = col / tile, c = col % tile, a0 = tile * j;
  float pv;
  if (l == col) pv = diag_one ? 1.0f - v : 0.0f;
  else if (l >= a0 && l < col) pv = 0.0f;
  else pv = -v;
  const int r = l & 31, s2 = r >> 1;
  float* pt = panel + j * per_tile;
  pt[(((((c >> 5) * nt + (l >> 5)) * 4 + (s2 >> 2)) * 2 + (r & 1)) * 32 + (c & 31)) * 4 + (s2 & 3)] = pv;
  const int t = l - a0;
  if (l / tile == j && c > t)
    pt[(int64_t)nb * nt * 1024 + (c & 1) * (tile * tile / 2) + t * (tile / 2) + (c >> 1)] = v;
}

// The same entries in the H split kernel's order (tiles of 32): per tile the three
// BF16 parts of the panel, [part][l / 8][column][l % 8] with l < 32 NT, then
// G[t][c] for c > t (zero elsewhere).
__device__ __forceinline__ void put_panel_split(float* panel, int K, int diag_one, int l, int col, float v) {
  const int nt = (K + 31) / 32, j = col / 32, c = col % 32, a0 = 32 * j;
  float pv;
  if (l == col) pv = diag_one ? 1.0f - v : 0.0f;
  else if (l >= a0 && l < col) pv = 0.0f;
  else pv = -v;
  unsigned char* tile = (unsigned char*)panel + (size_t)j * (3 * 32 * nt * 32 * 2 + 32 * 32 * 4);
  unsigned short* parts = (unsigned short*)tile;
  const unsigned x[8] = {__float_as_uint(pv), 0, 0, 0, 0, 0, 0, 0};
  uintx4 p[3];
  split8(x, p[0], p[1], p[2]);
#pragma unroll
  for (int q = 0; q < 3; q++)
    parts[((q * 4 * nt + l / 8) * 32 + c) * 8 + l % 8] = (unsigned short)(p[q][0] & 0xffffu);
  const int t = l - a0;
  if (l / 32 == j && c > t) ((float*)(tile + (size_t)3 * 32 * nt * 32 * 2))[t * 32 + c] = v;
}

__device__ __forceinline__ void put_panel(float* panel, int K, int diag_one, int tile, int l, int col,
                                          float v) {
  const int kp = (K + 7) / 8 * 8, ntiles = (K + tile - 1) / tile;
  const int j = col / tile, c = col % tile, a0 = tile * j;
  float pv;
  if (l == col) pv = diag_one ? 1.0f - v : 0.0f;
  else if (l >= a0 && l < col) pv = 0.0f;
  else pv = -v;
  panel[((int64_t)j * kp + l) * tile + c] = pv;
  if (l / tile == j)
    panel[(int64_t)ntiles * kp * tile + ((int64_t)j * tile + (l - a0)) * tile + c] = v;
}

__global__ __launch_bounds__(kRedThreads) void gram_reduce(const float* __restrict__ partial, int nchunks,
                                                    int K, float* __restrict__ C, int64_t ldc,
                                                    float* __restrict__ panel, int diag_one, int tile,
                                                    int order) {
  __shared__ floatx4 part[kRedThreads];
  const int nb = nblk(K), nu = upper_blocks(K);
  const int u = blockIdx.x / 8, piece = blockIdx.x % 8;
  const int t = threadIdx.x, f = piece * 32 + (t & 31), sl = t >> 5;
  floatx4 acc = floatx4{0, 0, 0, 0};
  int c = sl;
  for (; c + 3 * kRedSlices < nchunks; c += 4 * kRedSlices) {
    const floatx4 a0 = *(const floatx4*)(partial + ((int64_t)c * nu + u) * 1024 + 4 * f);
    const floatx4 a1 = *(const floatx4*)(partial + ((int64_t)(c + kRedSlices) * nu + u) * 1024 + 4 * f);
    const floatx4 a2 = *(const floatx4*)(partial + ((int64_t)(c + 2 * kRedSlices) * nu + u) * 1024 + 4 * f);
    const floatx4 a3 = *(const floatx4*)(partial + ((int64_t)(c + 3 * kRedSlices) * nu + u) * 1024 + 4 * f);
    acc += a0;
    acc += a1;
    acc += a2;
    acc += a3;
  }
  for (; c < nchunks; c += kRedSlices)
    acc += *(const floatx4*)(partial + ((int64_t)c * nu + u) * 1024 + 4 * f);
  part[t] = acc;
  __syncthreads();
  if (sl == 0) {
    floatx4 tot = part[t];
    for (int k = 1; k < kRedSlices; k++) tot += part[k * 32 + (t & 31)];
    int bi, bj;
    {
      int uu = u, i = 0, rowlen = nb;
      while (uu >= rowlen) {
        uu -= rowlen;
        i++;
        rowlen--;
      }
      bi = i;
      bj = i + uu;
    }
    const int rr = (4 * f) / 32, cc = (4 * f) % 32;  // element (rr, cc..cc+3) of the block
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const int gi = 32 * bi + rr, gj = 32 * bj + cc + e;
      // both triangles from the upper one (a diagonal block's halves differ by
      // the order of the split products)
      if (gi <= gj && gj < K) {
        C[(int64_t)gi * ldc + gj] = tot[e];
        if (gi != gj) C[(int64_t)gj * ldc + gi] = tot[e];
        if (panel && order == kPanelSplit) {
          put_panel_split(panel, K, diag_one, gi, gj, tot[e]);
          if (gi != gj) put_panel_split(panel, K, diag_one, gj, gi, tot[e]);
        } else if (panel && order == kPanelRows) {
          put_panel_rows(panel, K, diag_one, tile, gi, gj, tot[e]);
          if (gi != gj) put_panel_rows(panel, K, diag_one, tile, gj, gi, tot[e]);
        } else if (panel) {
          put_panel(panel, K, diag_one, tile, gi, gj, tot[e]);
          if (gi != gj) put_panel(panel, K, diag_one, tile, gj, gi, tot[e]);
        }
      }
    }
  }
}

}  // namespace

constexpr int kMaxChunks = 256;
constexpr int64_t kSplitRows = 65536;  // rows from which the split kernel runs

size_t gram_partial_floats(int K) { return (size_t)kMaxChunks * upper_blocks(K) * 1024; }

namespace {
template <int MODE>
hipError_t launch_split(const float* X, int64_t rows, int K, int cus, float* partial, int* chunks,
                          hipStream_t s) {
  using M = Mode<MODE>;
  const int units = upper_units(K), slots = unit_slots<MODE>();
  const int ny = (units + slots - 1) / slots, upw = (units + ny - 1) / ny;
  // as many chunks as keep every CU busy once, of at least two stages (one
  // where a stage is long)
  const int64_t least = M::BK >= 64 ? M::BK : 64;
  int64_t nc = (rows + least - 1) / least;
  const int64_t most = std::min(kMaxChunks, std::max(1, cus / ny));
  if (nc > most) nc = most;
  int64_t rpc = (rows + nc - 1) / nc;
  rpc = (rpc + M::BK - 1) / M::BK * M::BK;
  nc = (rows + rpc - 1) / rpc;
  *chunks = (int)nc;
  const size_t bytes = lds_bytes<MODE>(K);
  if (bytes > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)gram_partial_split<MODE>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  gram_partial_split<MODE><<<dim3((unsigned)nc, (unsigned)ny), kThreads, bytes, s>>>(X, rows, K, rpc, upw, partial);
  return hipGetLastError();
}

template <int BPW, bool VEC>
hipError_t launch_fp32(const float* X, int64_t rows, int K, int cus, float* partial, int* chunks,
                       hipStream_t s) {
  int64_t nc = (rows + 63) / 64;
  if (nc > cus) nc = cus;
  if (nc > kMaxChunks) nc = kMaxChunks;
  const int64_t rpc = (rows + nc - 1) / nc;
  *chunks = (int)nc;
  const int ny = (upper_blocks(K) + kWaves * BPW - 1) / (kWaves * BPW);
  const int rs = stage_rows(K);
  const size_t bytes = (size_t)(rpc > rs ? 2 : 1) * rs * 32 * nblk(K) * 4;
  if (bytes > 65536) {
    const hipError_t e = hipFuncSetAttribute((const void*)gram_partial<BPW, VEC>,
                                             hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  gram_partial<BPW, VEC><<<dim3((unsigned)nc, (unsigned)ny), kThreads, bytes, s>>>(X, rows, K, rpc, rs, partial);
  return hipGetLastError();
}

template <bool VEC>
hipError_t launch_fp32_width(const float* X, int64_t rows, int K, int cus, float* partial, int* chunks,
                             hipStream_t s) {
  // blocks per wave: the fewest block times on the fullest CU, a staging of the
  // rows counted as most of one (10,000 x 240: two blocks, three workgroups per
  // chunk, 20.8 us, against 21.7 with four blocks and two)
  const int64_t nc = std::min<int64_t>(std::min(cus, kMaxChunks), (rows + 63) / 64);
  const int nu = upper_blocks(K);
  int best = 1;
  double least = 0.0;
  for (int b = 1; b <= 5; b++) {
    const int64_t wgs = nc * ((nu + kWaves * b - 1) / (kWaves * b));
    const double t = (double)((wgs + cus - 1) / cus) * (b + 0.7);
    if (b == 1 || t < least) {
      best = b;
      least = t;
    }
  }
  switch (best) {
    case 1: return launch_fp32<1, VEC>(X, rows, K, cus, partial, chunks, s);
    case 2: return launch_fp32<2, VEC>(X, rows, K, cus, partial, chunks, s);
    case 3: return launch_fp32<3, VEC>(X, rows, K, cus, partial, chunks, s);
    case 4: return launch_fp32<4, VEC>(X, rows, K, cus, partial, chunks, s);
    default: return launch_fp32<5, VEC>(X, rows, K, cus, partial, chunks, s);
  }
}
}  // namespace

hipError_t gram_xtx(const float* X, int64_t rows, int K, float* C, int64_t ldc, float* partial,
                    int cus, hipStream_t s, float* panel, int diag_one, int tile, int order) {
  if (K <= 0) return hipSuccess;
  if (K > kMaxK || rows < 1) return hipErrorInvalidValue;
  int chunks = 1;
  hipError_t e;
  if (rows < kSplitRows) {
    const bool vec = K % 4 == 0 && ((uintptr_t)X & 15) == 0;
    e = vec ? launch_fp32_width<true>(X, rows, K, cus, partial, &chunks, s)
            : launch_fp32_width<false>(X, rows, K, cus, partial, &chunks, s);
  } else switch (mode_of(K)) {
    case 0: e = launch_split<0>(X, rows, K, cus, partial, &chunks, s); break;
    case 1: e = launch_split<1>(X, rows, K, cus, partial, &chunks, s); break;
    default: e = launch_split<2>(X, rows, K, cus, partial, &chunks, s); break;
  }
  if (e != hipSuccess) return e;
  gram_reduce<<<(unsigned)(upper_blocks(K) * 8), kRedThreads, 0, s>>>(partial, chunks, K, C, ldc, panel,
                                                                diag_one, tile, order);
  return hipGetLastError();
}

}  // namespace plnmf
