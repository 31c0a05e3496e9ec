// Sparse products of the sweep on CSR inputs: R = A^T W (over the CSR of A^T,
// gathering rows of W) and P = A H^T (over the CSR of A, gathering rows of
// Ht); the sparse-matrix/dense-matrix products of Alg. 1 (R and P statements)
// and of the GPU implementation in Sec. 4.2.
//
// Design: one wave per work item.  Items are planned once on the host from the
// row pointers: consecutive short rows are grouped until an item holds about
// L nonzeros (empty rows included, written as zeros), and a row longer than L
// -- the Zipf-skewed head of a term-by-document matrix -- is cut into segments
// of L.  So the grid stays balanced whatever the row-length skew.  Each nonzero
// gathers one K-contiguous factor row with 16-byte (FP32) or 8-byte (BF16)
// lane loads, several nonzeros in flight per wave.  Segments of long rows
// leave partial rows that a second pass adds up in segment order; nothing
// else needs a second pass, and no atomics are used: results are
// bitwise-reproducible.
//
// Wide rows (K > 128: one nonzero per wave step) take a flat variant.  A wave
// walking an item row by row waits, per step, for a column index and then for
// the factor row it names, a dependent chain of global loads of which the
// machine holds too few in flight (the gathers themselves mostly hit the L2).
// The flat variant loads the item's row pointers, column indices and values
// into registers at once (the item bounds are known), then walks the item's
// nonzeros as one list, 16 gathers in flight per step, and writes out each row
// as its end is passed.  BF16 rows stay packed in registers until use, so a
// batch holds 16 nonzeros at K up to 512 (FP32 at K > 256: 8); measured on
// the 10^5 x 3*10^5 corpus at K = 400, the BF16 product of A^T W runs at half
// the FP32 time that way, while deeper FP32 batches (16, at 3 waves/SIMD)
// gain nothing -- the FP32 gathers are bound by the memory system there.
// Summation order within a row is the nonzero order, as in the row-by-row
// kernel.
#include <algorithm>
#include <vector>

#include "internal.hpp"

namespace plnmf {
namespace {

struct SpmmKArgs {
  const int32_t* rowptr;
  const int32_t* col;
  const void* val;
  const int4* items;
  const int32_t* slot;
  const void* X;
  float* out;
  float* carry;
  int64_t n_items, nnz;
  // without a host plan (n_rows > 0): waves of group_rows consecutive rows, then
  // seg_waves waves that share the *n_seg planned segments of the long rows
  int64_t n_rows;
  int group_rows, seg_waves;
  const int32_t* n_seg;
  int K;             // columns computed (a slice of the factor's columns, or all)
  int64_t ldx, ldo;  // row strides of the factor and of the output
};

template <typename T>
__device__ __forceinline__ float ld_val(const void* p, int64_t j) {
  return (float)((const T*)p)[j];
}

// 16 bytes at any float's address
typedef float any4 __attribute__((ext_vector_type(4), aligned(4)));

// VEC: FP32 rows of any rank from 4 on are read and written 16 bytes at a time,
// which needs 4-byte alignment only.  At a rank not divisible by 4 the last
// lane takes columns K-4..K-1 and repeats sums of its neighbour's: the same
// loads in the same order, so both write the same bits.  On 6,037 x 2,741
// with 165,000 nonzeros at K = 77 (both products): 65 us with scalar loads, 43 so.
// BF16: K % 4 == 0 and aligned rows; the flat kernel stores its sums where they are
// (the moved column costs the packed form eight registers, a wave per SIMD and 8% at
// K = 400).
__device__ __forceinline__ void st_x4(float* row, int c, int K, bool vec, floatx4 v) {
  if (vec) {
    if (c < K) *(any4*)(row + min(c, K - 4)) = v;
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (c + e < K) row[c + e] = v[e];
  }
}

// Load 4 consecutive elements of a factor row (columns c..c+3) as floats.
template <typename TX, bool VEC>
__device__ __forceinline__ floatx4 ld_x4(const TX* row, int c, int K) {
  floatx4 r;
  if constexpr (VEC) {
    if (c < K) {
      if constexpr (sizeof(TX) == 4) {
        r = *(const any4*)(row + min(c, K - 4));
      } else {
        bf16x4 b = *(const bf16x4*)(row + c);
        r = floatx4{(float)b[0], (float)b[1], (float)b[2], (float)b[3]};
      }
    } else {
      r = floatx4{0, 0, 0, 0};
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; e++) r[e] = (c + e < K) ? (float)row[c + e] : 0.0f;
  }
  return r;
}

// The same, as they lie in memory: a conversion of a predicated load, next to it,
// would wait for it.
template <typename TX>
struct Raw4 {
  typedef TX T __attribute__((ext_vector_type(4)));
};
template <typename TX, bool VEC>
__device__ __forceinline__ typename Raw4<TX>::T ld_raw4(const TX* row, int c, int K) {
  typename Raw4<TX>::T r = {(TX)0.0f, (TX)0.0f, (TX)0.0f, (TX)0.0f};
  if constexpr (!VEC) {
#pragma unroll
    for (int e = 0; e < 4; e++)
      if (c + e < K) r[e] = row[c + e];
  } else if constexpr (sizeof(TX) == 4) {
    if (c < K) r = *(const any4*)(row + min(c, K - 4));
  } else {
    if (c < K) r = *(const bf16x4*)(row + c);
  }
  return r;
}
template <typename T>
__device__ __forceinline__ floatx4 to_floats(T x) {
  return floatx4{(float)x[0], (float)x[1], (float)x[2], (float)x[3]};
}

constexpr int kMaxRowsPerItem = 256;
constexpr int kFlatMaxNnz = 128;  // item nonzeros the flat kernel prefetches

// The items of one wave, each passed to work(item, slot): the planned item, or
// without a host plan the runs of its rows that the plan would make (rows that
// together hold at most kFlatMaxNnz nonzeros; longer ones are left to their
// planned segments), or its share of those segments.
template <bool PLANNED, typename F>
__device__ __forceinline__ void wave_items(const SpmmKArgs& a, F work) {
  if constexpr (PLANNED) {
    const int64_t it = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    if (it < a.n_items) work(a.items[it], a.slot[it]);
    return;
  }
  const int lane = threadIdx.x & 63;
  int64_t i = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), end = 0, step = 1;
  int64_t r0 = 0;
  int ptr = 0;
  const int64_t row_waves = (a.n_rows + a.group_rows - 1) / a.group_rows;
  const bool rows = i < row_waves;
  if (rows) {
    r0 = i * a.group_rows;
    i = 0;
    end = a.n_rows - r0 < a.group_rows ? a.n_rows - r0 : a.group_rows;  // <= 32
    ptr = a.rowptr[r0 + (lane <= end ? lane : end)];
  } else {
    i -= row_waves;
    end = *a.n_seg;
    step = a.seg_waves;
  }
  while (i < end) {
    int4 item;
    int slot = -1;
    if (rows) {
      const int ii = (int)i, j0 = __builtin_amdgcn_readlane(ptr, ii);
      // rows ii .. ii + n - 1 end within kFlatMaxNnz of row ii's start
      const int n = __popcll(__ballot(lane > ii && lane <= end && ptr - j0 <= kFlatMaxNnz));
      i += n > 0 ? n : 1;
      if (n == 0) continue;  // a long row
      item = make_int4((int)r0 + ii, (int)r0 + ii + n, j0, __builtin_amdgcn_readlane(ptr, ii + n));
    } else {
      item = a.items[i];
      slot = a.slot[i];
      i += step;
    }
    work(item, slot);
  }
}

// The item's nonzeros row by row, NPAR side by side.  Few items are in flight on
// small inputs, so a row's chain of loads sets the time: UNR gathers a step,
// the indices of the next step (of the next row, at a row's end) read one step
// ahead, and the last step of a row filled up with zeros (0 * 0 added leaves a
// sum as it is) instead of taken one nonzero at a time.  BF16 values and rows stay as
// they are loaded until they are used.  Ranks of 33 to 128: eight gathers a step below
// 524,288 nonzeros, where the chain is what there is; four above, where waves in
// flight count more and eight take half as many registers again (FP32 / BF16, one
// product, before / eight / four: 6,037 x 2,741 with 165,000 nonzeros, K = 100, 20 / 11.5 /
// 13 and 31 / 16 / 17.5 us; 60,000 x 60,000 with 4.5 million, K = 96, 134 / 143 / 133 and
// 181 / 146 / 144 us).
template <int VPL, int LPN, typename TV, typename TX, bool VEC, int UNR>
__device__ __forceinline__ void items_wave(const SpmmKArgs& a, const int4 item, const int slot) {
  constexpr int NPAR = 64 / LPN;  // nonzeros processed side by side per wave
  const int lane = threadIdx.x & 63;
  const int grp = lane / LPN, q = lane % LPN;
  const int K = a.K;
  const TX* X = (const TX*)a.X;
  int32_t cc[UNR];
  TV vv[UNR];
  auto fetch = [&](int64_t j, int64_t end) {
#pragma unroll
    for (int u = 0; u < UNR; u++) {
      const bool in = j + u * NPAR < end;
      cc[u] = in ? a.col[j + u * NPAR] : -1;
      vv[u] = in ? ((const TV*)a.val)[j + u * NPAR] : (TV)0.0f;
    }
  };
  int64_t rs = item.z, re = min(a.rowptr[item.x + 1], item.w);
  fetch(rs + grp, re);
  for (int r = item.x; r < item.y; r++) {
    const int64_t re2 = r + 1 < item.y ? min(a.rowptr[r + 2], item.w) : re;
    floatx4 acc[VPL];
#pragma unroll
    for (int v = 0; v < VPL; v++) acc[v] = floatx4{0, 0, 0, 0};
    if (rs == re) fetch(re + grp, re2);
    while (rs < re) {
      typename Raw4<TX>::T x[UNR][VPL];
      TV w[UNR];
#pragma unroll
      for (int u = 0; u < UNR; u++) {
        w[u] = vv[u];
#pragma unroll
        for (int v = 0; v < VPL; v++) {
          x[u][v] = typename Raw4<TX>::T{(TX)0.0f, (TX)0.0f, (TX)0.0f, (TX)0.0f};
          if (cc[u] >= 0) x[u][v] = ld_raw4<TX, VEC>(X + (int64_t)cc[u] * a.ldx, 4 * (q + LPN * v), K);
        }
      }
      rs += UNR * NPAR;
      if (rs < re) fetch(rs + grp, re);
      else fetch(re + grp, re2);
#pragma unroll
      for (int u = 0; u < UNR; u++)
#pragma unroll
        for (int v = 0; v < VPL; v++) acc[v] += (float)w[u] * to_floats(x[u][v]);
    }
    rs = re;
    re = re2;
    // combine the NPAR lane groups (fixed butterfly order)
#pragma unroll
    for (int off = LPN; off < 64; off <<= 1)
#pragma unroll
      for (int v = 0; v < VPL; v++)
#pragma unroll
        for (int e = 0; e < 4; e++) acc[v][e] += __shfl_xor(acc[v][e], off);
    float* dst = slot >= 0 ? a.carry + (int64_t)slot * K : a.out + (int64_t)r * a.ldo;
    if (grp == 0) {
#pragma unroll
      for (int v = 0; v < VPL; v++) st_x4(dst, 4 * (q + LPN * v), K, VEC, acc[v]);
    }
  }
}

template <int VPL, int LPN, typename TV, typename TX, bool VEC, bool PLANNED, int UNR>
__global__ __launch_bounds__(256) void spmm_items(SpmmKArgs a) {
  wave_items<PLANNED>(a, [&](const int4 item, const int slot) {
    items_wave<VPL, LPN, TV, TX, VEC, UNR>(a, item, slot);
  });
}

// Element k of a register array spread over the wave (element 64 m + l in lane
// l of arr[m]); k is wave-uniform.
template <int N, typename V>
__device__ __forceinline__ V wave_elem(const V (&arr)[N], int k) {
  V v = arr[0];
#pragma unroll
  for (int m = 1; m < N; m++)
    if ((k >> 6) == m) v = arr[m];
  return __builtin_bit_cast(V, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), k & 63));
}

// EPL: factor elements per lane and load -- 4 (FP32 float4, or BF16 8-byte
// loads), or 8 (BF16 16-byte loads; K % 8 == 0, rows 16-byte aligned).
template <int VPL, typename TV, typename TX, bool VEC, int EPL, int UNR_>
__device__ __forceinline__ void flat_wave(const SpmmKArgs& a, const int4 item, const int slot) {
  static_assert(EPL == 4 || (EPL == 8 && VEC && sizeof(TX) == 2 && VPL == 1),
                "16-byte BF16 loads only");
  constexpr int NQ = EPL / 4;  // float4 accumulators per load
  constexpr int UNR = UNR_ ? UNR_ : ((EPL == 8 || VPL == 1) ? 16 : 8);  // gathers per batch
  constexpr int MZ = kFlatMaxNnz / 64;
  constexpr int MR = (kMaxRowsPerItem + 1 + 63) / 64;
  const int lane = threadIdx.x & 63;
  const int K = a.K;
  const TX* X = (const TX*)a.X;
  const int r0 = item.x, nr = item.y - item.x;
  const int j0 = item.z, nz = item.w - item.z;  // nz <= kFlatMaxNnz, nr <= kMaxRowsPerItem
  int32_t pc[MZ], prp[MR];
  float pv[MZ];
#pragma unroll
  for (int m = 0; m < MZ; m++) {
    const int i = lane + 64 * m;
    pc[m] = i < nz ? a.col[j0 + i] : 0;
    pv[m] = i < nz ? ld_val<TV>(a.val, j0 + i) : 0.0f;
  }
#pragma unroll
  for (int m = 0; m < MR; m++) {
    const int i = lane + 64 * m;
    prp[m] = i <= nr ? a.rowptr[r0 + i] : 0;
  }
  // end (item-local nonzero index) of local row r; a long row's segment ends at nz
  auto row_end = [&](int r) {
    const int e = wave_elem(prp, r + 1) - j0;
    return e < nz ? e : nz;
  };
  floatx4 acc[VPL * NQ];
#pragma unroll
  for (int v = 0; v < VPL * NQ; v++) acc[v] = floatx4{0, 0, 0, 0};
  int r = 0;
  int rend = nr > 0 ? row_end(0) : nz;
  auto flush = [&]() {
    float* dst = slot >= 0 ? a.carry + (int64_t)slot * K : a.out + (int64_t)(r0 + r) * a.ldo;
#pragma unroll
    for (int v = 0; v < VPL; v++) {
      const int cb = EPL * (lane + 64 * v);
#pragma unroll
      for (int q = 0; q < NQ; q++) {
        if constexpr (VEC && sizeof(TX) == 2) {
          if (cb < K) *(floatx4*)(dst + cb + 4 * q) = acc[v * NQ + q];
        } else {
          st_x4(dst, cb + 4 * q, K, VEC, acc[v * NQ + q]);
        }
        acc[v * NQ + q] = floatx4{0, 0, 0, 0};
      }
    }
    r++;
    rend = r < nr ? row_end(r) : nz;
  };
  if constexpr (EPL == 8) {
    // BF16 rows kept packed until use (4 VGPRs per nonzero), so twice as
    // many gathers are in flight per wave as with unpacked floats
    for (int jb = 0; jb < nz; jb += UNR) {
      bf16x8 xb[UNR];
#pragma unroll
      for (int u = 0; u < UNR; u++) {
        const int j = jb + u;
        const int64_t col = j < nz ? wave_elem(pc, j) : 0;
        const int cb = 8 * lane;
        xb[u] = (j < nz && cb < K) ? *(const bf16x8*)((const __bf16*)X + col * a.ldx + cb)
                                   : bf16x8{};
      }
#pragma unroll
      for (int u = 0; u < UNR; u++) {
        const int j = jb + u;
        if (j < nz) {
          while (j >= rend && r < nr) flush();
          const float vv = wave_elem(pv, j);
          const bf16x8 b = xb[u];
          acc[0] += vv * floatx4{(float)b[0], (float)b[1], (float)b[2], (float)b[3]};
          acc[1] += vv * floatx4{(float)b[4], (float)b[5], (float)b[6], (float)b[7]};
        }
      }
    }
  } else {
    for (int jb = 0; jb < nz; jb += UNR) {
      floatx4 x[UNR][VPL];
#pragma unroll
      for (int u = 0; u < UNR; u++) {
        const int j = jb + u;
        const int64_t col = j < nz ? wave_elem(pc, j) : 0;
#pragma unroll
        for (int v = 0; v < VPL; v++) {
          const int cb = EPL * (lane + 64 * v);
          x[u][v] = j < nz ? ld_x4<TX, VEC>(X + col * a.ldx, cb, K) : floatx4{0, 0, 0, 0};
        }
      }
#pragma unroll
      for (int u = 0; u < UNR; u++) {
        const int j = jb + u;
        if (j < nz) {
          while (j >= rend && r < nr) flush();  // rows that end here, empty ones included
          const float vv = wave_elem(pv, j);
#pragma unroll
          for (int v = 0; v < VPL; v++) acc[v] += vv * x[u][v];
        }
      }
    }
  }
  while (r < nr) flush();
}

template <int VPL, typename TV, typename TX, bool VEC, bool PLANNED, int EPL = 4, int UNR_ = 0>
__global__ __launch_bounds__(256) void spmm_flat(SpmmKArgs a) {
  wave_items<PLANNED>(a, [&](const int4 item, const int slot) {
    flat_wave<VPL, TV, TX, VEC, EPL, UNR_>(a, item, slot);
  });
}

// One workgroup per long row: add its segments' partial rows.  Thread (v, sl)
// sums columns 4v..4v+3 over segments sl, sl + S, ... (S slices, in order, four
// loads in flight), then slice 0 adds the S slice sums in slice order: a fixed
// order for a given K and segment count, so results are bitwise reproducible.
constexpr int kFixThreads = 512;

template <bool VEC>
__global__ __launch_bounds__(kFixThreads, 8) void spmm_fixup(const int32_t* __restrict__ fix,
                                                          int64_t n_fix,
                                                          const int32_t* __restrict__ n_fix_dev,
                                                          const float* __restrict__ carry,
                                                          float* __restrict__ out, int K,
                                                          int64_t ldo) {
  __shared__ floatx4 part[kFixThreads];
  if (n_fix_dev) n_fix = *n_fix_dev;
  const int nv = (K + 3) / 4;
  const int S = kFixThreads / nv > 0 ? kFixThreads / nv : 1;
  const int t = threadIdx.x;
  const int v = t % nv, sl = t / nv;
  for (int64_t i = blockIdx.x; i < n_fix; i += gridDim.x) {
    const int64_t r = fix[3 * i], first = fix[3 * i + 1], cnt = fix[3 * i + 2];
    floatx4 acc = floatx4{0, 0, 0, 0};
    if (sl < S && t < nv * S) {
      auto seg = [&](int64_t g) -> floatx4 {
        return ld_x4<float, VEC>(carry + (first + g) * K, 4 * v, K);
      };
      int64_t g = sl;
      for (; g + 3 * S < cnt; g += 4 * S) {
        const floatx4 x0 = seg(g), x1 = seg(g + S), x2 = seg(g + 2 * S), x3 = seg(g + 3 * S);
        acc += x0;
        acc += x1;
        acc += x2;
        acc += x3;
      }
      for (; g < cnt; g += S) acc += seg(g);
    }
    part[t] = acc;
    __syncthreads();
    if (sl == 0 && t < nv) {
      floatx4 tot = part[v];
      const int used = cnt < S ? (int)cnt : S;  // slices that had a segment
      for (int k = 1; k < used; k++) tot += part[k * nv + v];
      st_x4(out + r * ldo, 4 * v, K, VEC, tot);
    }
    __syncthreads();  // `part` is written again for the next row
  }
}

hipError_t launch_fixup(unsigned blocks, const int32_t* fix, int64_t n_fix, const int32_t* n_fix_dev,
                        const float* carry, float* out, int K, int64_t ldo, hipStream_t s) {
  if (K >= 4) spmm_fixup<true><<<blocks, kFixThreads, 0, s>>>(fix, n_fix, n_fix_dev, carry, out, K, ldo);
  else spmm_fixup<false><<<blocks, kFixThreads, 0, s>>>(fix, n_fix, n_fix_dev, carry, out, K, ldo);
  return hipGetLastError();
}

unsigned blocks_of(const SpmmKArgs& a) {
  if (a.n_rows == 0) return (unsigned)((a.n_items + 3) / 4);
  return (unsigned)(((a.n_rows + a.group_rows - 1) / a.group_rows + a.seg_waves + 3) / 4);
}

// FP32 products: 16-byte rows at every rank but 1 .. 3 (LPN 1); only these go
// without a host plan
template <int VPL, int LPN, int UNR, typename TV, typename TX>
hipError_t launch_u(const SpmmKArgs& a, bool vec, hipStream_t s) {
  const unsigned blocks = blocks_of(a);
  if (blocks == 0) return hipSuccess;
  if constexpr (sizeof(TX) == 4) {
    if (LPN == 1 && !vec) {
      if (a.n_rows > 0) spmm_items<1, 1, TV, TX, false, false, UNR><<<blocks, 256, 0, s>>>(a);
      else spmm_items<1, 1, TV, TX, false, true, UNR><<<blocks, 256, 0, s>>>(a);
    } else if (a.n_rows > 0) {
      spmm_items<VPL, LPN, TV, TX, true, false, UNR><<<blocks, 256, 0, s>>>(a);
    } else {
      spmm_items<VPL, LPN, TV, TX, true, true, UNR><<<blocks, 256, 0, s>>>(a);
    }
  } else {
    if (vec) spmm_items<VPL, LPN, TV, TX, true, true, UNR><<<blocks, 256, 0, s>>>(a);
    else spmm_items<VPL, LPN, TV, TX, false, true, UNR><<<blocks, 256, 0, s>>>(a);
  }
  return hipGetLastError();
}

constexpr int64_t kFewNnz = 4096 * kFlatMaxNnz;  // below, less than a full item per wave slot

template <int VPL, int LPN, typename TV, typename TX>
hipError_t launch_t(const SpmmKArgs& a, bool vec, hipStream_t s) {
  if constexpr (VPL == 1 && LPN >= 16) {
    if (a.nnz < kFewNnz) return launch_u<VPL, LPN, 8, TV, TX>(a, vec, s);
  }
  return launch_u<VPL, LPN, 4, TV, TX>(a, vec, s);
}

template <int VPL, typename TV, typename TX>
hipError_t launch_f(const SpmmKArgs& a, bool vec, hipStream_t s) {
  const unsigned blocks = blocks_of(a);
  if (blocks == 0) return hipSuccess;
  if constexpr (sizeof(TX) == 4) {
    if (a.n_rows > 0) spmm_flat<VPL, TV, TX, true, false><<<blocks, 256, 0, s>>>(a);
    else spmm_flat<VPL, TV, TX, true, true><<<blocks, 256, 0, s>>>(a);
  } else {
    if (vec) spmm_flat<VPL, TV, TX, true, true><<<blocks, 256, 0, s>>>(a);
    else spmm_flat<VPL, TV, TX, false, true><<<blocks, 256, 0, s>>>(a);
  }
  return hipGetLastError();
}

template <typename TV, typename TX>
hipError_t launch_k(const SpmmKArgs& a, bool vec, bool vec8, bool flat, hipStream_t s) {
  const int n4 = (a.K + 3) / 4;
  if constexpr (sizeof(TX) == 2) {
    // BF16 rows longer than 256 elements: one 16-byte load of 8 per lane
    if (flat && n4 > 64 && vec8) {
      const unsigned blocks = blocks_of(a);
      if (blocks == 0) return hipSuccess;
      spmm_flat<1, TV, TX, true, true, 8><<<blocks, 256, 0, s>>>(a);
      return hipGetLastError();
    }
  }
  if (flat && n4 > 32) return n4 <= 64 ? launch_f<1, TV, TX>(a, vec, s) : launch_f<2, TV, TX>(a, vec, s);
  if (n4 <= 1) return launch_t<1, 1, TV, TX>(a, vec, s);
  if (n4 <= 2) return launch_t<1, 2, TV, TX>(a, vec, s);
  if (n4 <= 4) return launch_t<1, 4, TV, TX>(a, vec, s);
  if (n4 <= 8) return launch_t<1, 8, TV, TX>(a, vec, s);
  if (n4 <= 16) return launch_t<1, 16, TV, TX>(a, vec, s);
  if (n4 <= 32) return launch_t<1, 32, TV, TX>(a, vec, s);
  if (n4 <= 64) return launch_t<1, 64, TV, TX>(a, vec, s);
  return launch_t<2, 64, TV, TX>(a, vec, s);  // K <= 512
}

}  // namespace

int spmm_item_nnz(int64_t nnz) {
  (void)nnz;
  return 128;
}

SpmmSizes spmm_sizes(int64_t rows, int64_t nnz, int L) {
  SpmmSizes z;
  z.items = rows + 2 * (nnz / L) + 2;
  z.fix = nnz / L + 1;
  z.seg = 2 * (nnz / L) + 2;
  return z;
}

hipError_t spmm_build(SpmmPlan* p, hipStream_t s, const uint8_t* skip) {
  const int64_t rows = p->rows;
  const int L = p->L;
  std::vector<int32_t> rp((size_t)rows + 1);
  hipError_t e = hipMemcpyAsync(rp.data(), p->rowptr, rp.size() * sizeof(int32_t),
                                hipMemcpyDeviceToHost, s);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  std::vector<int4> items;
  std::vector<int32_t> slot, fix;
  int32_t nseg = 0;
  // short rows share an item of up to G nonzeros: L of them, or fewer where that
  // would leave less than four waves to a SIMD (a row's sums don't depend on it)
  const int64_t G = std::max<int64_t>(32, std::min<int64_t>(L, p->nnz / 4096));
  int64_t r = 0;
  while (r < rows) {
    const int64_t len = (int64_t)rp[r + 1] - rp[r];
    if (len > L && skip && skip[r]) {  // a long row computed elsewhere: no items
      r++;
      continue;
    }
    if (len > L) {  // a long row: segments of L nonzeros, summed by the fixup pass
      const int32_t first = nseg;
      int32_t cnt = 0;
      for (int64_t j = rp[r]; j < rp[r + 1]; j += L) {
        const int64_t je = std::min<int64_t>(j + L, rp[r + 1]);
        items.push_back(make_int4((int)r, (int)r + 1, (int)j, (int)je));
        slot.push_back(nseg++);
        cnt++;
      }
      fix.push_back((int32_t)r);
      fix.push_back(first);
      fix.push_back(cnt);
      r++;
      continue;
    }
    const int64_t r0 = r, j0 = rp[r];
    while (r < rows && r - r0 < kMaxRowsPerItem && (int64_t)rp[r + 1] - rp[r] <= L &&
           (r == r0 || (int64_t)rp[r + 1] - j0 <= G))
      r++;
    items.push_back(make_int4((int)r0, (int)r, (int)j0, (int)rp[r]));
    slot.push_back(-1);
  }
  const SpmmSizes cap = spmm_sizes(rows, p->nnz, L);
  if ((int64_t)items.size() > cap.items || (int64_t)fix.size() / 3 > cap.fix || nseg > cap.seg)
    return hipErrorInvalidValue;  // cannot happen: the bounds cover every partition
  p->n_items = (int64_t)items.size();
  p->n_fix = (int64_t)fix.size() / 3;
  p->n_seg = nseg;
  if (!items.empty()) {
    e = hipMemcpyAsync(p->items, items.data(), items.size() * sizeof(int4), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
    e = hipMemcpyAsync(p->item_slot, slot.data(), slot.size() * sizeof(int32_t),
                       hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
  }
  if (!fix.empty()) {
    e = hipMemcpyAsync(p->fix, fix.data(), fix.size() * sizeof(int32_t), hipMemcpyHostToDevice, s);
    if (e != hipSuccess) return e;
  }
  return hipStreamSynchronize(s);  // the host vectors go out of scope
}

hipError_t spmm(const SpmmPlan& p, Elem t, const void* X, int K, float* out, hipStream_t s) {
  return spmm_slice(p, t, X, K, 0, K, out, K, s);
}

hipError_t spmm_slice(const SpmmPlan& p, Elem t, const void* X0, int64_t ldx, int k0, int K,
                      float* out0, int64_t ldo, hipStream_t s) {
  const size_t esz = t == Elem::F32 ? 4 : 2;
  const void* X = (const char*)X0 + (size_t)k0 * esz;
  float* out = out0 + k0;
  SpmmKArgs a{};
  a.ldx = ldx;
  a.ldo = ldo;
  a.rowptr = p.rowptr;
  a.col = p.col;
  a.val = p.val;
  a.items = p.items;
  a.slot = p.item_slot;
  a.X = X;
  a.out = out;
  a.carry = p.carry;
  a.n_items = p.n_items;
  a.nnz = p.nnz;
  a.K = K;
  const bool vec = t == Elem::F32 ? K >= 4 : K % 4 == 0 && ldx % 4 == 0 && ldo % 4 == 0 &&
                                                (uintptr_t)X % 8 == 0 && (uintptr_t)out % 16 == 0 &&
                                                (uintptr_t)p.carry % 16 == 0;
  const bool vec8 = vec && K % 8 == 0 && ldx % 8 == 0 && ((uintptr_t)X) % 16 == 0;
  const bool flat = p.L <= kFlatMaxNnz;  // the flat kernel holds a whole item in registers
  hipError_t e = t == Elem::F32 ? launch_k<float, float>(a, vec, vec8, flat, s)
                                : launch_k<__bf16, __bf16>(a, vec, vec8, flat, s);
  if (e != hipSuccess) return e;
  if (p.n_fix > 0) {
    e = launch_fixup((unsigned)p.n_fix, p.fix, p.n_fix, nullptr, p.carry, out, K, ldo, s);
  }
  return e;
}

// For matrices used once (the new documents of a fold-in) the plan is made on the
// device: the long rows' segments by csr_check, the runs of short rows by each
// wave from the row pointers.  A call on 100,000 documents of
// 78 terms at K = 200 took 1,457 us with the host plan (row pointers down, a
// loop over the rows, items up, three synchronisations), 1,100 us without.
hipError_t spmm_unplanned(const SpmmPlan& p, const int32_t* counts, const float* X, int K, float* out,
                          hipStream_t s) {
  if (p.rows <= 0) return hipSuccess;
  SpmmKArgs a{};
  a.ldx = K;
  a.ldo = K;
  a.rowptr = p.rowptr;
  a.col = p.col;
  a.val = p.val;
  a.items = p.items;
  a.slot = p.item_slot;
  a.X = X;
  a.out = out;
  a.carry = p.carry;
  a.n_rows = p.rows;
  a.nnz = p.nnz;
  // rows per wave: as many as about one full item holds
  const int64_t mean = p.nnz / p.rows;
  a.group_rows = (int)std::max<int64_t>(1, std::min<int64_t>(kFlatMaxNnz / std::max<int64_t>(mean, 1), 32));
  const int64_t most = p.nnz / p.L;  // long rows, and half of their segments, at most
  a.seg_waves = (int)std::min<int64_t>(2 * most, 4096);
  a.n_seg = counts;
  a.K = K;
  hipError_t e = launch_k<float, float>(a, K >= 4, false, true, s);
  if (e != hipSuccess || most == 0) return e;
  return launch_fixup((unsigned)std::min<int64_t>(most, 512), p.fix, 0, counts + 1, p.carry, out, K, K, s);
}

// ------------------------------------------------------- CSR transpose ----
namespace {

__global__ void tr_count(const int32_t* __restrict__ rowptr, const int32_t* __restrict__ col,
                         int64_t rows, int64_t cols, int nblk, int32_t* __restrict__ cnt) {
  const int b = blockIdx.x;
  const int64_t r0 = rows * b / nblk, r1 = rows * (b + 1) / nblk;
  const int64_t j0 = rowptr[r0], j1 = rowptr[r1];
  for (int64_t j = j0 + threadIdx.x; j < j1; j += blockDim.x)
    atomicAdd(&cnt[(int64_t)b * cols + col[j]], 1);
}

// per column: exclusive running offsets over blocks; column total -> tot[c]
__global__ void tr_colscan(int32_t* __restrict__ cnt, int64_t cols, int nblk,
                           int32_t* __restrict__ tot) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= cols) return;
  int32_t run = 0;
  for (int b = 0; b < nblk; b++) {
    const int32_t t = cnt[(int64_t)b * cols + c];
    cnt[(int64_t)b * cols + c] = run;
    run += t;
  }
  tot[c] = run;
}

// single-workgroup exclusive scan of tot[0..n) into out[0..n], out[n] = total
__global__ __launch_bounds__(1024) void tr_scan(const int32_t* __restrict__ tot, int64_t n,
                                                int32_t* __restrict__ out) {
  __shared__ int64_t part[1024];
  const int t = threadIdx.x;
  const int64_t per = (n + 1023) / 1024;
  const int64_t b = per * t, e = b + per < n ? b + per : n;
  int64_t s = 0;
  for (int64_t i = b; i < e; i++) s += tot[i];
  part[t] = s;
  __syncthreads();
  if (t == 0) {
    int64_t run = 0;
    for (int i = 0; i < 1024; i++) {
      const int64_t v = part[i];
      part[i] = run;
      run += v;
    }
    out[n] = (int32_t)run;
  }
  __syncthreads();
  int64_t run = part[t];
  for (int64_t i = b; i < e; i++) {
    out[i] = (int32_t)run;
    run += tot[i];
  }
}

// one wave per row block, rows in order: keeps each output row sorted by the
// source row index (entries of one source row hit distinct columns)
__global__ __launch_bounds__(64) void tr_scatter(const int32_t* __restrict__ rowptr,
                                                 const int32_t* __restrict__ col,
                                                 const float* __restrict__ val, int64_t rows,
                                                 int64_t cols, int nblk, int32_t* __restrict__ cnt,
                                                 const int32_t* __restrict__ t_rowptr,
                                                 int32_t* __restrict__ t_col,
                                                 float* __restrict__ t_val) {
  const int b = blockIdx.x;
  const int64_t r0 = rows * b / nblk, r1 = rows * (b + 1) / nblk;
  int32_t* mycnt = cnt + (int64_t)b * cols;
  for (int64_t r = r0; r < r1; r++) {
    const int64_t j0 = rowptr[r], j1 = rowptr[r + 1];
    for (int64_t j = j0 + threadIdx.x; j < j1; j += 64) {
      const int32_t cc = col[j];
      const int32_t pos = t_rowptr[cc] + atomicAdd(&mycnt[cc], 1);
      t_col[pos] = (int32_t)r;
      t_val[pos] = val[j];
    }
    __threadfence_block();
  }
}

// One wave per row (the last wave checks the end pointers): every nonzero is
// checked by its own lane, so the long rows of a Zipf corpus cost no more than
// a few wave steps.
__global__ __launch_bounds__(256) void csr_check(int64_t rows, int64_t cols, int64_t nnz,
                                                 const int32_t* __restrict__ rowptr,
                                                 const int32_t* __restrict__ col,
                                                 const float* __restrict__ val,
                                                 int32_t* __restrict__ flag, CsrSegments seg) {
  const int64_t r = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (r > rows) return;
  if (r == rows) {
    if (lane == 0 && (rowptr[rows] != nnz || rowptr[0] != 0)) atomicOr(flag, 1);
    return;
  }
  const int64_t a = rowptr[r], b = rowptr[r + 1];
  if (a > b || a < 0 || b > nnz) {
    if (lane == 0) atomicOr(flag, 1);
    return;
  }
  if (seg.items && b - a > seg.L) {
    // a long row's segments: their places follow the order in which rows arrive,
    // what is added up does not
    const int cnt = (int)((b - a + seg.L - 1) / seg.L);
    int first = 0, f = 0;
    if (lane == 0) {
      first = atomicAdd(seg.counts, cnt);
      f = atomicAdd(seg.counts + 1, 1);
    }
    first = __builtin_amdgcn_readfirstlane(first);
    f = __builtin_amdgcn_readfirstlane(f);
    // room for every valid matrix; row pointers that are not could claim more
    if (first >= 0 && first + (int64_t)cnt <= seg.max_seg && f < seg.max_fix) {
      for (int i = lane; i < cnt; i += 64) {
        const int64_t j = a + (int64_t)i * seg.L;
        seg.items[first + i] = make_int4((int)r, (int)r + 1, (int)j, (int)(j + seg.L < b ? j + seg.L : b));
        seg.slot[first + i] = first + i;
      }
      if (lane < 3) seg.fix[3 * f + lane] = lane == 0 ? (int)r : lane == 1 ? first : cnt;
    }
  }
  int bad = 0;
  for (int64_t j = a + lane; j < b; j += 64) {
    const int32_t c = col[j];
    if (c < 0 || c >= cols || (j > a && col[j - 1] >= c)) bad |= 2;  // in range, strictly increasing
    const float v = val[j];
    if (!(v >= 0.0f) || isinf(v)) bad |= 4;
  }
  if (bad) atomicOr(flag, bad);
}

}  // namespace

int csr_transpose_blocks(int64_t rows, int64_t cols, size_t scratch_ints) {
  int64_t nb = (int64_t)(scratch_ints / (size_t)(cols > 0 ? cols : 1));
  if (nb > 1024) nb = 1024;
  if (nb > rows) nb = rows;
  if (nb < 1) nb = 1;
  return (int)nb;
}

hipError_t csr_transpose(int64_t rows, int64_t cols, int64_t nnz, const int32_t* rowptr,
                         const int32_t* col, const float* val, int32_t* t_rowptr, int32_t* t_col,
                         float* t_val, int32_t* scratch, int nblk, hipStream_t s) {
  // scratch layout: cnt [nblk * cols], tot [cols]
  int32_t* cnt = scratch;
  int32_t* tot = scratch + (int64_t)nblk * cols;
  hipError_t e = hipMemsetAsync(cnt, 0, sizeof(int32_t) * (size_t)nblk * (size_t)cols, s);
  if (e != hipSuccess) return e;
  if (rows > 0) tr_count<<<nblk, 256, 0, s>>>(rowptr, col, rows, cols, nblk, cnt);
  if (cols > 0) tr_colscan<<<(unsigned)((cols + 255) / 256), 256, 0, s>>>(cnt, cols, nblk, tot);
  tr_scan<<<1, 1024, 0, s>>>(tot, cols, t_rowptr);
  if (rows > 0)
    tr_scatter<<<nblk, 64, 0, s>>>(rowptr, col, val, rows, cols, nblk, cnt, t_rowptr, t_col, t_val);
  (void)nnz;
  return hipGetLastError();
}

hipError_t csr_validate(int64_t rows, int64_t cols, int64_t nnz, const int32_t* rowptr,
                        const int32_t* col, const float* val, int32_t* flag, hipStream_t s,
                        const CsrSegments& seg) {
  csr_check<<<(unsigned)((rows + 1 + 3) / 4), 256, 0, s>>>(rows, cols, nnz, rowptr, col, val, flag, seg);
  return hipGetLastError();
}

}  // namespace plnmf
