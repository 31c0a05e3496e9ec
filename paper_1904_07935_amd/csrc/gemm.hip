// Matrix-core GEMM for gfx950: C = op(A) op(B) with FP32 accumulation.
//
// Used for every dense product of the sweep (A H^T and A^T W on dense A, Alg. 1
// statements forming R and P), the dense-row block of P on sparse A, the dense
// residual of the objective (Eq. 2), the multiplicative updates' denominators,
// and the warm-start network's forward and backward products.
//
// FP32 operands run on the BF16 matrix cores.  Each FP32 value is split into
// three BF16 parts that add up to it exactly (8 + 8 + 8 significand bits), and
// a product x y is the sum of the six part products of order 2^-16 and above:
// xh yh + (xh ym + xm yh) + (xh yl + xm ym + xl yh).  What is left out, xm yl +
// xl ym + xl yl, is at most 2^-24 of the product and of either sign (RMS 5.3e-9;
// an FP32 rounding is at most 2^-24, RMS 2.5e-8).  Six v_mfma_f32_32x32x16_bf16
// cover 16 terms in 192 cycles per 32 x 32 block; eight v_mfma_f32_32x32x2_f32
// take 512.
//
// One operand layout serves both element types: lane l of the 32x32x16 product
// supplies A[l%32][8(l/32)..+7] and B[8(l/32)..+7][l%32], so a tile is staged in
// LDS as 16-byte chunks of 8 consecutive contraction terms, chunk (part, k/8,
// row) at [part][k/8][row]: a wave's operand read is 32 consecutive chunks per
// half, without bank conflicts, whichever way the operand lies in memory.  The
// split runs once per element on the way from registers to LDS.
// Output block layout: lane l holds C[8j + 4(l/32) + i][l%32], j,i < 4.
// Split-K writes FP32 partials that a pass adds in 64 bits and in a fixed order
// (deterministic).
//
// What bounds it and what it measured (kernel times, against the 128 x 128 kernel
// on the FP32 matrix cores that it replaced, same box): 10,000 x 240 x 10,000 FP32
// 502 -> 335 us (A H^T) and 488 -> 319 us (A^T W), with the splitting (about 5.5
// VALU instructions per element), the LDS and the matrix cores each near half of
// the time or above; the dense-row block (256 x 400 x 300,000) 707 -> 417 us; BF16
// 10,000 x 240 x 10,000 127 -> 92 us, bound by the latency of the operand loads;
// 1,000 x 16 x 800 33 and 28 -> 8.5 and 8 us, 4,096 x 100 x 100 32 -> 13 us,
// latency (small tiles, more splits).  Errors against 64 bits, RMS over all
// elements, FP32 matrix cores / here: 9.5e-8 / 9.4e-8 at 10,000 terms, 5.3e-8 /
// 2.7e-8 at 3,000, 6.6e-8 / 5.5e-8 at 100, 2.5e-8 / 2.6e-8 for single products.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "bf16x3.hpp"
#include "internal.hpp"

namespace plnmf {
namespace {

// Workgroup tiles.  BM x BN outputs by waves of 32 BI x 32 BJ; BK32 / BK16 terms
// of FP32 / BF16 operands per K-step; one LDS buffer, so that more workgroups
// fit on a CU and one's staging overlaps another's products, or two.
template <int CFG>
struct Tile;
template <>
struct Tile<0> {  // large products
  static constexpr int BM = 128, BN = 128, BI = 2, BJ = 2, BK32 = 32, BK16 = 64, BUFS = 1;
};
template <>
struct Tile<1> {  // few outputs: more workgroups
  static constexpr int BM = 64, BN = 64, BI = 1, BJ = 1, BK32 = 32, BK16 = 64, BUFS = 1;
};
template <>
struct Tile<2> {  // few tiles of 128 x 128, or narrow outputs
  static constexpr int BM = 128, BN = 32, BI = 1, BJ = 1, BK32 = 32, BK16 = 64, BUFS = 2;
};
template <int CFG>
constexpr int threads_of() {
  return 64 * (Tile<CFG>::BM / (32 * Tile<CFG>::BI)) * (Tile<CFG>::BN / (32 * Tile<CFG>::BJ));
}
template <typename T, int CFG>
constexpr int bk_of() {
  return sizeof(T) == 4 ? Tile<CFG>::BK32 : Tile<CFG>::BK16;
}
template <typename T>
constexpr int parts_of() {
  return sizeof(T) == 4 ? 3 : 1;
}
// LDS rows of a chunk plane: padded so that the eight lanes of one write cycle
// (consecutive k/8 of one or two rows) fall on different banks
template <int R, int BK>
constexpr int pitch_of() {
  return R + (BK >= 64 ? 1 : BK == 32 ? 2 : 4);
}
template <typename T, int CFG>
constexpr size_t lds_bytes_of() {
  constexpr int BK = bk_of<T, CFG>();
  return (size_t)Tile<CFG>::BUFS * parts_of<T>() * (BK / 8) *
         (pitch_of<Tile<CFG>::BM, BK>() + pitch_of<Tile<CFG>::BN, BK>()) * 16;
}

// Operand tiles are read through buffer descriptors whose base is the step's
// tile origin.  A lane whose element lies outside the matrix (a row past M or
// N, a term past the end of its split) uses an offset past the descriptor's
// range (kOutside): no branches, so the loads of a step issue back to back.
// Valid offsets stay below 2^31 bytes (leading dimensions of 2^22 or more, and
// BF16 rows that are not 4-byte aligned, take the element-wise path).
__device__ __forceinline__ float gelu_grad_f(float z) {
  float cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752f));
  float pdf = expf(-0.5f * z * z) * 0.39894228040143268f;
  return cdf + z * pdf;
}

// Global -> register -> LDS staging of one K-step of one operand: R rows (of A,
// or columns of B) by BK terms.  TR: the rows are contiguous in memory (a dword
// per lane, consecutive lanes along the rows), else the terms are (16 bytes per
// lane).  FAR: element-wise loads at 64-bit addresses, any alignment.
template <typename T, bool TR, bool FAR, int R, int BK, int NTHR>
struct Stage {
  static constexpr int K8 = BK / 8, RP = pitch_of<R, BK>();
  static constexpr bool F32 = sizeof(T) == 4;
  static constexpr bool PAIR = !F32 && TR && !FAR;  // a dword holds two rows of a term
  static constexpr int ITEMS = PAIR ? R / 2 * K8 : R * K8;
  static constexpr int NI = (ITEMS + NTHR - 1) / NTHR;
  static constexpr int REGS = F32 || PAIR ? 8 : 4;
  unsigned v[NI][REGS];
  uint32_t off[NI];  // byte offset of each item's first element from a step's tile origin

  static __device__ __forceinline__ void place(int i, int tid, int& r, int& k8, bool& in) {
    const int c = tid + NTHR * i;
    in = ITEMS % NTHR == 0 || c < ITEMS;
    if constexpr (PAIR) {
      r = 2 * (c % (R / 2));
      k8 = c / (R / 2);
    } else if constexpr (TR) {
      r = c % R;
      k8 = c / R;
    } else {
      r = c / K8;
      k8 = c % K8;
    }
  }

  __device__ __forceinline__ void init(int64_t ld, int64_t rows, int64_t r0, int tid) {
    if constexpr (!FAR) {
#pragma unroll
      for (int i = 0; i < NI; i++) {
        int r, k8;
        bool in;
        place(i, tid, r, k8, in);
        off[i] = in && r < rows - r0
                     ? (uint32_t)((TR ? 8 * k8 * ld + r : r * ld + 8 * k8) * (int64_t)sizeof(T))
                     : kOutside;
      }
    }
  }

  __device__ __forceinline__ void load(const T* __restrict__ X, int64_t ld, int64_t rows, int64_t r0,
                                       int64_t k0, int64_t ke, int64_t Kd, int tid) {
    const int rem = ke - k0 >= BK ? BK : (ke > k0 ? (int)(ke - k0) : 0);
    if constexpr (FAR) {
      const int left = rows - r0 >= R ? R : (int)(rows - r0);
#pragma unroll
      for (int i = 0; i < NI; i++) {
        int r, k8;
        bool in;
        place(i, tid, r, k8, in);
        T e[8];
#pragma unroll
        for (int q = 0; q < 8; q++) {
          const bool ok = in && r < left && 8 * k8 + q < rem;
          const int64_t kk = k0 + 8 * k8 + q;
          e[q] = ok ? (TR ? X[kk * ld + r0 + r] : X[(r0 + r) * ld + kk]) : (T)0.0f;
        }
        if constexpr (F32) {
#pragma unroll
          for (int q = 0; q < 8; q++) v[i][q] = __builtin_bit_cast(unsigned, e[q]);
        } else {
#pragma unroll
          for (int q = 0; q < 4; q++)
            v[i][q] = __builtin_bit_cast(unsigned, bf16x2{(__bf16)e[2 * q], (__bf16)e[2 * q + 1]});
        }
      }
    } else {
      constexpr int ES = sizeof(T);
      const int64_t o = TR ? k0 * ld + r0 : r0 * ld + k0;
      // one past the last element; an odd last BF16 row (column) is followed by
      // its padding element
      const int64_t wide = F32 ? 0 : 1;
      const int64_t end = TR ? (Kd - 1) * ld + ((rows + wide) & ~wide)
                             : (rows - 1) * ld + ((Kd + wide) & ~wide);
      const __amdgpu_buffer_rsrc_t view = tile_view(X + o, (end - o) * ES);
      const uint32_t st = (uint32_t)(ld * ES);
      if (rem == BK) {
        // every term in range: one vector offset per item, the rest scalar
#pragma unroll
        for (int i = 0; i < NI; i++) {
          if constexpr (TR) {
#pragma unroll
            for (int q = 0; q < 8; q++)
              v[i][q] = __builtin_amdgcn_raw_buffer_load_b32(view, off[i], q * st, 0);
          } else {
#pragma unroll
            for (int q = 0; q < REGS / 4; q++) {
              const uintx4 x = ld16(view, off[i] + 16 * q);
#pragma unroll
              for (int e = 0; e < 4; e++) v[i][4 * q + e] = x[e];
            }
          }
        }
      } else {
        // the ragged last step: dword by dword, terms past the end cleared
#pragma unroll
        for (int i = 0; i < NI; i++) {
          int r, k8;
          bool in;
          place(i, tid, r, k8, in);
          constexpr int PER = TR ? 1 : 4 / ES;
#pragma unroll
          for (int q = 0; q < REGS; q++) {
            const int k = 8 * k8 + PER * q;
            unsigned x = ld4(view, off[i] != kOutside && k < rem ? off[i] + (TR ? q * st : 4u * q) : kOutside);
            if (!F32 && !TR && k + 1 >= rem) x &= 0xffffu;
            v[i][q] = x;
          }
        }
      }
    }
  }

  __device__ __forceinline__ void store(uintx4* lds, int tid) const {
#pragma unroll
    for (int i = 0; i < NI; i++) {
      int r, k8;
      bool in;
      place(i, tid, r, k8, in);
      if (!in) continue;
      uintx4* d = lds + k8 * RP + r;
      if constexpr (F32) {
        uintx4 h, m, l;
        split8(v[i], h, m, l);
        d[0] = h;
        d[K8 * RP] = m;
        d[2 * K8 * RP] = l;
      } else if constexpr (PAIR) {
        uintx4 a, b;
#pragma unroll
        for (int q = 0; q < 4; q++) {
          a[q] = lo_halves(v[i][2 * q], v[i][2 * q + 1]);
          b[q] = hi_halves(v[i][2 * q], v[i][2 * q + 1]);
        }
        d[0] = a;
        d[1] = b;
      } else {
        d[0] = uintx4{v[i][0], v[i][1], v[i][2], v[i][3]};
      }
    }
  }
};

// Epilogue over one wave's BI x BJ blocks.  `acc[i][j]` is the 32x32 block at
// rows r0 + 32 i, cols c0 + 32 j.  The epilogue kind and whether the wave's
// block lies wholly inside C are template parameters: each instantiation is
// one straight run of element updates, with no per-element dispatch on the kind
// and, inside C, no bounds checks.
template <int EPI, bool FULL, int BI, int BJ>
__device__ __forceinline__ void epi_block(int64_t M, int64_t N, float* __restrict__ out,
                                          int64_t ldo, const float* __restrict__ bs,
                                          const float* Dm, int64_t ldd, void* C2, float* C,
                                          int64_t ldc, floatx16 (&acc)[BI][BJ], int64_t r0,
                                          int64_t c0, float mu_delta, float scale, double& ss,
                                          double (&cs)[BJ]) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int i = 0; i < BI; i++)
#pragma unroll
    for (int j = 0; j < BJ; j++)
#pragma unroll
      for (int jj = 0; jj < 4; jj++)
#pragma unroll
        for (int ii = 0; ii < 4; ii++) {
          const int64_t m = r0 + 32 * i + 8 * jj + 4 * (lane >> 5) + ii;
          const int64_t n = c0 + 32 * j + (lane & 31);
          if (!FULL && (m >= M || n >= N)) continue;
          const float v = acc[i][j][jj * 4 + ii];
          if constexpr (EPI == EPI_STORE) {
            out[m * ldo + n] = bs ? v + bs[n] : v;
          } else if constexpr (EPI == EPI_RESID_SQ) {
            const float e = Dm[m * ldd + n] - v;
            ss += (double)e * (double)e;
          } else if constexpr (EPI == EPI_BIAS_GELU) {
            const float z = v + bs[n];
            if (C) C[m * ldc + n] = z;
            ((__bf16*)C2)[m * ldc + n] = (__bf16)gelu_f(z);
          } else if constexpr (EPI == EPI_BIAS_SOFTPLUS) {
            const float z = v + bs[n];
            if (C) C[m * ldc + n] = z;
            ((float*)C2)[m * ldc + n] = softplus_f(z);
          } else if constexpr (EPI == EPI_GELU_GRAD) {
            const float d = v * gelu_grad_f(Dm[m * ldd + n]);
            ((__bf16*)C2)[m * ldc + n] = (__bf16)d;
            cs[j] += (double)d;
          } else if constexpr (EPI == EPI_OUT_GRAD) {
            const float z = v + bs[n];
            const float e = softplus_f(z) - Dm[m * ldd + n];
            ss += (double)e * (double)e;
            const float sg = z > 20.0f ? 1.0f : 1.0f / (1.0f + expf(-z));
            const float d = scale * e * sg;
            ((__bf16*)C2)[m * ldc + n] = (__bf16)d;
            cs[j] += (double)d;
          } else if constexpr (EPI == EPI_MU) {
            const float num = Dm[m * ldd + n], x = ((const float*)C2)[m * ldc + n];
            C[m * ldc + n] = x * num / (v + mu_delta);
          }
        }
}

// The epilogues each operand form is used with.
template <typename T, bool AT, bool BT>
__host__ __device__ constexpr bool epi_used(int epi) {
  if (epi == EPI_STORE) return true;
  if (sizeof(T) == 4) return (epi == EPI_MU && !AT && !BT) || (epi == EPI_RESID_SQ && !AT && BT);
  if (!AT && BT) return epi == EPI_BIAS_GELU || epi == EPI_BIAS_SOFTPLUS || epi == EPI_OUT_GRAD;
  return epi == EPI_GELU_GRAD && !AT && !BT;
}

// XCD-aware tile order.  Workgroups go to the eight XCDs round robin by
// linear id; this maps the ids that land on one XCD to a contiguous run of
// tiles, N-tile fastest, so the tiles that share an A row block (and, for a
// split, a B block) run on the same XCD and find it in that XCD's L2.  A
// bijection on [0, tiles) whatever the dispatch order.
__device__ __forceinline__ void tile_of(int& tx, int& ty, int& tz) {
  const unsigned gx = gridDim.x, gy = gridDim.y, gz = gridDim.z;
  const unsigned total = gx * gy * gz;
  const unsigned lin = blockIdx.x + gx * (blockIdx.y + gy * blockIdx.z);
  const unsigned xcd = lin & 7, q = lin >> 3, per = total >> 3, rem = total & 7;
  const unsigned t = xcd < rem ? xcd * (per + 1) + q : rem * (per + 1) + (xcd - rem) * per + q;
  ty = (int)(t % gy);
  tx = (int)((t / gy) % gx);
  tz = (int)(t / (gx * gy));
}

// Whether a wave's sums hold an infinity or a NaN.
template <int BI, int BJ>
__device__ __forceinline__ bool any_not_finite(const floatx16 (&x)[BI][BJ]) {
  float z = 0.0f;
#pragma unroll
  for (int i = 0; i < BI; i++)
#pragma unroll
    for (int j = 0; j < BJ; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) z = fmaf(x[i][j][e], 0.0f, z);
  return __any(z != z);
}

// An operand that is infinite, or above the largest BF16, leaves NaN in the sums
// of the parts where the values' own products are infinite or large.  Sums that are
// not finite are therefore formed again from the values, on the FP32 matrix cores
// and straight from memory; the others stay.
template <bool AT, bool BT, int BI, int BJ>
__device__ __forceinline__ void whole_products(const float* __restrict__ A, const float* __restrict__ B,
                                               int64_t lda, int64_t ldb, int64_t M, int64_t N, int64_t r0,
                                               int64_t c0, int64_t kb, int64_t ke, floatx16 (&tot)[BI][BJ]) {
  const int lane = threadIdx.x & 63, h = lane >> 5, l = lane & 31;
  floatx16 x[BI][BJ];
#pragma unroll
  for (int i = 0; i < BI; i++)
#pragma unroll
    for (int j = 0; j < BJ; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) x[i][j][e] = 0.0f;
#pragma unroll 1
  for (int64_t k0 = kb; k0 < ke; k0 += 8) {
    float a[4][BI], b[4][BJ];  // one memory round trip for eight terms
#pragma unroll
    for (int q = 0; q < 4; q++) {
      const int64_t k = k0 + 2 * q + h;
#pragma unroll
      for (int i = 0; i < BI; i++) {
        const int64_t m = r0 + 32 * i + l;
        a[q][i] = m < M && k < ke ? (AT ? A[k * lda + m] : A[m * lda + k]) : 0.0f;
      }
#pragma unroll
      for (int j = 0; j < BJ; j++) {
        const int64_t n = c0 + 32 * j + l;
        b[q][j] = n < N && k < ke ? (BT ? B[n * ldb + k] : B[k * ldb + n]) : 0.0f;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; q++)
#pragma unroll
      for (int i = 0; i < BI; i++)
#pragma unroll
        for (int j = 0; j < BJ; j++)
          x[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[q][i], b[q][j], x[i][j], 0, 0, 0);
  }
#pragma unroll
  for (int i = 0; i < BI; i++)
#pragma unroll
    for (int j = 0; j < BJ; j++)
#pragma unroll
      for (int e = 0; e < 16; e++)
        if (!isfinite(tot[i][j][e])) tot[i][j][e] = x[i][j][e];
}

// Main loop.  One LDS buffer (128 x 128 and 64 x 64): the next step's loads are
// issued before a step's products and stored (split) after the barrier that
// follows them.  Two buffers (128 x 32): the step after goes to the other buffer,
// and BF16, whose products take less time than a load, loads two steps ahead.
//
// FP32: the matrix core adds the products of eight terms, cut to 2^-23 of the
// largest, and rounds the sum into the accumulator; an accumulator smaller than
// the sum is cut.  So the high products and the small ones (2^-8 of them and less)
// have accumulators of their own.  The small ones' runs through the whole
// contraction and is added at the end: its roundings are 2^-8 of the others'.  The
// high ones' takes a step's 32 terms and is then added to the running total: a
// single chain over n terms carries a rounding error that grows like the square
// root of its length.  Single products are off by 2.6e-8 (RMS) and 1.0e-7 at most;
// with one accumulator for both it was 4.1e-8 and 2.9e-7, on the FP32 matrix cores
// 2.5e-8 and 6e-8.
// BF16: one chain.  The inputs' rounding (2^-9 relative) dwarfs the FP32
// chain's, and at BF16 rates the chunk additions would cost as much VALU time
// as the products take on the matrix cores.
template <typename T, bool AT, bool BT, bool FAR, int CFG>
__global__ __launch_bounds__(threads_of<CFG>(), 2) void gemm_kernel(GemmArgs g) {
  using Tl = Tile<CFG>;
  constexpr int BM = Tl::BM, BN = Tl::BN, BI = Tl::BI, BJ = Tl::BJ, BK = bk_of<T, CFG>();
  constexpr int NTHR = threads_of<CFG>(), NWN = BN / (32 * BJ), K8 = BK / 8, PL = parts_of<T>();
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int NB = Tl::BUFS, DIST = F32 || NB == 1 ? 1 : 2, STEPS = 2;
  using SA = Stage<T, AT, FAR, BM, BK, NTHR>;
  using SB = Stage<T, !BT, FAR, BN, BK, NTHR>;
  constexpr int RPA = SA::RP, RPB = SB::RP, ABUF = PL * K8 * RPA, BUF = ABUF + PL * K8 * RPB;
  extern __shared__ __align__(16) unsigned char gemm_lds[];
  uintx4* lds = (uintx4*)gemm_lds;
  // scalar copies of the argument block (keeps its address untaken)
  const T* __restrict__ A = (const T*)g.A;
  const T* __restrict__ B = (const T*)g.B;
  const int64_t M = g.M, N = g.N, Kd = g.Kd, lda = g.lda, ldb = g.ldb;
  const int splits = g.splits;
  int tx, ty, tz;
  tile_of(tx, ty, tz);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int wm = w / NWN, wn = w % NWN;
  const int64_t m0 = (int64_t)tx * BM, n0 = (int64_t)ty * BN;
  int64_t kb = 0, ke = Kd;
  if (splits > 1) {
    kb = (int64_t)tz * g.k_per_split;
    ke = kb + g.k_per_split < Kd ? kb + g.k_per_split : Kd;
  }
  const int nk = (int)((ke - kb + BK - 1) / BK);
  floatx16 tot[BI][BJ];
#pragma unroll
  for (int i = 0; i < BI; i++)
#pragma unroll
    for (int j = 0; j < BJ; j++)
#pragma unroll
      for (int e = 0; e < 16; e++) tot[i][j][e] = 0.0f;

  floatx16 lo[F32 ? BI : 1][F32 ? BJ : 1];
  if constexpr (F32) {
#pragma unroll
    for (int i = 0; i < BI; i++)
#pragma unroll
      for (int j = 0; j < BJ; j++)
#pragma unroll
        for (int e = 0; e < 16; e++) lo[i][j][e] = 0.0f;
  }

  SA sa[DIST];
  SB sb[DIST];
#pragma unroll
  for (int s = 0; s < DIST; s++) {
    sa[s].init(lda, M, m0, tid);
    sb[s].init(ldb, N, n0, tid);
  }
  auto fetch = [&](int s, int kt) {
    const int64_t k0 = kb + (int64_t)kt * BK;
    sa[s].load(A, lda, M, m0, k0, ke, Kd, tid);
    sb[s].load(B, ldb, N, n0, k0, ke, Kd, tid);
  };
  auto put = [&](int s, int b) {
    sa[s].store(lds + b * BUF, tid);
    sb[s].store(lds + b * BUF + ABUF, tid);
  };
  auto products = [&](int b) {
    const uintx4* la = lds + b * BUF + (lane >> 5) * RPA + wm * 32 * BI + (lane & 31);
    const uintx4* lb = lds + b * BUF + ABUF + (lane >> 5) * RPB + wn * 32 * BJ + (lane & 31);
    auto read_a = [&](int s, int p, int i) {
      return __builtin_bit_cast(bf16x8, la[(p * K8 + 2 * s) * RPA + 32 * i]);
    };
    auto read_b = [&](int s, int p, int j) {
      return __builtin_bit_cast(bf16x8, lb[(p * K8 + 2 * s) * RPB + 32 * j]);
    };
    auto mul = [](bf16x8 x, bf16x8 y, floatx16& c) {
      c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, y, c, 0, 0, 0);
    };
    if constexpr (F32) {
      // One block after the other, its products in the order high, middle and low
      // part of B; each part is read during the products of the part before.  The
      // next row of blocks starts at the column where this one ends, whose B is there.
      constexpr int S = BK / 16;
      bf16x8 a[3][S], c[3][S];
      auto load_a = [&](int p, int i) {
#pragma unroll
        for (int s = 0; s < S; s++) a[p][s] = read_a(s, p, i);
      };
      auto load_b = [&](int p, int j) {
#pragma unroll
        for (int s = 0; s < S; s++) c[p][s] = read_b(s, p, j);
      };
      load_a(0, 0);
      load_b(0, 0);
      load_a(2, 0);
      load_a(1, 0);
#pragma unroll
      for (int i = 0; i < BI; i++) {
#pragma unroll
        for (int jj = 0; jj < BJ; jj++) {
          const int j = i & 1 ? BJ - 1 - jj : jj;
          const bool have_b = i > 0 && jj == 0, last_j = jj + 1 == BJ, last = last_j && i + 1 == BI;
          floatx16 hi;
#pragma unroll
          for (int e = 0; e < 16; e++) hi[e] = 0.0f;
          if (!have_b) load_b(1, j);
#pragma unroll
          for (int s = 0; s < S; s++) {
            mul(a[0][s], c[0][s], hi);
            mul(a[2][s], c[0][s], lo[i][j]);
            mul(a[1][s], c[0][s], lo[i][j]);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (!have_b) load_b(2, j);
          if (last_j && !last) load_a(2, i + 1);
#pragma unroll
          for (int s = 0; s < S; s++) {
            mul(a[0][s], c[1][s], lo[i][j]);
            mul(a[1][s], c[1][s], lo[i][j]);
          }
          __builtin_amdgcn_sched_barrier(0);
          if (!last_j) load_b(0, i & 1 ? j - 1 : j + 1);
          if (last_j && !last) load_a(1, i + 1);
#pragma unroll
          for (int s = 0; s < S; s++) mul(a[0][s], c[2][s], lo[i][j]);
          tot[i][j] += hi;
          // added here and now: the next block takes hi's registers
          asm volatile("" : "+v"(tot[i][j]));
          if (last_j && !last) load_a(0, i + 1);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    } else {
#pragma unroll
      for (int s = 0; s < BK / 16; s++) {
        bf16x8 a[BI], c[BJ];
#pragma unroll
        for (int i = 0; i < BI; i++) a[i] = read_a(s, 0, i);
#pragma unroll
        for (int j = 0; j < BJ; j++) c[j] = read_b(s, 0, j);
#pragma unroll
        for (int i = 0; i < BI; i++)
#pragma unroll
          for (int j = 0; j < BJ; j++) mul(a[i], c[j], tot[i][j]);
      }
    }
  };
  if (nk > 0) {
#pragma unroll
    for (int s = 0; s < DIST; s++)
      if (s < nk) fetch(s, s);
    put(0, 0);
    __syncthreads();
  }
#pragma unroll 1
  for (int kt = 0; kt < nk; kt += STEPS) {
#pragma unroll
    for (int u = 0; u < STEPS; u++) {
      if (kt + u < nk) {
        if (kt + u + DIST < nk) fetch(u % DIST, kt + u + DIST);
        products(u % NB);
        if (NB == 1) __syncthreads();
        if (kt + u + 1 < nk) put((u + 1) % DIST, (u + 1) % NB);
        __syncthreads();
      }
    }
  }

  if constexpr (F32) {
#pragma unroll
    for (int i = 0; i < BI; i++)
#pragma unroll
      for (int j = 0; j < BJ; j++) tot[i][j] += lo[i][j];
    if (any_not_finite(tot))  // rare
      whole_products<AT, BT, BI, BJ>(A, B, lda, ldb, M, N, m0 + wm * 32 * BI, n0 + wn * 32 * BJ, kb, ke, tot);
    // results over the operand: every wave has its products
    if (g.epi == EPI_MU && g.C == (const float*)g.A) __syncthreads();
  }

  const bool split = splits > 1;
  float* out = split ? g.partial + (int64_t)tz * M * N : g.C;
  const int64_t ldo = split ? N : g.ldc;
  const int64_t r0 = m0 + wm * 32 * BI, c0 = n0 + wn * 32 * BJ;
  const bool full = r0 + 32 * BI <= M && c0 + 32 * BJ <= N;
  const float* bias = split ? nullptr : g.bias;
  double ss = 0.0, cs[BJ];
#pragma unroll
  for (int j = 0; j < BJ; j++) cs[j] = 0.0;
#define PLNMF_EPI(E)                                                                           \
  if constexpr (epi_used<T, AT, BT>(E)) {                                                      \
    if (g.epi == E) {                                                                          \
      if (full)                                                                                \
        epi_block<E, true, BI, BJ>(M, N, out, ldo, bias, g.D, g.ldd, g.C2, g.C, g.ldc, tot, r0, \
                                   c0, g.mu_delta, g.scale, ss, cs);                           \
      else                                                                                     \
        epi_block<E, false, BI, BJ>(M, N, out, ldo, bias, g.D, g.ldd, g.C2, g.C, g.ldc, tot,    \
                                    r0, c0, g.mu_delta, g.scale, ss, cs);                      \
    }                                                                                          \
  }
  PLNMF_EPI(EPI_STORE)
  PLNMF_EPI(EPI_RESID_SQ)
  PLNMF_EPI(EPI_BIAS_GELU)
  PLNMF_EPI(EPI_BIAS_SOFTPLUS)
  PLNMF_EPI(EPI_GELU_GRAD)
  PLNMF_EPI(EPI_MU)
  PLNMF_EPI(EPI_OUT_GRAD)
#undef PLNMF_EPI
  constexpr bool kSums = epi_used<T, AT, BT>(EPI_RESID_SQ) || epi_used<T, AT, BT>(EPI_OUT_GRAD);
  constexpr bool kCols = epi_used<T, AT, BT>(EPI_GELU_GRAD) || epi_used<T, AT, BT>(EPI_OUT_GRAD);
  double* red = (double*)gemm_lds;  // the operand tiles are no longer read
  if constexpr (kSums) {
    if (g.epi == EPI_RESID_SQ || g.epi == EPI_OUT_GRAD) {
      for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
      if (lane == 0) red[w] = ss;
      __syncthreads();
      if (tid == 0) {
        double t = 0.0;
        for (int i = 0; i < NTHR / 64; i++) t += red[i];
        g.red_out[(int64_t)ty * gridDim.x + tx] = t;
      }
    }
  }
  if constexpr (kCols) {
    if (g.epi == EPI_GELU_GRAD || g.epi == EPI_OUT_GRAD) {
      // the tile's column sums: a lane's rows, the other half's, then the wave rows
      double* col = red + NTHR / 64;  // [wave row][BN]
#pragma unroll
      for (int j = 0; j < BJ; j++) {
        const double t = cs[j] + __shfl_xor(cs[j], 32);
        if (lane < 32) col[wm * BN + wn * 32 * BJ + 32 * j + lane] = t;
      }
      __syncthreads();
      if (tid < BN && n0 + tid < N) {
        double t = 0.0;
        for (int i = 0; i < NTHR / 64 / NWN; i++) t += col[i * BN + tid];
        g.col_part[(int64_t)tx * N + n0 + tid] = t;
      }
    }
  }
}

__global__ void splitk_reduce_kernel(const float* __restrict__ partial, int splits, int64_t M,
                                     int64_t N, float* __restrict__ C, int64_t ldc,
                                     const float* __restrict__ bias) {
  const int64_t total = M * N;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
       i += (int64_t)gridDim.x * blockDim.x) {
    const int64_t m = i / N, n = i - m * N;
    double s = 0.0;  // the partials are as large as the sum: one rounding for all
    int z = 0;
    for (; z + 3 < splits; z += 4) {  // four loads in flight, added in split order
      const float a = partial[(int64_t)z * total + i], b = partial[(int64_t)(z + 1) * total + i];
      const float c = partial[(int64_t)(z + 2) * total + i], d = partial[(int64_t)(z + 3) * total + i];
      s += (double)a;
      s += (double)b;
      s += (double)c;
      s += (double)d;
    }
    for (; z < splits; z++) s += (double)partial[(int64_t)z * total + i];
    C[m * ldc + n] = bias ? (float)s + bias[n] : (float)s;
  }
}

bool aligned(const void* p, size_t a) { return ((uintptr_t)p & (a - 1)) == 0; }

template <typename T, bool AT, bool BT, bool FAR, int CFG>
hipError_t launch(const GemmArgs& g, hipStream_t s) {
  constexpr size_t bytes = lds_bytes_of<T, CFG>();
  const void* fn = (const void*)gemm_kernel<T, AT, BT, FAR, CFG>;
  if constexpr (bytes > 65536) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) return e;
  }
  const dim3 grid((unsigned)((g.M + Tile<CFG>::BM - 1) / Tile<CFG>::BM),
                  (unsigned)((g.N + Tile<CFG>::BN - 1) / Tile<CFG>::BN),
                  (unsigned)(g.splits > 1 ? g.splits : 1));
  gemm_kernel<T, AT, BT, FAR, CFG><<<grid, threads_of<CFG>(), bytes, s>>>(g);
  return hipGetLastError();
}

// The form launched is the form planned: the caller sizes and adds the tiles' sums
// (red_out, col_part) by it.
template <typename T, bool AT, bool BT, bool FAR>
hipError_t launch_form(const GemmArgs& g, hipStream_t s) {
  if (!epi_used<T, AT, BT>(g.epi)) return hipErrorInvalidValue;
  if (g.cfg == 0) return launch<T, AT, BT, FAR, 0>(g, s);
  if (g.cfg == 1) return launch<T, AT, BT, FAR, 1>(g, s);
  if constexpr (!FAR) {
    if (g.cfg == 2) return launch<T, AT, BT, FAR, 2>(g, s);
  }
  return hipErrorInvalidValue;
}

template <typename T, bool FAR>
hipError_t launch_elem(bool a_trans, bool b_trans, const GemmArgs& g, hipStream_t s) {
  if (a_trans) return b_trans ? hipErrorInvalidValue : launch_form<T, true, false, FAR>(g, s);
  return b_trans ? launch_form<T, false, true, FAR>(g, s) : launch_form<T, false, false, FAR>(g, s);
}

template <typename T>
hipError_t launch_type(bool a_trans, bool b_trans, const GemmArgs& g, bool far, hipStream_t s) {
  return far ? launch_elem<T, true>(a_trans, b_trans, g, s) : launch_elem<T, false>(a_trans, b_trans, g, s);
}

// The forms as gemm_plan sees them: `occ` workgroups fit on a CU (by LDS and
// registers), and a full CU then runs at about `rate` (FP32 and BF16 products: 159 and
// 666 TFLOP/s over the chip for form 0, where 10,000 x 240 x 10,000 reaches 143 to 150
// and 520 with its start and end; what the choice depends on is the forms' ratio).
struct CfgCost {
  int BM, BN, bk32, bk16, occ;
  double rate32, rate16;  // FLOP/s of one full CU
};
constexpr CfgCost kCfg[3] = {
    {Tile<0>::BM, Tile<0>::BN, Tile<0>::BK32, Tile<0>::BK16, 2, 0.62e12, 2.6e12},
    {Tile<1>::BM, Tile<1>::BN, Tile<1>::BK32, Tile<1>::BK16, 4, 0.48e12, 1.7e12},
    {Tile<2>::BM, Tile<2>::BN, Tile<2>::BK32, Tile<2>::BK16, 2, 0.37e12, 1.3e12},
};

}  // namespace

// Tile and split-K choice: the estimated time of each is the number of rounds
// of workgroups over the chip's slots times one split's share of the
// contraction -- at the CU's rate shared by the workgroups on it, or at one
// load latency per K-step where that is longer -- plus the time of writing and
// summing the partial products.  A form is not tied to a width: the 128 x 32 one is
// chosen where its tiles fill the CUs better (rows x 512 or x 200 columns at two to
// four thousand rows), and 16 columns may well go to the 64 x 64 one.  kCus is the
// MI355X's CU count, not the device's, so that a product's sums, which the split
// decides, are the same on a partition.
GemmPlan gemm_plan(Elem t, int64_t M, int64_t N, int64_t Kd, int max_splits, bool far) {
  constexpr double kCus = 256.0, kBytesPerSec = 4.0e12;
  constexpr double kStart = 3.0e-6, kStep = 0.6e-6, kReduce = 3.0e-6;
  GemmPlan best{};
  double best_t = 0.0;
  for (int c = 0; c < (far ? 2 : 3); c++) {
    const CfgCost& f = kCfg[c];
    const int bk = t == Elem::F32 ? f.bk32 : f.bk16;
    const double rate = t == Elem::F32 ? f.rate32 : f.rate16;
    const int64_t tiles = ((M + f.BM - 1) / f.BM) * ((N + f.BN - 1) / f.BN);
    for (int s = 1; s <= max_splits; s++) {
      if (s > 1 && Kd / s < 64) break;
      int64_t kps = (Kd + s - 1) / s;
      kps = (kps + 63) / 64 * 64;
      if ((Kd + kps - 1) / kps != s) continue;
      const double wgs = (double)tiles * s;
      // workgroups on a CU; fewer than fit use less of its rate (one of two: 70%)
      const double on_cu = std::min((double)f.occ, std::ceil(wgs / kCus));
      const double share = on_cu * (1.0 + 0.9 * (f.occ - on_cu) / f.occ);
      const double rounds = std::ceil(wgs / (kCus * f.occ));
      const double steps = std::ceil((double)kps / bk);
      const double step = std::max(share * 2.0 * f.BM * f.BN * bk / rate, kStep);
      double e = rounds * (kStart + steps * step);
      if (s > 1) e += kReduce + (2.0 * s + 1.0) * (double)M * (double)N * 4.0 / kBytesPerSec;
      if (best_t == 0.0 || e < best_t * 0.97) {  // a change must pay for itself
        best = GemmPlan{c, s, kps};
        best_t = e;
      }
    }
  }
  return best;
}

int gemm_tile_cols(int cfg) { return kCfg[cfg].BN; }
int gemm_tile_rows(int cfg) { return kCfg[cfg].BM; }

// The residual's partial sums: one per tile of the 128 x 128 form.
int64_t gemm_resid_tiles(int64_t M, int64_t N) {
  return ((M + kCfg[0].BM - 1) / kCfg[0].BM) * ((N + kCfg[0].BN - 1) / kCfg[0].BN);
}

hipError_t splitk_reduce(const float* partial, int splits, int64_t M, int64_t N, float* C,
                         int64_t ldc, const float* bias, hipStream_t s) {
  const int64_t total = M * N;
  int blocks = (int)((total + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  splitk_reduce_kernel<<<blocks, 256, 0, s>>>(partial, splits, M, N, C, ldc, bias);
  return hipGetLastError();
}

// Dword-aligned rows within 32-bit tile offsets are loaded as dwords, others element
// by element.
bool gemm_far(Elem t, const GemmArgs& g) {
  const size_t es = t == Elem::F32 ? 4 : 2;
  return !aligned(g.A, 4) || !aligned(g.B, 4) || (g.lda * es) % 4 || (g.ldb * es) % 4 ||
         g.lda >= (int64_t(1) << 22) || g.ldb >= (int64_t(1) << 22);
}

hipError_t gemm(Elem t, bool a_trans, bool b_trans, const GemmArgs& g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return hipSuccess;
  if (g.epi == EPI_RESID_SQ && g.cfg != 0) return hipErrorInvalidValue;
  const bool far = gemm_far(t, g);
  const hipError_t e = t == Elem::F32 ? launch_type<float>(a_trans, b_trans, g, far, s)
                                      : launch_type<__bf16>(a_trans, b_trans, g, far, s);
  if (e != hipSuccess) return e;
  if (g.splits > 1 && g.epi == EPI_STORE && g.C)  // without C the caller sums the partials
    return splitk_reduce(g.partial, g.splits, g.M, g.N, g.C, g.ldc, g.bias, s);
  return hipSuccess;
}

}  // namespace plnmf
