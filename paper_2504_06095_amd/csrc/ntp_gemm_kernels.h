// Device code of the bf16 MFMA GEMM family (kernels and their helpers); included by
// ntp_gemm.hip, which holds the host-side checks and the launch logic.
#ifndef NTP_GEMM_KERNELS_H_
#define NTP_GEMM_KERNELS_H_

#include <hip/hip_runtime.h>

#include "ntp_internal.h"

namespace ntp_gemm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxRowSegs = 16;

struct GemmArgs {
  const uint16_t* A;
  const uint16_t* B;
  void* C;
  void* C2;
  const uint16_t* AUX;
  int64_t lda, ldb, ldc, ldc2, ldaux;
  int32_t M, N, K;
  int32_t n_store;  // columns stored: N, or N rounded up to 8 with zero fill
  int32_t gelu_mode;
  int32_t tiles_m, tiles_n;
  // fp32 epilogues only: where the output rows go.  n_segs == 0: to C / ldc.  Otherwise every row m
  // is stored to each segment with begin <= m < end, at ptr + (m - begin) * ld.
  int32_t n_segs;
  struct RowSeg {
    int32_t begin, end;
    float* ptr;
    int64_t ld;
  } seg[kMaxRowSegs];
  // every row of [0, M) goes somewhere: the epilogue of a whole tile then issues a known number of instructions (at least)
  int32_t all_rows;
  // split-K launches only: number of K chunks, chunk length (elements, a multiple of 64) and the
  // distance in floats between the partial-sum slices that start at C
  int32_t k_splits, k_chunk;
  int64_t split_stride;
  // ring kernel: bytes of A and of B from their first element to the end of the last chunk the kernel may
  // read (operand_extent_bytes); its DMA loads are range-checked against them
  uint32_t a_extent, b_extent;
  // ring kernel, A K-contiguous and B K-strided: the K tail goes through the ring as one more tile.  A's rows
  // hold zeros from K up to the next multiple of 64 (a_extent reaches that far); the lines of B's tail tile at
  // k >= K lie past b_extent and read as zeros
  int32_t ring_tail;
  // persistent launches: workgroups that are resident at a time (compute units of the device, times two for
  // the 4-wavefront tile)
  int32_t resident;
};

// ---- GeLU and its derivative -------------------------------------------------------------------------
// Bound by vector issue: a 256 x 224 tile's epilogue evaluates 112 of them a lane, and nothing but the SIMD's other wavefront overlaps
// them.  The library's erff and tanhf branch on the argument, element by element, so that a wavefront runs both sides under changing
// execution masks, one element's chain after the other.  Here both sides are computed without a branch and one is selected, and eight elements at a
// time go through the same instructions (gelu_values, gelu_slopes).
//   about zero: 0.5 plus an odd polynomial, so that the only rounding of its size is the last one;
//   elsewhere:  the smaller tail (of the normal distribution, of the logistic function), from one hardware exponential: taken as it is for
//               negative arguments (0.5 (1 + erf) loses it to cancellation there), from one for positive ones.
// The coefficients are least-maximum fits of the two functions (errors 1e-9 and 4.8e-9; logistic 2.4e-9), made for these ranges.  Error
// against 64 bits, rms over N(0, 0.1) to N(0, 5) inputs: values 5.9e-9 to 5.7e-8 (with erff and tanhf 6.6e-9 to 6.4e-8), slopes 2.0e-8 to 2.7e-8 (2.0e-8 to
// 1.1e-7); relative to the tail itself 1.9e-5 from -3 to -6.5 (0.5 (1 + erf) has nothing right there).  MLP shard, forward and backward: 512 x 1024 x 586 15.7 -> 15.2 and 20.9 -> 19.8 us,
// 2048 x 4096 x 2341 98.3 -> 95.7 and 192.6 -> 186.4, 4096 x 6144 x 3511 with the tanh form 293.6 -> 285.8 and 632.6 -> 625.6.  What it costs: pre-activations so narrow that whole
// wavefronts stay below erff's branch at sqrt(2) had the cheaper half of it alone, which launches of a few tiles show (rms 0.4, 143 x 384 x 68 forward 22.4 -> 23.3,
// 2406 x 512 x 2163 34.2 -> 35.0; rms 1.4 and 2.0 26.4 -> 23.7 and 37.6 -> 35.1).
__device__ __forceinline__ float normal_cdf(float x, float u) {  // u: x^2
  float p = -1.0864513569686096e-05f;
  p = fmaf(p, u, 0.00012061750021530315f);
  p = fmaf(p, u, -0.0011920799734070897f);
  p = fmaf(p, u, 0.00997534766793251f);
  p = fmaf(p, u, -0.06649065017700195f);
  p = fmaf(p, u, 0.3989422917366028f);
  const float a = fabsf(x);
  float q = -2.045686642304645e-06f;  // log2 of the tail: falls for every a, so that large arguments end at 0
  q = fmaf(q, a, 6.652198499068618e-05f);
  q = fmaf(q, a, -0.000975924835074693f);
  q = fmaf(q, a, 0.008718324825167656f);
  q = fmaf(q, a, -0.05447777360677719f);
  q = fmaf(q, a, -0.457806259393692f);
  q = fmaf(q, a, -1.1516375541687012f);
  q = fmaf(q, a, -0.9999180436134338f);
  const float e = __builtin_amdgcn_exp2f(q);
  return a < 0.9f ? fmaf(x, p, 0.5f) : x < 0.0f ? e : 1.0f - e;
}

// 1 / (1 + 2^-z), and in *tail the smaller of it and its complement.
__device__ __forceinline__ float logistic2(float z, float* tail) {
  const float v = z * z, a = fabsf(z);
  float p = 5.92694959777873e-07f;
  p = fmaf(p, v, -1.5798006643308327e-05f);
  p = fmaf(p, v, 0.0003329587634652853f);
  p = fmaf(p, v, -0.0069378698244690895f);
  p = fmaf(p, v, 0.1732867807149887f);
  const float t = __builtin_amdgcn_exp2f(-a);
  const float s = t * __builtin_amdgcn_rcpf(1.0f + t);
  const bool centre = a < 1.5f;
  *tail = centre ? fmaf(-a, p, 0.5f) : s;
  return centre ? fmaf(z, p, 0.5f) : z < 0.0f ? s : 1.0f - s;
}

constexpr float kTanhA = 2.302208185195923f, kTanhB = 0.10294324159622192f;  // 2 log2(e) sqrt(2 / pi), and that times 0.044715

__device__ __forceinline__ float gelu_erf(float x) { return x * normal_cdf(x, x * x); }
__device__ __forceinline__ float gelu_tanh(float x) {
  float tail;
  return x * logistic2(x * fmaf(x * x, kTanhB, kTanhA), &tail);
}
__device__ __forceinline__ float gelu_erf_slope(float x) {
  const float u = x * x;
  return fmaf(0.3989422804014327f * x, __builtin_amdgcn_exp2f(-0.7213475204444817f * u), normal_cdf(x, u));
}
__device__ __forceinline__ float gelu_tanh_slope(float x) {
  const float u = fminf(x * x, 1.0e30f);  // (infinite, it would meet a tail of zero below)
  float tail;
  const float t = logistic2(x * fmaf(u, kTanhB, kTanhA), &tail);
  // x times the derivative of the logistic function, T (1 - T), times that of its argument
  return fmaf(x * (tail * (1.0f - tail)), fmaf(0.2140644488370838f, u, 1.5957691216057308f), t);
}

// One branch for all of them (the mode is the same for the whole launch).
template <int N>
__device__ __forceinline__ void gelu_values(float (&y)[N], const float (&x)[N], int mode) {
  if (mode == NTP_GELU_TANH) {
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = gelu_tanh(x[i]);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = gelu_erf(x[i]);
  }
}
template <int N>
__device__ __forceinline__ void gelu_slopes(float (&y)[N], const float (&x)[N], int mode) {
  if (mode == NTP_GELU_TANH) {
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = gelu_tanh_slope(x[i]);
  } else {
#pragma unroll
    for (int i = 0; i < N; ++i) y[i] = gelu_erf_slope(x[i]);
  }
}

__device__ __forceinline__ uint16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(uint16_t, static_cast<__bf16>(f));  // round to nearest even
}
__device__ __forceinline__ float bf16_to_f32(uint16_t h) {
  return __builtin_bit_cast(float, uint32_t(h) << 16);
}

// ------------------------------------------------------------------------------
// Generic kernel: 128 x 128 x 32 tile, 4 wavefronts (2 x 2), each 64 x 64 via
// 2 x 2 MFMA 32x32x16.  Operands go global -> registers -> LDS; LDS always holds
// [row][k] with k contiguous, so K-strided operands are transposed on the LDS write.
constexpr int BM = 128, BN = 128, BK = 32;
constexpr int LDS_LD = BK + 8;  // elements; 80-byte rows keep 16-byte alignment and spread banks

template <bool KC>
struct TileLoader {
  // Two 16-byte chunks per thread per tile.
  u16x8 v[2];

  // rows_lim: extent of the non-K dimension; ld in elements
  __device__ __forceinline__ void load(const uint16_t* __restrict__ base, int64_t ld, int row0, int rows_lim,
                                       int k0, int K, int tid) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = tid + i * 256;
      u16x8 val = {0, 0, 0, 0, 0, 0, 0, 0};
      if constexpr (KC) {
        const int r = c >> 2, kc = (c & 3) * 8;
        const int row = row0 + r, k = k0 + kc;
        if (row < rows_lim && k < K) {
          val = *reinterpret_cast<const u16x8*>(base + int64_t(row) * ld + k);
          if (k + 8 > K) {
#pragma unroll
            for (int j = 0; j < 8; ++j)
              if (k + j >= K) val[j] = 0;
          }
        }
      } else {
        const int kk = c >> 4, rc = (c & 15) * 8;
        const int k = k0 + kk, row = row0 + rc;
        if (k < K && row < rows_lim) {
          // a chunk that straddles rows_lim stays inside the padded leading dimension;
          // its extra lanes feed rows/columns that are never stored
          val = *reinterpret_cast<const u16x8*>(base + int64_t(k) * ld + row);
        }
      }
      v[i] = val;
    }
  }

  __device__ __forceinline__ void store(uint16_t* __restrict__ lds, int tid) const {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int c = tid + i * 256;
      if constexpr (KC) {
        const int r = c >> 2, kc = (c & 3) * 8;
        *reinterpret_cast<u16x8*>(lds + r * LDS_LD + kc) = v[i];
      } else {
        const int kk = c >> 4, rc = (c & 15) * 8;
#pragma unroll
        for (int j = 0; j < 8; ++j) lds[(rc + j) * LDS_LD + kk] = v[i][j];
      }
    }
  }
};

// pre: the pre-activations (EPI_DGELU)
template <int EPI>
__device__ __forceinline__ void store4(const GemmArgs& g, int m, int n0, f32x4 acc, u16x4 pre) {
  if (m >= g.M || n0 >= g.n_store) return;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (n0 + j >= g.N) acc[j] = 0.0f;
  if constexpr (EPI == ntp::EPI_F32 || EPI == ntp::EPI_F32_ACCUM) {
    if (g.n_segs == 0) {
      f32x4* p = reinterpret_cast<f32x4*>(static_cast<float*>(g.C) + int64_t(m) * g.ldc + n0);
      if constexpr (EPI == ntp::EPI_F32) *p = acc;
      else *p = *p + acc;
    } else {
      for (int s = 0; s < g.n_segs; ++s) {
        if (m < g.seg[s].begin || m >= g.seg[s].end) continue;
        f32x4* p = reinterpret_cast<f32x4*>(g.seg[s].ptr + int64_t(m - g.seg[s].begin) * g.seg[s].ld + n0);
        if constexpr (EPI == ntp::EPI_F32) *p = acc;
        else *p = *p + acc;
      }
    }
  } else {
    if constexpr (EPI == ntp::EPI_DGELU) {
      const float x[4] = {bf16_to_f32(pre[0]), bf16_to_f32(pre[1]), bf16_to_f32(pre[2]), bf16_to_f32(pre[3])};
      float d[4];
      gelu_slopes(d, x, g.gelu_mode);
#pragma unroll
      for (int j = 0; j < 4; ++j) acc[j] = (n0 + j < g.N) ? acc[j] * d[j] : 0.0f;
    }
    u16x4 o;
#pragma unroll
    for (int j = 0; j < 4; ++j) o[j] = f32_to_bf16(acc[j]);
    *reinterpret_cast<u16x4*>(static_cast<uint16_t*>(g.C) + int64_t(m) * g.ldc + n0) = o;
    if constexpr (EPI == ntp::EPI_GELU) {
      const float x[4] = {acc[0], acc[1], acc[2], acc[3]};
      float v[4];
      gelu_values(v, x, g.gelu_mode);
      u16x4 y;
#pragma unroll
      for (int j = 0; j < 4; ++j) y[j] = f32_to_bf16(v[j]);
      *reinterpret_cast<u16x4*>(static_cast<uint16_t*>(g.C2) + int64_t(m) * g.ldc2 + n0) = y;
    }
  }
}

template <int EPI>
__device__ __forceinline__ void store4(const GemmArgs& g, int m, int n0, f32x4 acc) {
  u16x4 pre = {};
  if constexpr (EPI == ntp::EPI_DGELU) {
    if (m < g.M && n0 < g.n_store) pre = *reinterpret_cast<const u16x4*>(g.AUX + int64_t(m) * g.ldaux + n0);
  }
  store4<EPI>(g, m, n0, acc, pre);
}

// Accumulating epilogue of a wavefront's MI x NI blocks when the rows have one destination: the old values of a block row are
// asked for before the previous block row is stored.  (Block by block, every load waits for the store before it: the
// memory counter is in order.  dA, dB of 4096 x 3511 x 6144 234 -> 228 us, 148 x 15520 x 11640 403 -> 361 us, 3000 x 1600 x 2776 50.6 -> 48 us.)  m0, n0: this lane's row and first column
// of the first block.
template <int MI, int NI>
__device__ __forceinline__ void accumulate_blocks(const GemmArgs& g, int m0, int n0, const f32x4 (&acc)[MI][NI]) {
  const GemmArgs::RowSeg& sg = g.seg[0];
  f32x4 c[2][NI];
  auto row_ok = [&](int i) { return m0 + i * 16 >= sg.begin && m0 + i * 16 < sg.end; };
  auto at = [&](int i, int j) { return reinterpret_cast<f32x4*>(sg.ptr + int64_t(m0 + i * 16 - sg.begin) * sg.ld + n0 + j * 16); };
  auto load = [&](int i) {
    if (!row_ok(i)) return;
#pragma unroll
    for (int j = 0; j < NI; ++j)
      if (n0 + j * 16 < g.N) c[i & 1][j] = *at(i, j);
  };
  load(0);
#pragma unroll
  for (int i = 0; i < MI; ++i) {
    if (i + 1 < MI) load(i + 1);
    __builtin_amdgcn_sched_barrier(0);
    if (row_ok(i)) {
#pragma unroll
      for (int j = 0; j < NI; ++j)
        if (n0 + j * 16 < g.N) *at(i, j) = c[i & 1][j] + acc[i][j];
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// Pre-activations of a block row (EPI_DGELU): this lane's four values of each of its NI blocks, zeros where nothing is stored.  m: the lane's
// row, n0: its first column of the first block.  They are asked for well before they are used (the pairs' stores would stand between them: the
// memory counter is in order).  Against a block row's loads right before its use, whole backward calls: 64 x 64 tiles 0.976-0.997 of the time (1024 x 768 x 512
// 22.6 -> 22.2 us), ping-pong tiles 0.992-1.003, 128 x 128 and 128 x 256 tiles 0.986-1.012.
template <int NI>
__device__ __forceinline__ void load_aux_row(const GemmArgs& g, int m, int n0, u16x4 (&p)[NI]) {
  const uint16_t* const src = g.AUX + int64_t(m) * g.ldaux + n0;
#pragma unroll
  for (int j = 0; j < NI; ++j) {
    p[j] = u16x4{0, 0, 0, 0};
    if (m < g.M && n0 + j * 16 < g.n_store) p[j] = *reinterpret_cast<const u16x4*>(src + j * 16);
  }
}

// bf16 epilogues of the ring kernel, two adjacent 16 x 16 accumulator blocks at once.  Lane l holds row
// l % 16 and columns 4 (l / 16) + {0..3} of both blocks (a0: columns from nb, a1: from nb + 16), 8 bytes of
// bf16 each.  After the element-wise part, the four 16-lane rows trade halves (v_permlane16_swap: odd rows
// of the first register against even rows of the second), so that a lane ends up with 8 consecutive
// columns, 16 bytes: rows 0 / 2 take columns 0-7 / 8-15 of the first block, rows 1 / 3 those of the second.
// A store instruction then writes 64 contiguous bytes per output row instead of 32, and there are half as many.
template <int EPI>
__device__ __forceinline__ void store8_pair(const GemmArgs& g, int m, int nb, int lh, f32x4 a0, f32x4 a1, u16x4 p0 = {}, u16x4 p1 = {}) {
  const int n0 = nb + lh * 4, n1 = n0 + 16;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (n0 + j >= g.N) a0[j] = 0.0f;
    if (n1 + j >= g.N) a1[j] = 0.0f;
  }
  if constexpr (EPI == ntp::EPI_DGELU) {
    float x[8], d[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = bf16_to_f32(j < 4 ? p0[j & 3] : p1[j & 3]);
    gelu_slopes(d, x, g.gelu_mode);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      a0[j] = (n0 + j < g.N) ? a0[j] * d[j] : 0.0f;
      a1[j] = (n1 + j < g.N) ? a1[j] * d[4 + j] : 0.0f;
    }
  }
  auto pack = [](float lo, float hi) { return uint32_t(f32_to_bf16(lo)) | (uint32_t(f32_to_bf16(hi)) << 16); };
  // the lane's 8 output columns after the trade, and the trade itself
  const int c = nb + (lh & 1) * 16 + (lh >> 1) * 8;
  auto trade_store = [&](void* base, int64_t ld, uint32_t x0, uint32_t x1, uint32_t y0, uint32_t y1) {
    const auto r0 = __builtin_amdgcn_permlane16_swap(x0, y0, false, false);
    const auto r1 = __builtin_amdgcn_permlane16_swap(x1, y1, false, false);
    if (m >= g.M) return;
    uint16_t* dst = static_cast<uint16_t*>(base) + int64_t(m) * ld + c;
    if (c + 8 <= g.n_store) {
      typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
      *reinterpret_cast<u32x4*>(dst) = u32x4{r0[0], r1[0], r0[1], r1[1]};
    } else if (c + 4 <= g.n_store) {
      typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
      *reinterpret_cast<u32x2*>(dst) = u32x2{r0[0], r1[0]};
    }
  };
  trade_store(g.C, g.ldc, pack(a0[0], a0[1]), pack(a0[2], a0[3]), pack(a1[0], a1[1]), pack(a1[2], a1[3]));
  if constexpr (EPI == ntp::EPI_GELU) {
    float x[8], y[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = j < 4 ? a0[j & 3] : a1[j & 3];
    gelu_values(y, x, g.gelu_mode);
    trade_store(g.C2, g.ldc2, pack(y[0], y[1]), pack(y[2], y[3]), pack(y[4], y[5]), pack(y[6], y[7]));
  }
}

template <bool AKC, bool BKC, int EPI>
__global__ __launch_bounds__(256) void gemm_generic_kernel(const GemmArgs g) {
  __shared__ __attribute__((aligned(16))) uint16_t sA[BM * LDS_LD];
  __shared__ __attribute__((aligned(16))) uint16_t sB[BN * LDS_LD];
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63;
  const int wm = wave >> 1, wn = wave & 1;
  // N-major tile order: consecutive workgroups share the A tile rows
  const int tile_m = blockIdx.x / g.tiles_n, tile_n = blockIdx.x - tile_m * g.tiles_n;
  const int row0 = tile_m * BM, col0 = tile_n * BN;

  f32x16 acc[2][2];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.0f;

  TileLoader<AKC> la;
  TileLoader<BKC> lb;
  const int ktiles = (g.K + BK - 1) / BK;
  if (ktiles > 0) {
    la.load(g.A, g.lda, row0, g.M, 0, g.K, tid);
    lb.load(g.B, g.ldb, col0, g.N, 0, g.K, tid);
  }
  for (int kt = 0; kt < ktiles; ++kt) {
    la.store(sA, tid);
    lb.store(sB, tid);
    __syncthreads();
    if (kt + 1 < ktiles) {
      la.load(g.A, g.lda, row0, g.M, (kt + 1) * BK, g.K, tid);
      lb.load(g.B, g.ldb, col0, g.N, (kt + 1) * BK, g.K, tid);
    }
#pragma unroll
    for (int ks = 0; ks < BK / 16; ++ks) {
      bf16x8 fa[2], fb[2];
      const int koff = ks * 16 + (lane >> 5) * 8;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        fa[i] = *reinterpret_cast<const bf16x8*>(sA + (wm * 64 + i * 32 + (lane & 31)) * LDS_LD + koff);
#pragma unroll
      for (int j = 0; j < 2; ++j)
        fb[j] = *reinterpret_cast<const bf16x8*>(sB + (wn * 64 + j * 32 + (lane & 31)) * LDS_LD + koff);
      // operands swapped: the product comes out transposed, so that each lane holds
      // 4 consecutive columns of one row (vector stores along N)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fb[j], fa[i], acc[i][j], 0, 0, 0);
    }
    __syncthreads();
  }

  // lane (l) of a 32x32 block holds row l % 32 and columns 8 q + 4 (l / 32) + {0..3}, q = 0..3
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int m = row0 + wm * 64 + i * 32 + (lane & 31);
        const int n0 = col0 + wn * 64 + j * 32 + q * 8 + (lane >> 5) * 4;
        f32x4 v = {acc[i][j][q * 4 + 0], acc[i][j][q * 4 + 1], acc[i][j][q * 4 + 2], acc[i][j][q * 4 + 3]};
        store4<EPI>(g, m, n0, v);
      }
}

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

}  // namespace ntp_gemm

#endif  // NTP_GEMM_KERNELS_H_
