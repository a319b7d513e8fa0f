// Kernels for RAW-layout factor pairs (row-major as a checkpoint has them; any size, any leading
// dimension, element alignment), fp32, bf16 or fp16 storage with fp32 arithmetic:
//   C[M x N] = A[M x K] . B[K x N]            (one stage of y = (x U) V, Sec. 4.1)
// and, for the GLU sub-layer, C = silu(A1 . B1) * (A2 . B2) in one pass.
#pragma once
#include "common.h"

namespace deinfer {

// How the product is laid on the matrix cores: 16x16x4 fp32 products (256 flops per clock and compute unit,
// twice the vector rate; every operand is converted to fp32 exactly, so nothing is rounded before the sum).
// A wavefront owns (16 MB) rows x (16 NV) columns and reads both operands from memory straight into the
// registers the product wants, no LDS and no barrier in the loop:
//   * a step is 16 k: lane l works for the k-group g = l / 16 on k = 4 g .. 4 g + 3 of A row l % 16.  Loaded that way, 16
//     neighbouring lanes touch 16 rows and the address unit, which the wavefronts share, takes four times as long as for
//     whole pieces: four neighbouring lanes load the 16 k of one row instead, and a lane permutation (ds_bpermute)
//     brings each value to its lane, one step ahead of the products;
//   * B rows are read NV elements per lane: lane l holds columns NV (l % 16) .. + NV - 1 of row 4 g + e, and
//     product j takes element j, i.e. column block j is the columns NV c + j.  A load instruction covers
//     16 NV consecutive columns of four rows, and a lane ends up with NV consecutive output columns.
// The wavefronts of a workgroup share one tile and split its k range; their sums meet in LDS, in wavefront
// order (deterministic).  A 64 x 64 tile reads 16 bytes per clock and compute unit at the full matrix rate,
// half of what a compute unit takes in from L2.  What bounds it: the fp32 matrix rate (157 TFLOP/s) for
// many rows, the stream of B and the latency of the first loads for few.
// Measured (first stage alone / both, us): 201 x 4096 x 1638 in fp32 53.4 -> 49.3 / 84.9 -> 81.1 with the permutation,
// 47.5 / 79.2 with runs of tiles per XCD (below); 100 x 4096 x 2000 37.7 -> 34.3 -> 29.8; 64 x 4096 x 1638 33.3 -> 33.2 ->
// 26.1; 2048 x 512 x 200 14.5 -> 13.1.  Eight wavefronts on a tile (61.3) and 32 k per step, so that A's lines are
// loaded whole (54.0), were no faster than 53.4.
template <typename T> struct RawStore { typedef uint16_t type; };
template <> struct RawStore<float> { typedef float type; };
// (loads of several elements need no more than element alignment)
template <typename T, int N> struct RawVec {
  typedef typename RawStore<T>::type type __attribute__((ext_vector_type(N), aligned(sizeof(T))));
};
template <typename T> __device__ __forceinline__ float raw_cvt(typename RawStore<T>::type v) {
  if constexpr (sizeof(T) == 4) return v;
  else return cvt_in<DtOf<T>::value>(v);
}

template <typename TA, typename TB> struct RawOperands {
  const TA *A;
  int64_t lda;
  const TB *B;
  int64_t ldb;
  int K;
};

// Register buffers of k-steps: one is multiplied while the next D - 1 are on their way.  A step of a 64 x 64 tile is 8 KiB
// per wavefront in fp32 and 2000 matrix cycles, so its loads are requested 4000 cycles ahead; smaller steps, more of them.
// One buffer more (4, 5, 7) is 1 to 5 % slower, by tile, on average over 3000 random products, the most where the k range is
// a few steps, and no faster on long ones (first stages in fp32, us: 201 x 4096 x 1638 47.6, 47.5; 16 x 700 x 300
// 6.26, 6.57; 201 x 1638 x 4096 35.5, 35.2).
constexpr int raw_depth(int mb, int nv) { return mb * nv >= 16 ? 3 : mb * nv >= 8 ? 4 : 6; }

// acc[i][j] += A[m0 + 16 i .., :] . B[:, column block j of n0 ..], this wavefront's part of the k range.
// EDGE: the tile reaches beyond column N - 1 (columns clamped; what they give is not stored).
template <typename TA, typename TB, int MB, int NV, int NW, bool EDGE>
__device__ __forceinline__ void raw_product(const RawOperands<TA, TB> &P, int M, int N, int64_t m0, int64_t n0, f32x4_t (&acc)[MB][NV]) {
#if defined(__HIP_DEVICE_COMPILE__)
  typedef typename RawVec<TA, 4>::type AV;
  typedef typename RawVec<TB, NV>::type BV;
  typedef typename RawStore<TB>::type BS;
  typedef typename RawStore<TA>::type AS;
  constexpr int D = raw_depth(MB, NV);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const int c = lane & 15, g = lane >> 4;
  const int steps = (P.K + 15) / 16, full = P.K / 16;
  const int s_begin = (int)((int64_t)steps * wave / NW), s_end = (int)((int64_t)steps * (wave + 1) / NW);
  // A is loaded with four neighbouring lanes on 4 x 4 consecutive k of one row, and crosses to the lanes that multiply
  // it (row l % 16, k-group l / 16) by a lane permutation
  const int ak = 4 * (lane & 3);
  const int from = (4 * c + g) * 4;
  const AS *a[MB];
#pragma unroll
  for (int i = 0; i < MB; ++i) {
    int64_t row = m0 + 16 * i + (lane >> 2);
    row = row < M ? row : M - 1;                       // (rows beyond M - 1 are not stored)
    a[i] = reinterpret_cast<const AS *>(P.A) + row * P.lda + ak;
  }
  int64_t col[EDGE ? NV : 1];
#pragma unroll
  for (int j = 0; j < (EDGE ? NV : 1); ++j) {
    col[j] = n0 + NV * c + j;
    if (EDGE && col[j] >= N) col[j] = N - 1;
  }
  const BS *b = reinterpret_cast<const BS *>(P.B) + (int64_t)(4 * g) * P.ldb;
  struct Step { AV a[MB]; BV b[4]; } buf[D];
  // part e of a step's loads: B rows 4 g + e and the A rows of every fourth row block
  auto load = [&](Step &t, int s, int e) {
    const BS *p = b + ((int64_t)16 * s + e) * P.ldb;
    if constexpr (EDGE) {
#pragma unroll
      for (int j = 0; j < NV; ++j) t.b[e][j] = p[col[j]];
    } else {
      t.b[e] = *reinterpret_cast<const BV *>(p + col[0]);
    }
    if (e < MB) t.a[e] = *reinterpret_cast<const AV *>(a[e] + (int64_t)16 * s);
  };
  struct Rows { AV a[MB]; };
  auto cross = [&](const AV &v) -> AV {
    constexpr int W = (int)sizeof(AV) / 4;
    typedef int words __attribute__((ext_vector_type(W)));
    words w = __builtin_bit_cast(words, v);
#pragma unroll
    for (int q = 0; q < W; ++q) w[q] = __builtin_amdgcn_ds_bpermute(from, w[q]);
    return __builtin_bit_cast(AV, w);
  };
  auto multiply = [&](const Rows &r, const Step &t, int e) {
#pragma unroll
    for (int j = 0; j < NV; ++j)
#pragma unroll
      for (int i = 0; i < MB; ++i)
        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(raw_cvt<TA>(r.a[i][e]), raw_cvt<TB>(t.b[e][j]), acc[i][j], 0, 0, 0);
  };
  const bool tail = s_end == steps && full < steps;
  const int s_stop = s_end < full ? s_end : full;
  const int last = s_stop - 1;                         // (requests past the end repeat the last step)
  // the last K % 16 of the k range: zeros beyond K - 1 (what is read there is row K - 1 and is replaced)
  Step rest;
  if (tail) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      int k = 16 * full + 4 * g + e, ka = 16 * full + ak + e;
      k = k < P.K ? k : P.K - 1;
      ka = ka < P.K ? ka : P.K - 1;
#pragma unroll
      for (int i = 0; i < MB; ++i) rest.a[i][e] = a[i][ka - ak];
#pragma unroll
      for (int j = 0; j < NV; ++j) rest.b[e][j] = b[(int64_t)(k - 4 * g) * P.ldb + (EDGE ? col[EDGE ? j : 0] : col[0] + j)];
    }
  }
  if (s_begin < s_stop) {
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        load(buf[d], s_begin + d < last ? s_begin + d : last, e);
        __builtin_amdgcn_sched_barrier(0);             // (in this order: the waits of the loop count on it)
      }
  }
  if (tail) {
    Rows r;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) rest.a[i][e] = 16 * full + ak + e < P.K ? rest.a[i][e] : AS{};
      r.a[i] = cross(rest.a[i]);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const bool in = 16 * full + 4 * g + e < P.K;
#pragma unroll
      for (int j = 0; j < NV; ++j) rest.b[e][j] = in ? rest.b[e][j] : BS{};
      multiply(r, rest, e);
    }
  }
  if (s_begin < s_stop) {
    int s = s_begin;
    // Step s is multiplied while step s + D - 1 is requested and the rows of step s + 1 cross, a quarter behind each
    // quarter of the products.
    // (No exit inside a round of D steps: with one, the compiler waits for every outstanding load at the top.)
    Rows r;
#pragma unroll
    for (int i = 0; i < MB; ++i) r.a[i] = cross(buf[0].a[i]);
    for (; s + D <= s_stop; s += D) {
#pragma unroll
      for (int d = 0; d < D; ++d) {
        Rows next;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          multiply(r, buf[d], e);
          __builtin_amdgcn_sched_barrier(0);
          load(buf[(d + D - 1) % D], s + d + D - 1 < last ? s + d + D - 1 : last, e);
          if (e < MB) next.a[e] = cross(buf[(d + 1) % D].a[e]);
          __builtin_amdgcn_sched_barrier(0);
        }
        r = next;
      }
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d)
      if (s + d < s_stop) {
#pragma unroll
        for (int i = 0; i < MB; ++i) r.a[i] = cross(buf[d].a[i]);
#pragma unroll
        for (int e = 0; e < 4; ++e) multiply(r, buf[d], e);
      }
  }
#else
  (void)P; (void)M; (void)N; (void)m0; (void)n0; (void)acc;
#endif
}

// Runs of tiles per XCD: up to 8 row tiles, and for 16 x 16 tiles from 1600 k or one round of workgroups on.  4500 random
// products with runs and without (the tile that is taken): 16 x 16 within a round 4 to 6 % slower below 800 k (0.2 us of 3.5
// to 7), 2 % to 1600, 1 % faster from there on; 16 x 16 in more rounds 1 to 8 % faster; larger tiles within a round 1 % slower
// to 5 % faster, the more the longer k, in more rounds 3 to 19 % faster.
constexpr unsigned RAW_RUN_ROWS = 8;
constexpr int RAW_RUN_K = 1600;
// C = act(A.B + bias), or (DUAL) C = silu(A.B) * (A2.B2).  One workgroup of NW wavefronts = one tile of
// 16 MB rows x 16 NV columns; the tiles of a column block are consecutive workgroups (they share B's columns).
// bias: one value per column of C (may be null), act: see act_f32.
template <typename TA, typename TB, typename TC, bool DUAL, int MB, int NV, int NW>
__global__ __launch_bounds__(64 * NW) void raw_gemm_kernel(
    const RawOperands<TA, TB> P, const RawOperands<TA, TB> P2, TC *__restrict__ C, int64_t ldc, int M, int N,
    const TC *__restrict__ bias, int act) {
  constexpr int UNITS = 4 * MB;                        // accumulator element e of row block i: unit 4 i + e
  constexpr int UPW = (UNITS + NW - 1) / NW;           // units that a wavefront sums and stores
  typedef float sum_t __attribute__((ext_vector_type(NV)));
  __shared__ sum_t part[NW][UNITS][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  // Few row tiles: an XCD takes a run of tiles, so that the row tiles of a column block share one L2, which fetches B's
  // columns once
  int mt = blockIdx.x;
  int64_t nt = (int64_t)blockIdx.z * gridDim.y + blockIdx.y;
  // (16 x 16 tiles in one round with a short k are done before that counts, and the mapping costs them 0.2 us)
  if (gridDim.x > 1 && gridDim.x <= RAW_RUN_ROWS && gridDim.z == 1 && (MB * NV > 1 || P.K >= RAW_RUN_K || gridDim.x * gridDim.y > 256)) {
    const int tile = run_tile_of((int)(blockIdx.y * gridDim.x + blockIdx.x), (int)(gridDim.y * gridDim.x));
    nt = tile / (int)gridDim.x;
    mt = tile - (int)nt * (int)gridDim.x;
  }
  const int64_t m0 = (int64_t)mt * (16 * MB), n0 = nt * (16 * NV);
  if (n0 >= N) return;                                 // (the last slice of the column blocks)
  const bool edge = n0 + 16 * NV > N;
  float sum[DUAL ? 2 : 1][UPW][NV];
#pragma unroll
  for (int q = 0; q < (DUAL ? 2 : 1); ++q) {
    f32x4_t acc[MB][NV];
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int j = 0; j < NV; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
    if (edge) raw_product<TA, TB, MB, NV, NW, true>(q ? P2 : P, M, N, m0, n0, acc);
    else raw_product<TA, TB, MB, NV, NW, false>(q ? P2 : P, M, N, m0, n0, acc);
    if (q) __syncthreads();                            // the first product's sums have been read
#pragma unroll
    for (int i = 0; i < MB; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sum_t v;
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] = acc[i][j][e];
        part[wave][4 * i + e][lane] = v;
      }
    __syncthreads();
#pragma unroll
    for (int t = 0; t < UPW; ++t) {
      const int u = wave + t * NW;
#pragma unroll
      for (int j = 0; j < NV; ++j) sum[q][t][j] = 0.f;
      if (u < UNITS) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
          const sum_t v = part[w][u][lane];
#pragma unroll
          for (int j = 0; j < NV; ++j) sum[q][t][j] += v[j];
        }
      }
    }
  }
  const int64_t col0 = n0 + NV * (lane & 15);
#pragma unroll
  for (int t = 0; t < UPW; ++t) {
    const int u = wave + t * NW;
    const int64_t row = m0 + 16 * (u >> 2) + 4 * (lane >> 4) + (u & 3);
    if (u >= UNITS || row >= M) continue;
    float v[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
      const float z = sum[0][t][j];
      if constexpr (DUAL) v[j] = (z / (1.0f + expf(-z))) * sum[DUAL ? 1 : 0][t][j];
      else v[j] = act_f32(z + ((bias && col0 + j < N) ? Elem<TC>::load(bias + col0 + j) : 0.0f), act);
    }
    TC *dst = C + row * ldc + col0;
    if (col0 + NV <= N) {
      typedef typename RawVec<TC, NV>::type CV;
      CV o;
#pragma unroll
      for (int j = 0; j < NV; ++j) {
        if constexpr (sizeof(TC) == 4) o[j] = v[j];
        else o[j] = cvt_out<DtOf<TC>::value>(v[j]);
      }
      *reinterpret_cast<CV *>(dst) = o;
    } else {
#pragma unroll
      for (int j = 0; j < NV; ++j)
        if (col0 + j < N) Elem<TC>::store(dst + j, v[j]);
    }
  }
}

// C[r][c] = act(bias[c]): the non-GLU sub-layer of a pair of rank 0 (empty product).
template <typename TC>
__global__ void bias_act_fill_kernel(TC *C, int64_t ldc, int M, int N, const TC *bias, int act) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)M * N) {
    const int64_t r = i / N, c = i % N;
    Elem<TC>::store(C + r * ldc + c, act_f32(bias ? Elem<TC>::load(bias + c) : 0.0f, act));
  }
}

// Zero-fill of a strided 2-D region (r == 0 outputs) and of raw words (workspace init).
template <typename TC>
__global__ void zero2d_kernel(TC *C, int64_t ldc, int M, int N) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)M * N) C[(i / N) * ldc + (i % N)] = TC{};
}
__global__ void fill_words_kernel(uint32_t *p, size_t n, uint32_t v) {
  size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Copy a column block of a row-major matrix (used to hand out the rank-space
// intermediates of k and v, the low-rank KV cache of Sec. 2.1).
template <typename TS, typename TD>
__global__ void copy2d_kernel(const TS *S, int64_t lds, TD *D, int64_t ldd, int M, int N) {
  int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < (int64_t)M * N) {
    int64_t r = i / N, c = i % N;
    Elem<TD>::store(D + r * ldd + c, Elem<TS>::load(S + r * lds + c));
  }
}

// Rows of 16-bit elements copied with zero padding: D[row][c] = c < n_valid ? S[row][c] : 0 for
// c < N (the caller's rank-space rows brought to the 16-byte row layout the packed kernels read,
// with exact zeros where the zero-padded weights are met).  One thread = one 16-byte chunk of 8
// columns of D (D 16-byte aligned, ldd % 8 == 0, N % 8 == 0); a chunk that lies wholly inside the
// valid columns of a 16-byte aligned source row is one 16-byte load, any other chunk is read
// element by element, and never beyond column n_valid - 1.
__global__ void pad_rows16_kernel(const uint16_t *S, int64_t lds, uint16_t *D, int64_t ldd, int M, int n_valid, int N, int vec) {
  const int c8 = N / 8;
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= (int64_t)M * c8) return;
  const int64_t r = i / c8;
  const int c = (int)(i % c8) * 8;
  uint4 v = make_uint4(0u, 0u, 0u, 0u);
  const uint16_t *src = S + r * lds + c;
  if (vec && c + 8 <= n_valid) {
    v = *reinterpret_cast<const uint4 *>(src);
  } else if (c < n_valid) {
    uint16_t e[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) e[k] = c + k < n_valid ? src[k] : (uint16_t)0;
    v = make_uint4((unsigned)e[0] | ((unsigned)e[1] << 16), (unsigned)e[2] | ((unsigned)e[3] << 16),
                   (unsigned)e[4] | ((unsigned)e[5] << 16), (unsigned)e[6] | ((unsigned)e[7] << 16));
  }
  *reinterpret_cast<uint4 *>(D + r * ldd + c) = v;
}

}  // namespace deinfer
