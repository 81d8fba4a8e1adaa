// Offline calibration (Section 5.1 "Quantization setup"; Section 4.2): an fp32 forward of the
// unquantized mixer over the calibration batch with absmax observers, the percentile maximum
// for the scan input x, the Hadamard-space scale of the scan output and the folding of H_n
// into W_out, followed by the per-tensor symmetric quantization of every weight (Eq. 2).
// This runs once per layer.  4 x 256 tokens of the 2.8B layer: 54 GFLOP of fp32 input projection are the floor.
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <vector>

#include "common.h"

namespace quamba {

// defined in hadamard.hip: fp32 rows in, fp32 rows out (no quantization)
int launch_hadamard_f32(const float *x, int M, int n, float *y, hipStream_t st);

namespace {

constexpr float LOG2E = 1.44269504088896340736f;

// Pieces of four values of master weights and outputs, which promise no more than their own alignment.
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4u __attribute__((ext_vector_type(4), aligned(4)));
typedef float f2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// ---------------------------------------------------------------- fp32 GEMM, C = A W^T
// fp32 matrix units (fp32 operands, fp32 sums, 256 flop per clock and CU).  Every scale of the layer hangs on these sums, and a
// scale that moves in its last bit moves int8 codes, so their order is fixed: an output is one chain of fused
// multiply-adds over k = 0, 1, 2, ..., whatever the tile (the matrix instructions add their two or four products in the order
// of k, each with one rounding: compared with v_fma_f32 bit for bit), and K is never split.
//
// Large outputs (v_mfma_f32_32x32x2_f32): a wave owns 32 rows x 64 columns; the weight rows are the MFMA A operand, so a
// lane ends with four consecutive columns of one row.  A slice is 32 of K, register-prefetched into one padded LDS
// buffer; a lane reads four consecutive k of every eight as 16 bytes, and two swaps between the halves of the wave make of
// the four registers the operands of four products in the order of k (stored in that order instead, as pairs, the
// products took 600 us at the size below), so a wave reads 16 bytes per lane three times for eight products.
// Small tiles, so that several workgroups cover each other's barriers: 74 vector and 32 accumulation registers leave room for
// four on a CU.  Where the last round of them is nearly empty (the 1280 of 1024 x 10240 are a full round and a quarter of one: 479 us, 112
// TFLOP/s of the 157 that fp32 matrix products reach at most) the wide tiles below take over (a 64 x 64 tile on the vector units: 935 us).
// WM x WN waves: 128 x 64, 64 x 128, 32 x 256 outputs per workgroup.
constexpr int GK = 32, GLD = GK + 4;

template <int WM, int WN>
__global__ __launch_bounds__(256) void sgemm_tn_kernel(const float *__restrict__ A, int lda, const float *__restrict__ W,
                                                       int ldw, float *__restrict__ C, int ldc, int M, int N, int K) {
  constexpr int BM = 32 * WM, BN = 64 * WN;
  __shared__ __attribute__((aligned(16))) float sa[BM * GLD], sw[BN * GLD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave % WM, wn = wave / WM, l31 = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;

  f4 ra[WM], rw[2 * WN];
  const int prow = tid >> 3, pk = (tid & 7) * 4;  // eight 16-byte pieces per row and slice
  auto fetch = [&](int k) {                        // K is a multiple of 16: a piece is in range or out of it
#pragma unroll
    for (int i = 0; i < WM; ++i) {
      const int r = m0 + prow + 32 * i;
      ra[i] = f4{0.f, 0.f, 0.f, 0.f};
      if (r < M && k + pk < K) ra[i] = *reinterpret_cast<const f4u *>(A + (size_t)r * lda + k + pk);
    }
#pragma unroll
    for (int i = 0; i < 2 * WN; ++i) {
      const int r = n0 + prow + 32 * i;
      rw[i] = f4{0.f, 0.f, 0.f, 0.f};
      if (r < N && k + pk < K) rw[i] = *reinterpret_cast<const f4u *>(W + (size_t)r * ldw + k + pk);
    }
  };
  // k = 4 h .. 4 h + 3 of eight -> k = h, 2 + h, 4 + h, 6 + h
  auto in_order = [](const f4 &v) {
    const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[0]), __float_as_uint(v[1]), false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[2]), __float_as_uint(v[3]), false, false);
    return f4{__uint_as_float(a[0]), __uint_as_float(b[0]), __uint_as_float(a[1]), __uint_as_float(b[1])};
  };

  f32x16 acc[2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  fetch(0);
  for (int k = 0; k < K; k += GK) {
    __syncthreads();  // the previous slice has been read
#pragma unroll
    for (int i = 0; i < WM; ++i) *reinterpret_cast<f4 *>(&sa[(prow + 32 * i) * GLD + pk]) = ra[i];
#pragma unroll
    for (int i = 0; i < 2 * WN; ++i) *reinterpret_cast<f4 *>(&sw[(prow + 32 * i) * GLD + pk]) = rw[i];
    __syncthreads();
    if (k + GK < K) fetch(k + GK);
#pragma unroll
    for (int kk = 0; kk < GK / 8; ++kk) {
      const f4 fa = in_order(*reinterpret_cast<const f4 *>(&sa[(wm * 32 + l31) * GLD + kk * 8 + 4 * h]));
      const f4 f0 = in_order(*reinterpret_cast<const f4 *>(&sw[(wn * 64 + l31) * GLD + kk * 8 + 4 * h]));
      const f4 f1 = in_order(*reinterpret_cast<const f4 *>(&sw[(wn * 64 + 32 + l31) * GLD + kk * 8 + 4 * h]));
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        acc[0] = __builtin_amdgcn_mfma_f32_32x32x2f32(f0[e], fa[e], acc[0], 0, 0, 0);
        acc[1] = __builtin_amdgcn_mfma_f32_32x32x2f32(f1[e], fa[e], acc[1], 0, 0, 0);
      }
    }
  }
  const int m = m0 + wm * 32 + l31;
  if (m >= M) return;
  float *row = C + (size_t)m * ldc;
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = n0 + wn * 64 + j * 32 + 8 * q + 4 * h;  // N is a multiple of 16
      if (n < N) *reinterpret_cast<f4u *>(row + n) = f4u{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
    }
}

// Large outputs whose tiles come out even over the CUs: 128 x 32 TN outputs per workgroup, a wave 32 rows x 32 TN columns (TN = 3 to 5; 80
// accumulators at 5), at most two workgroups per CU.  A wave reads TN + 1 operand pieces for 4 TN products; slices of 32 in two unpadded LDS
// buffers (the pieces of a row exchanged by the row's low bits), so one barrier per slice, and the slice after next is on its way meanwhile.
// Bound by the matrix unit: 1024 x 10240 x 2560 431 us = 125 TFLOP/s, 479 in tiles of 128 x 64 (467 with these tiles and the swaps above:
// here the even k of every eight are stored in one piece and the odd ones in the next, which costs a second store per piece).
template <int TN>
__global__ __launch_bounds__(256, 2) void sgemm_wide_kernel(const float *__restrict__ A, int lda, const float *__restrict__ W,
                                                            int ldw, float *__restrict__ C, int ldc, int M, int N, int K) {
  constexpr int BM = 128, BN = 32 * TN, ROWS = BM + BN, PIECES = ROWS / 32;
  extern __shared__ __attribute__((aligned(16))) float tile[];  // [2][ROWS][GK]
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, l31 = lane & 31, h = lane >> 5;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int prow = tid >> 3, piece = tid & 7;
  // row r of the tile: rows of A, then rows of W; past the end: read again, never stored
  const float *src[PIECES];
#pragma unroll
  for (int i = 0; i < PIECES; ++i) {
    const int r = prow + 32 * i;
    src[i] = (r < BM ? A + (size_t)min(m0 + r, M - 1) * lda : W + (size_t)min(n0 + r - BM, N - 1) * ldw) + piece * 4;
  }
  f4 reg[PIECES];
  auto fetch = [&](int k) {  // K is a multiple of 16: a piece is in range or out of it
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      reg[i] = f4{0.f, 0.f, 0.f, 0.f};
      if (k + piece * 4 < K) reg[i] = *reinterpret_cast<const f4u *>(src[i] + k);
    }
  };
  // of every eight k, the even ones go to one 16-byte piece and the odd ones to the next (rows 32 apart share their low bits)
  const int to0 = prow * GK + ((((piece & ~1) + 0) ^ (prow & 7)) * 4) + 2 * (piece & 1);
  const int to1 = prow * GK + ((((piece & ~1) + 1) ^ (prow & 7)) * 4) + 2 * (piece & 1);
  auto park = [&](int buf) {
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
      float *row = tile + buf * (ROWS * GK) + 32 * i * GK;
      *reinterpret_cast<f2 *>(row + to0) = f2{reg[i][0], reg[i][2]};
      *reinterpret_cast<f2 *>(row + to1) = f2{reg[i][1], reg[i][3]};
    }
  };
  f32x16 acc[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[j][r] = 0.f;
  fetch(0);
  park(0);
  if (GK < K) fetch(GK);
  __syncthreads();
  for (int k = 0, buf = 0; k < K; k += GK, buf ^= 1) {
    if (k + GK < K) park(buf ^ 1);  // read last before the barrier at the end of the previous slice
    if (k + 2 * GK < K) fetch(k + 2 * GK);
    const float *a = tile + buf * (ROWS * GK) + (wave * 32 + l31) * GK, *w = tile + buf * (ROWS * GK) + (BM + l31) * GK;
#pragma unroll
    for (int kk = 0; kk < GK / 8; ++kk) {
      const int at = ((2 * kk + h) ^ (l31 & 7)) * 4;
      const f4 fa = *reinterpret_cast<const f4 *>(a + at);
      f4 fw[TN];
#pragma unroll
      for (int j = 0; j < TN; ++j) fw[j] = *reinterpret_cast<const f4 *>(w + j * 32 * GK + at);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(fw[j][e], fa[e], acc[j], 0, 0, 0);
    }
    __syncthreads();
  }
  const int m = m0 + wave * 32 + l31;
  if (m >= M) return;
  float *row = C + (size_t)m * ldc;
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int n = n0 + j * 32 + 8 * q + 4 * h;  // N is a multiple of 16
      if (n < N) *reinterpret_cast<f4u *>(row + n) = f4u{acc[j][4 * q], acc[j][4 * q + 1], acc[j][4 * q + 2], acc[j][4 * q + 3]};
    }
}

// Skinny outputs (x_proj: 1024 x 192 x 5120, 24 tiles of the form above): the chain over K is what takes the time, so the
// output is cut as small as the matrix unit allows, one 16 x 16 block (v_mfma_f32_16x16x4_f32, 32 clocks per four of K)
// for each of the four waves of a 32 x 32 tile; slices of 64 in two buffers, the one after
// them in registers (two in registers measure the same).  Groups of 16 k are stored by
// k mod 4, so that the quarter-wave g reads k = g, 4 + g, 8 + g, 12 + g as 16 bytes.  1024 x 192 x 5120: 51 us (one chain per
// thread on the vector units: 728).
constexpr int NK = 64, NLD = NK + 4;

__global__ __launch_bounds__(256) void sgemm_skinny_kernel(const float *__restrict__ A, int lda, const float *__restrict__ W,
                                                           int ldw, float *__restrict__ C, int ldc, int M, int N, int K) {
  __shared__ __attribute__((aligned(16))) float sa[2][32 * NLD], sw[2][32 * NLD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = (wave & 1) * 16, wn = (wave >> 1) * 16, l15 = lane & 15, g = lane >> 4;
  const int m0 = blockIdx.y * 32, n0 = blockIdx.x * 32;
  f4 ra[2], rw[2];
  const int prow = tid >> 4, pk = (tid & 15) * 4;  // 16 pieces per row and slice, rows prow and prow + 16
  auto fetch = [&](int k) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int r = prow + 16 * i;
      ra[i] = rw[i] = f4{0.f, 0.f, 0.f, 0.f};
      if (m0 + r < M && k + pk < K) ra[i] = *reinterpret_cast<const f4u *>(A + (size_t)(m0 + r) * lda + k + pk);
      if (n0 + r < N && k + pk < K) rw[i] = *reinterpret_cast<const f4u *>(W + (size_t)(n0 + r) * ldw + k + pk);
    }
  };
  const int at = (pk & ~15) + ((pk >> 2) & 3);
  auto park = [&](int buf) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        sa[buf][(prow + 16 * i) * NLD + at + 4 * e] = ra[i][e];
        sw[buf][(prow + 16 * i) * NLD + at + 4 * e] = rw[i][e];
      }
  };
  f4 acc = {0.f, 0.f, 0.f, 0.f};
  fetch(0);
  park(0);
  if (NK < K) fetch(NK);
  __syncthreads();
  for (int k = 0, buf = 0; k < K; k += NK, buf ^= 1) {
    if (k + NK < K) park(buf ^ 1);  // read last before the barrier at the end of the previous slice
    if (k + 2 * NK < K) fetch(k + 2 * NK);
    f4 fa[NK / 16], fw[NK / 16];
#pragma unroll
    for (int q = 0; q < NK / 16; ++q) {
      fa[q] = *reinterpret_cast<const f4 *>(&sa[buf][(wm + l15) * NLD + 16 * q + 4 * g]);
      fw[q] = *reinterpret_cast<const f4 *>(&sw[buf][(wn + l15) * NLD + 16 * q + 4 * g]);
    }
#pragma unroll
    for (int q = 0; q < NK / 16; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(fw[q][e], fa[q][e], acc, 0, 0, 0);
    __syncthreads();
  }
  const int m = m0 + wm + l15, n = n0 + wn + 4 * g;
  if (m < M && n < N) *reinterpret_cast<f4u *>(C + (size_t)m * ldc + n) = f4u{acc[0], acc[1], acc[2], acc[3]};
}

template <int TN>
int run_wide(const float *A, int lda, const float *W, int ldw, float *C, int M, int N, int K, hipStream_t st) {
  constexpr size_t lds = 2 * (128 + 32 * TN) * GK * sizeof(float);
  if (lds > 64 * 1024) {  // the attribute is per device: one bit per device index
    static std::atomic<unsigned long long> attr_set{0};
    int dev = 0;
    QUAMBA_HIP(hipGetDevice(&dev));
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
      QUAMBA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&sgemm_wide_kernel<TN>), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      attr_set.fetch_or(bit, std::memory_order_release);
    }
  }
  hipLaunchKernelGGL(sgemm_wide_kernel<TN>, dim3((N + 32 * TN - 1) / (32 * TN), (M + 127) / 128), dim3(256), lds, st, A, lda, W, ldw, C, N,
                     M, N, K);
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}

// Width of the wide tiles in blocks of 32 columns, 0: the 128 x 64 tiles.  Prices are us at K = 2560 (1024, 768, 512, 256 rows x 10240
// columns, and 3072, 8192 and 16384 columns at other K in proportion): 50 and 85 for every 256 of the 128 x 64 tiles begun; the wide ones
// up to one and up to two per CU.  Beyond two per CU, and within 7 %, the 128 x 64 tiles stay (measured there: 0.85 to 1.02 of the wide).
int wide_tiles(int M, int N) {
  const long rows = (M + 127) / 128;
  auto tiles = [&](int cols) { return rows * ((N + cols - 1) / cols); };
  double best = 0.93 * (50.0 + 85.0 * (double)((tiles(64) + 255) / 256));
  int tn = 0;
  constexpr double one[3] = {180, 218, 260}, two[3] = {280, 353, 428};
  for (int t = 3; t <= 5; ++t) {
    const long n = tiles(32 * t);
    const double price = n <= 256 ? one[t - 3] : two[t - 3];
    if (n <= 512 && price < best) {
      best = price;
      tn = t;
    }
  }
  return tn;
}

// K and N multiples of 16; the rows of C are N long
int sgemm(const float *A, int lda, const float *W, int ldw, float *C, int M, int N, int K, hipStream_t st) {
  const int wm = M > 64 ? 4 : (M > 32 ? 2 : 1), wn = 4 / wm;
  const dim3 block(256), grid((N + 64 * wn - 1) / (64 * wn), (M + 32 * wm - 1) / (32 * wm));
  // under half a tile per CU the time is one tile's chain over K, which the small blocks walk in half the clocks
  if ((size_t)grid.x * grid.y < 128) {
    hipLaunchKernelGGL(sgemm_skinny_kernel, dim3((N + 31) / 32, (M + 31) / 32), block, 0, st, A, lda, W, ldw, C, N, M, N, K);
  } else if (wm == 4) {
    switch (wide_tiles(M, N)) {
      case 3: return run_wide<3>(A, lda, W, ldw, C, M, N, K, st);
      case 4: return run_wide<4>(A, lda, W, ldw, C, M, N, K, st);
      case 5: return run_wide<5>(A, lda, W, ldw, C, M, N, K, st);
      default: break;
    }
    hipLaunchKernelGGL((sgemm_tn_kernel<4, 1>), grid, block, 0, st, A, lda, W, ldw, C, N, M, N, K);
  } else if (wm == 2) {
    hipLaunchKernelGGL((sgemm_tn_kernel<2, 2>), grid, block, 0, st, A, lda, W, ldw, C, N, M, N, K);
  } else {
    hipLaunchKernelGGL((sgemm_tn_kernel<1, 4>), grid, block, 0, st, A, lda, W, ldw, C, N, M, N, K);
  }
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}

// ---------------------------------------------------------------- small elementwise kernels
__global__ void half_to_float_kernel(const __half *x, float *y, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) y[i] = __half2float(x[i]);
}

__global__ void neg_exp_kernel(const float *a_log, float *a, size_t n) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) a[i] = static_cast<float>(-exp(static_cast<double>(a_log[i])));  // once, offline: fp64
}

__global__ void fill_u32_kernel(unsigned *p, size_t n, unsigned v) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n) p[i] = v;
}

// max |x| over column ranges of matrices, each as the bit pattern of a non-negative float (which orders like an unsigned
// integer) combined with atomicMax, once per workgroup: thousands of waves on one word took 100 us per tensor.  All
// tensors of a calibration go in one launch, in which a segment has workgroups in proportion to its size and a row as
// many threads as it has pieces of four (the 16 columns of B: 64 rows at once; one row at a time took 490 us).  4 x 256
// tokens of the 2.8B layer, 320 MB: 63 us, fifteen launches before it 980.
constexpr int MAX_SEGS = 16;
struct AbsmaxSegs {
  const float *p[MAX_SEGS];  // first element of the range
  size_t rows[MAX_SEGS], total[MAX_SEGS];
  int ld[MAX_SEGS], w[MAX_SEGS], slot[MAX_SEGS];
  int lt[MAX_SEGS];        // log2 of the threads per row
  unsigned end[MAX_SEGS];  // workgroups up to and with this segment
};

__global__ __launch_bounds__(256) void absmax_kernel(AbsmaxSegs s, unsigned *slots) {
  int i = 0;
  while (blockIdx.x >= s.end[i]) ++i;
  const unsigned first = i ? s.end[i - 1] : 0u, nb = s.end[i] - first;
  const int w = s.w[i], lt = s.lt[i], at = threadIdx.x & ((1 << lt) - 1);
  float m = 0.f;
  for (size_t r = ((blockIdx.x - first) << (8 - lt)) + (threadIdx.x >> lt); r < s.rows[i]; r += (size_t)nb << (8 - lt)) {
    const float *row = s.p[i] + r * s.ld[i];
    const int n = (int)min((size_t)w, s.total[i] - r * w);
#pragma unroll 4
    for (int c = at * 4; c < n; c += 4 << lt) {  // every range is a multiple of four long
      const f4 v = *reinterpret_cast<const f4u *>(row + c);
      m = fmaxf(fmaxf(m, fmaxf(fabsf(v[0]), fabsf(v[1]))), fmaxf(fabsf(v[2]), fabsf(v[3])));
    }
  }
  __shared__ float part[4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0)
    atomicMax(slots + s.slot[i], __float_as_uint(fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]))));
}

struct Obs {
  const float *p;
  size_t rows;
  int ld, c0, c1, slot;
};

int absmax(const Obs *obs, int count, unsigned *slots, hipStream_t st) {
  AbsmaxSegs s{};
  unsigned end = 0;
  for (int i = 0; i < count; ++i) {
    const Obs &o = obs[i];
    int w = o.c1 - o.c0, ld = o.ld;
    size_t rows = o.rows;
    const size_t total = rows * (size_t)w;
    if (w == ld) {  // one long row: cut it into pieces of 4096
      w = ld = 4096;
      rows = (total + 4095) / 4096;
    }
    s.p[i] = o.p + o.c0; s.rows[i] = rows; s.total[i] = total; s.ld[i] = ld; s.w[i] = w; s.slot[i] = o.slot;
    int lt = 2;
    while (lt < 8 && (4 << lt) < w) ++lt;
    s.lt[i] = lt;
    // a workgroup for every 8192 values begun, at most 512
    s.end[i] = end += (unsigned)std::min<size_t>((total + 8191) / 8192, 512);
  }
  hipLaunchKernelGGL(absmax_kernel, dim3(end), dim3(256), 0, st, s, slots);
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}

// causal conv (width 4, zero history) + bias + SiLU in fp32, four channels per thread; xz has row stride ld
__global__ __launch_bounds__(256) void conv_silu_f32_kernel(const float *__restrict__ xz, int ld, const float *__restrict__ w,
                                                            const float *__restrict__ b, int L, int Di,
                                                            float *__restrict__ x, size_t total4) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i >= total4) return;
  const unsigned per = Di / 4;
  const size_t row = i / per;
  const int d = static_cast<int>(i % per) * 4, t = static_cast<int>(row % L);
  f4 wv[4], v = *reinterpret_cast<const f4u *>(b + d);
#pragma unroll
  for (int c = 0; c < 4; ++c) wv[c] = *reinterpret_cast<const f4u *>(w + (size_t)(d + c) * 4);
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    if (t - 3 + j >= 0) {
      const f4 s = *reinterpret_cast<const f4 *>(xz + (row - 3 + j) * ld + d);
#pragma unroll
      for (int c = 0; c < 4; ++c) v[c] += wv[c][j] * s[c];
    }
  }
#pragma unroll
  for (int c = 0; c < 4; ++c) v[c] = v[c] / (1.f + expf(-v[c]));
  *reinterpret_cast<f4 *>(x + row * Di + d) = v;
}

// fp32 selective scan + gate.  A workgroup owns 32 channels of one sequence, 8 lanes per channel with two of the 16
// states each, and walks the tokens in blocks of 32.  What is per (token, channel) is done once by all threads, a block
// ahead of the recurrence, and handed over in LDS together with B and C; the sum C h of a token is one chain over the
// states 0 .. 15 (the scale of the output hangs on its last bit): it travels from lane to lane, each lane one token behind
// the one before it.  It is gated by all threads again, so every access of global memory is a row of 32 channels.  With one
// thread per channel (80 workgroups at 4 x 5120 channels, 256 tokens) the serial chain of loads and exponentials took 367
// us; this takes 96.
constexpr int ST = 32, SC = 32;

__global__ __launch_bounds__(256) void scan_f32_kernel(const float *__restrict__ x, const float *__restrict__ dt_raw,
                                                       const float *__restrict__ dt_bias, const float *__restrict__ A,
                                                       const float *__restrict__ dbc, int nx, int R,
                                                       const float *__restrict__ D, const float *__restrict__ xz, int L,
                                                       int Di, float *__restrict__ g) {
  __shared__ float2 sdt[ST][SC + 1];  // (dt, dt x)
  __shared__ float sy[ST][SC + 1];
  __shared__ __attribute__((aligned(16))) float sbc[ST][32];  // B then C of a token
  const int tid = threadIdx.x;
  const int nc = (Di + SC - 1) / SC;
  const int c0 = (blockIdx.x % nc) * SC;
  const size_t row0 = (size_t)(blockIdx.x / nc) * L;
  // elementwise part: thread -> channel tid % 32, tokens tid / 32 + 8 i
  const int ec = tid & 31, et = tid >> 5, ed = c0 + ec;
  const bool eon = ed < Di;
  const float bias = eon ? dt_bias[ed] : 0.f, Dv = eon ? D[ed] : 0.f;
  // recurrence part: thread -> channel tid / 8, states 2 (tid % 8) and the next
  const int rc = tid >> 3, rg = tid & 7, rd = c0 + rc;
  float a0 = 0.f, a1 = 0.f, h0 = 0.f, h1 = 0.f;
  if (rd < Di) {
    a0 = A[(size_t)rd * 16 + 2 * rg] * LOG2E;
    a1 = A[(size_t)rd * 16 + 2 * rg + 1] * LOG2E;
  }
  float xv[4], pv[4], zv[4], bc[4];
  auto fetch = [&](int t0) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = t0 + et + 8 * i;
      xv[i] = pv[i] = zv[i] = bc[i] = 0.f;
      if (t < L) {
        const size_t row = row0 + t;
        bc[i] = dbc[row * nx + R + ec];
        if (eon) {
          xv[i] = x[row * Di + ed];
          pv[i] = dt_raw[row * Di + ed];
          zv[i] = xz[row * (2 * (size_t)Di) + Di + ed];
        }
      }
    }
  };
  fetch(0);
  for (int t0 = 0; t0 < L; t0 += ST) {
    float xg[4], zg[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float pre = pv[i] + bias;
      const float dt = pre > 20.f ? pre : log1pf(expf(pre));
      sdt[et + 8 * i][ec] = make_float2(dt, dt * xv[i]);
      sbc[et + 8 * i][ec] = bc[i];
      xg[i] = xv[i];
      zg[i] = zv[i];
    }
    __syncthreads();
    if (t0 + ST < L) fetch(t0 + ST);
    const int nt = min(ST, L - t0);
    float y = 0.f;
    for (int i = 0; i < nt + 7; ++i) {
      const int t = i - rg;  // lane rg is rg tokens behind lane 0, whose sum comes to it through the lanes between
      const bool on = t >= 0 && t < nt;
      const int tt = on ? t : 0;
      const float2 d = sdt[tt][rc];
      const float2 B = *reinterpret_cast<const float2 *>(&sbc[tt][2 * rg]);
      const float2 C = *reinterpret_cast<const float2 *>(&sbc[tt][16 + 2 * rg]);
      const float n0 = __builtin_fmaf(exp2f(d.x * a0), h0, d.y * B.x), n1 = __builtin_fmaf(exp2f(d.x * a1), h1, d.y * B.y);
      h0 = on ? n0 : h0;
      h1 = on ? n1 : h1;
      const float in = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), 0x111, 0xf, 0xf, true));  // row_shr:1
      y = __builtin_fmaf(C.y, h1, __builtin_fmaf(C.x, h0, rg ? in : 0.f));
      if (rg == 7 && on) sy[t][rc] = y;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int t = et + 8 * i;
      if (t < nt && eon) {
        const float y = __builtin_fmaf(Dv, xg[i], sy[t][ec]);
        g[(row0 + t0 + t) * Di + ed] = y * zg[i] / (1.f + expf(-zg[i]));
      }
    }
  }
}

// Radix select: the value of 1-based rank `rank` among |x|, most significant byte first.  Pass p counts byte 3 - p of the bit
// patterns whose higher bytes are those already found; every workgroup finds these again from the earlier histograms
// (hist[4][256], cleared beforehand), so that the four passes follow one another without the host in between (it used
// to read 2 KB and wait after each: four round trips of about 55 us).
__device__ unsigned select_prefix(const unsigned long long *hist, int passes, unsigned long long rank,
                                  unsigned long long *sum) {
  __shared__ unsigned byte;
  unsigned prefix = 0;
  unsigned long long below = 0;  // elements known to be smaller than every candidate
  const int t = threadIdx.x;
  for (int p = 0; p < passes; ++p) {
    const unsigned long long own = hist[p * 256 + t];
    sum[t] = own;
    if (t == 0) byte = 255u;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {  // inclusive scan
      const unsigned long long v = t >= off ? sum[t - off] : 0ull;
      __syncthreads();
      sum[t] += v;
      __syncthreads();
    }
    const unsigned long long upto = below + sum[t];
    if (upto >= rank && upto - own < rank) byte = t;  // at most one bin
    __syncthreads();
    prefix |= byte << (24 - 8 * p);
    below += byte ? sum[byte - 1] : 0ull;
    __syncthreads();
  }
  return prefix;
}

// Workgroups, one per 20480 values between one and three per CU: in the first two passes all of them add to the same few bins, and additions to one
// word in memory come 14 ns apart, while many values need the loads of several workgroups per CU.  Calibration with 256 / 512 / 768 / 1024
// of them: 1.6 M values (4 x 256 tokens of the 130M layer) 275 / 282 / 289 / 295 us, 5.2 M (4 x 256 of the 2.8B layer) 865 / 866 / 870 /
// 876, 8.4 M 1054 / 1050 / 1053 / 1057, 12.6 M 1012 / 989 / 988 / 992, 21 M 2770 / 2721 / 2712 / 2711 (copies of the bins in LDS change nothing).
int hist_workgroups(size_t n) { return (int)std::min<size_t>(std::max<size_t>(n / 20480, 256), 768); }

__global__ __launch_bounds__(256) void select_hist_kernel(const float *__restrict__ x, size_t n, int pass,
                                                          unsigned long long rank, unsigned long long *hist) {
  __shared__ unsigned long long sum[256];
  __shared__ unsigned local[256];
  local[threadIdx.x] = 0;
  const unsigned prefix = select_prefix(hist, pass, rank, sum);
  const unsigned mask = pass ? ~0u << (32 - 8 * pass) : 0u;
  const int shift = 24 - 8 * pass;
  __syncthreads();
#pragma unroll 4
  for (size_t i = ((size_t)blockIdx.x * 256 + threadIdx.x) * 4; i < n; i += (size_t)gridDim.x * 1024) {  // n: a multiple of 16
    const f4 v = *reinterpret_cast<const f4 *>(x + i);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const unsigned bits = __float_as_uint(fabsf(v[e]));
      if ((bits & mask) == prefix) atomicAdd(&local[(bits >> shift) & 255u], 1u);
    }
  }
  __syncthreads();
  if (local[threadIdx.x]) atomicAdd(&hist[pass * 256 + threadIdx.x], (unsigned long long)local[threadIdx.x]);
}

__global__ __launch_bounds__(256) void select_finish_kernel(const unsigned long long *hist, unsigned long long rank,
                                                            unsigned *out) {
  __shared__ unsigned long long sum[256];
  const unsigned prefix = select_prefix(hist, 4, rank, sum);
  if (threadIdx.x == 0) *out = prefix;
}

// ---------------------------------------------------------------- model-optimal clipping scalar
// Section 5.1 names a clipping optimisation as the enhanced variant; the rule is the stationary
// point of (4^-bits / 3) s^2 #{0 < |x| <= s} + sum_{|x| > s} (|x| - s)^2, iterated as
//   s <- sum(|x| : |x| > s) / (4^-bits / 3 * #{0 < |x| <= s} + #{|x| > s}).
// One pass gathers the three sums per workgroup, a one-workgroup pass adds them in a fixed order
// (same result on every run) and moves s.  state[0] = s, state[1] = updates made, state[2] = done.
struct ClipPart {
  double sum_out;
  unsigned long long n_out, n_in;
};
constexpr int CLIP_BLOCKS = 1024;

__global__ __launch_bounds__(256) void clip_stats_kernel(const float *__restrict__ x, size_t n,
                                                         const double *__restrict__ state, ClipPart *parts) {
  const double s = state[0];
  double sum = 0.0;
  unsigned long long n_out = 0, n_in = 0;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) {
    const double a = static_cast<double>(fabsf(x[i]));
    if (a > s) {
      sum += a;
      ++n_out;
    } else if (a > 0.0) {
      ++n_in;
    }
  }
  __shared__ ClipPart part[256];
  part[threadIdx.x] = ClipPart{sum, n_out, n_in};
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      part[threadIdx.x].sum_out += part[threadIdx.x + off].sum_out;
      part[threadIdx.x].n_out += part[threadIdx.x + off].n_out;
      part[threadIdx.x].n_in += part[threadIdx.x + off].n_in;
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) parts[blockIdx.x] = part[0];
}

__global__ __launch_bounds__(256) void clip_update_kernel(const ClipPart *__restrict__ parts, int nparts, double c,
                                                          int first, double *state) {
  __shared__ ClipPart part[256];
  ClipPart acc{0.0, 0, 0};
  for (int i = threadIdx.x; i < nparts; i += 256) {
    acc.sum_out += parts[i].sum_out;
    acc.n_out += parts[i].n_out;
    acc.n_in += parts[i].n_in;
  }
  part[threadIdx.x] = acc;
  __syncthreads();
  for (int off = 128; off > 0; off >>= 1) {
    if ((int)threadIdx.x < off) {
      part[threadIdx.x].sum_out += part[threadIdx.x + off].sum_out;
      part[threadIdx.x].n_out += part[threadIdx.x + off].n_out;
      part[threadIdx.x].n_in += part[threadIdx.x + off].n_in;
    }
    __syncthreads();
  }
  if (threadIdx.x != 0 || state[2] != 0.0) return;
  const ClipPart t = part[0];
  if (first) {  // the start value: every element counts as outside, which makes the quotient mean |x|
    state[0] = t.n_out ? t.sum_out / static_cast<double>(t.n_out) : 0.0;
    return;
  }
  if (t.n_out == 0) {
    state[2] = 1.0;
    return;
  }
  const double nxt = t.sum_out / (c * static_cast<double>(t.n_in) + static_cast<double>(t.n_out));
  if (nxt == state[0]) {
    state[2] = 1.0;
    return;
  }
  state[0] = nxt;
  state[1] += 1.0;
}

__global__ void clip_init_kernel(double *state) {
  if (threadIdx.x == 0) {
    state[0] = -1.0;  // below every |x|
    state[1] = 0.0;
    state[2] = 0.0;
  }
}

constexpr size_t CLIP_WS_BYTES = 256 + CLIP_BLOCKS * sizeof(ClipPart);

// The scale of a tensor with this largest magnitude (1 if it is zero) and its reciprocal, each rounded once from 64 bits.
__host__ __device__ inline float scale_of(float m) { return m > 0.f ? (float)((double)m / 127.0) : 1.0f; }
__host__ __device__ inline float inverse_scale(float m) { return (float)(1.0 / (double)scale_of(m)); }

typedef unsigned u1u __attribute__((aligned(1)));
struct QuantSegs {
  const float *x[MAX_SEGS];
  void *q[MAX_SEGS];
  size_t n[MAX_SEGS];
  const unsigned *max_bits[MAX_SEGS];  // largest magnitude: 1 / scale is formed here, by the operations the host takes
  int copy[MAX_SEGS];
  unsigned end[MAX_SEGS];
};
constexpr int Q_PER_WG = 8192;

// Eq. 2 for several tensors in one launch: q = clamp(rne(x * inv_s)), four values per thread and step; every tensor is a
// multiple of four long.  A segment marked `copy` is copied as fp32 instead.
__global__ __launch_bounds__(256) void quantize_f32_kernel(QuantSegs s) {
  int i = 0;
  while (blockIdx.x >= s.end[i]) ++i;
  const size_t at = (size_t)(blockIdx.x - (i ? s.end[i - 1] : 0u)) * Q_PER_WG;
  const size_t stop = min(s.n[i], at + Q_PER_WG);
  const float *x = s.x[i];
  const bool copy = s.copy[i];
  const float inv_s = copy ? 0.f : inverse_scale(__uint_as_float(*s.max_bits[i]));
#pragma unroll 4
  for (size_t k = at + threadIdx.x * 4; k < stop; k += 1024) {
    const f4 v = *reinterpret_cast<const f4u *>(x + k);
    if (copy) {
      *reinterpret_cast<f4u *>(static_cast<float *>(s.q[i]) + k) = v;
      continue;
    }
    unsigned word = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float r = fminf(fmaxf(__builtin_rintf(v[e] * inv_s), -128.f), 127.f);
      word |= ((unsigned)static_cast<int>(r) & 255u) << (8 * e);
    }
    *reinterpret_cast<u1u *>(static_cast<int8_t *>(s.q[i]) + k) = word;
  }
}

struct Quant {
  const float *x;
  void *q;
  size_t n;
  const unsigned *max_bits;
  int copy;
};

int quantize_f32(const Quant *qs, int count, hipStream_t st) {
  QuantSegs s{};
  unsigned end = 0;
  for (int i = 0; i < count; ++i) {
    s.x[i] = qs[i].x; s.q[i] = qs[i].q; s.n[i] = qs[i].n; s.max_bits[i] = qs[i].max_bits; s.copy[i] = qs[i].copy;
    s.end[i] = end += (unsigned)((qs[i].n + Q_PER_WG - 1) / Q_PER_WG);
  }
  hipLaunchKernelGGL(quantize_f32_kernel, dim3(end), dim3(256), 0, st, s);
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}

// max(0, -min x) over x[0, n), as the bit pattern of a non-negative float
__global__ __launch_bounds__(256) void negmax_kernel(const float *__restrict__ x, size_t n, unsigned *slot) {
  float m = 0.f;
  for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n; i += (size_t)gridDim.x * 256) m = fmaxf(m, -x[i]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
  if ((threadIdx.x & 63) == 0) atomicMax(slot, __float_as_uint(m));
}

// out[r] = factor * sum_k w[r, k] (int32; |sum| <= 128 K): one workgroup per row
__global__ __launch_bounds__(256) void scaled_rowsum_i8_kernel(const int8_t *__restrict__ w, int K, int factor,
                                                               int32_t *__restrict__ out) {
  int acc = 0;
  for (int k = threadIdx.x; k < K; k += 256) acc += w[(size_t)blockIdx.x * K + k];
  __shared__ int part[4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) out[blockIdx.x] = factor * (part[0] + part[1] + part[2] + part[3]);
}

inline unsigned nblk(size_t n) { return (unsigned)((n + 255) / 256); }

struct CalPlan {
  size_t u32, xz, x, dbc, dtr, g, gH, woh, a, slots, hist, clip, total;
};

CalPlan cal_plan(const quamba_dims *d, int nb, int Lc) {
  const size_t M = (size_t)nb * Lc, Di = d->d_inner, Dm = d->d_model, NX = d->dt_rank + 2 * d->d_state;
  CalPlan p{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += align_up(bytes, 256);
    return at;
  };
  p.u32 = take(M * Dm * 4);
  p.xz = take(M * 2 * Di * 4);
  p.x = take(M * Di * 4);
  p.dbc = take(M * NX * 4);
  p.dtr = take(M * Di * 4);
  p.g = take(M * Di * 4);
  p.gH = take(M * Di * 4);
  p.woh = take(Dm * Di * 4);
  p.a = take(Di * d->d_state * 4);
  p.slots = take(32 * 4);
  // four histograms of 2 KB: the last three lie in the area of the clip search, which only the other rule for x uses
  static_assert(CLIP_WS_BYTES >= 3 * 256 * 8, "the histograms fit");
  p.hist = take(256 * 8);
  p.clip = take(CLIP_WS_BYTES);
  p.total = off;
  return p;
}

enum Slot { S_U, S_XPRE, S_Z, S_DTL, S_B, S_C, S_DT, S_Y, S_WIN, S_CW, S_WX, S_WDT, S_A, S_D, S_WOH, S_COUNT };

struct CalBufs {
  float *u32, *xz, *x, *dbc, *dtr, *g, *gH, *woh, *A;
  unsigned *slots;
  unsigned long long *hist;
};

CalBufs carve(const CalPlan &p, void *ws) {
  char *base = static_cast<char *>(ws);
  auto f = [&](size_t off) { return reinterpret_cast<float *>(base + off); };
  return CalBufs{f(p.u32), f(p.xz), f(p.x), f(p.dbc), f(p.dtr), f(p.g), f(p.gH), f(p.woh), f(p.a),
                 reinterpret_cast<unsigned *>(base + p.slots), reinterpret_cast<unsigned long long *>(base + p.hist)};
}

// The unquantized mixer up to the gated scan output (Section 3.1), fp32: leaves x_pre | z, x,
// dt_low | B | C, dt_raw and g in the workspace.  calib_u == nullptr: the input is already in b.u32.
int fp_forward(const quamba_dims *d, const quamba_fp_weights *w, const __half *calib_u, int nb, int Lc,
               const CalBufs &b, hipStream_t st) {
  const int Dm = d->d_model, Di = d->d_inner, N = d->d_state, R = d->dt_rank, NX = R + 2 * N;
  const size_t M = (size_t)nb * Lc;
  if (calib_u) hipLaunchKernelGGL(half_to_float_kernel, dim3(nblk(M * Dm)), dim3(256), 0, st, calib_u, b.u32, M * Dm);
  hipLaunchKernelGGL(neg_exp_kernel, dim3(nblk((size_t)Di * N)), dim3(256), 0, st, w->A_log, b.A, (size_t)Di * N);
  QUAMBA_LAUNCH_CHECK();
  int rc;
  if ((rc = sgemm(b.u32, Dm, w->W_in, Dm, b.xz, (int)M, 2 * Di, Dm, st))) return rc;
  hipLaunchKernelGGL(conv_silu_f32_kernel, dim3(nblk(M * Di / 4)), dim3(256), 0, st, b.xz, 2 * Di, w->conv_w,
                     w->conv_b, Lc, Di, b.x, M * Di / 4);
  QUAMBA_LAUNCH_CHECK();
  if ((rc = sgemm(b.x, Di, w->W_x, Di, b.dbc, (int)M, NX, Di, st))) return rc;
  if ((rc = sgemm(b.dbc, NX, w->W_dt, R, b.dtr, (int)M, Di, R, st))) return rc;
  hipLaunchKernelGGL(scan_f32_kernel, dim3((unsigned)((Di + SC - 1) / SC) * nb), dim3(256), 0, st, b.x, b.dtr, w->dt_bias, b.A, b.dbc, NX,
                     R, w->D, b.xz, Lc, Di, b.g);
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}

}  // namespace

size_t calibrate_workspace_bytes(const quamba_dims *d, int nb, int Lc) { return cal_plan(d, nb, Lc).total; }

size_t clip_search_workspace_bytes() { return CLIP_WS_BYTES; }

// Runs the fixed-point iteration above on x[0, n) and returns the scalar and the number of updates
// on the host (synchronises the stream).
int clip_search(const float *x, size_t n, int bits, int max_iters, double *clip_out, int *iters_out, void *ws,
                size_t ws_bytes, hipStream_t st) {
  if (ws_bytes < CLIP_WS_BYTES) return fail(QUAMBA_EWORKSPACE, "clip_search: workspace %zu < %zu", ws_bytes, CLIP_WS_BYTES);
  double *state = static_cast<double *>(ws);
  ClipPart *parts = reinterpret_cast<ClipPart *>(static_cast<char *>(ws) + 256);
  const double c = std::pow(4.0, -static_cast<double>(bits)) / 3.0;
  const int blocks = (int)std::min<size_t>(std::max<size_t>((n + 255) / 256, 1), CLIP_BLOCKS);
  hipLaunchKernelGGL(clip_init_kernel, dim3(1), dim3(64), 0, st, state);
  for (int it = 0; it <= max_iters; ++it) {  // pass 0 produces the start value
    hipLaunchKernelGGL(clip_stats_kernel, dim3(blocks), dim3(256), 0, st, x, n, state, parts);
    hipLaunchKernelGGL(clip_update_kernel, dim3(1), dim3(256), 0, st, parts, blocks, c, it == 0 ? 1 : 0, state);
    QUAMBA_LAUNCH_CHECK();
  }
  double h[3];
  QUAMBA_HIP(hipMemcpyAsync(h, state, sizeof(h), hipMemcpyDeviceToHost, st));
  QUAMBA_HIP(hipStreamSynchronize(st));
  *clip_out = h[0];
  if (iters_out) *iters_out = static_cast<int>(h[1]);
  return QUAMBA_OK;
}

// The unquantized mixer of Section 3.1 in fp32 on u [nb, Lc, Dm] (fp16), each sequence from an
// empty history: out [nb * Lc, Dm] fp32.  The reference the quantized path is compared with.
int fp_mixer(const quamba_dims *d, const quamba_fp_weights *w, const __half *u, int nb, int Lc, float *out,
             void *ws, size_t ws_bytes, hipStream_t st) {
  const CalPlan p = cal_plan(d, nb, Lc);
  if (ws_bytes < p.total) return fail(QUAMBA_EWORKSPACE, "fp mixer: workspace %zu < %zu", ws_bytes, p.total);
  const CalBufs b = carve(p, ws);
  int rc;
  if ((rc = fp_forward(d, w, u, nb, Lc, b, st))) return rc;
  return sgemm(b.g, d->d_inner, w->W_out, d->d_inner, out, nb * Lc, d->d_model, d->d_inner, st);
}

int calibrate(const quamba_dims *d, const quamba_fp_weights *w, const __half *calib_u, int nb, int Lc,
              int x_rule, double x_percentile, quamba_qweights *oq, quamba_scales *os, void *ws, size_t ws_bytes,
              hipStream_t st, float *out_f32, float *x_clip_out = nullptr);

namespace {
// res[row] += out[row]; u[row] = res[row] / sqrt(mean(res[row]^2) + eps) * w   (fp32; one workgroup per row)
__global__ __launch_bounds__(256) void add_rmsnorm_f32_kernel(float *__restrict__ res, const float *__restrict__ out,
                                                              const __half *__restrict__ w, float eps, int Dm,
                                                              float *__restrict__ u) {
  const size_t row = blockIdx.x;
  float ss = 0.f;
  for (int i = threadIdx.x; i < Dm; i += 256) {
    const float r = res[row * Dm + i] + out[row * Dm + i];
    res[row * Dm + i] = r;
    ss += r * r;
  }
  __shared__ float part[4];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = ss;
  __syncthreads();
  const float rinv = 1.f / sqrtf((part[0] + part[1] + part[2] + part[3]) / static_cast<float>(Dm) + eps);
  for (int i = threadIdx.x; i < Dm; i += 256) u[row * Dm + i] = res[row * Dm + i] * rinv * __half2float(w[i]);
}
}  // namespace

// One block of a stack (Section 5.1: every layer gets its own static scales): the block input is
// the RMSNorm of the unquantized residual stream, which the call advances.
int calibrate_block(const quamba_dims *d, const quamba_fp_weights *w, const __half *norm_w, float eps, float *res,
                    float *out, int nb, int Lc, double x_percentile, quamba_qweights *oq, quamba_scales *os, void *ws,
                    size_t ws_bytes, hipStream_t st) {
  const CalPlan p = cal_plan(d, nb, Lc);
  if (ws_bytes < p.total) return fail(QUAMBA_EWORKSPACE, "calibrate: workspace %zu < %zu", ws_bytes, p.total);
  float *u32 = reinterpret_cast<float *>(static_cast<char *>(ws) + p.u32);
  hipLaunchKernelGGL(add_rmsnorm_f32_kernel, dim3((unsigned)((size_t)nb * Lc)), dim3(256), 0, st, res, out, norm_w, eps,
                     d->d_model, u32);
  QUAMBA_LAUNCH_CHECK();
  return calibrate(d, w, nullptr, nb, Lc, QUAMBA_X_PERCENTILE, x_percentile, oq, os, ws, ws_bytes, st, out);
}

// calib_u == nullptr: the fp32 block input is already in the workspace's own input buffer
// (calibrate_block puts it there).  out_f32 != nullptr: also receives the unquantized block output
// g W_out^T, which feeds the next block of a stack.
int calibrate(const quamba_dims *d, const quamba_fp_weights *w, const __half *calib_u, int nb, int Lc,
              int x_rule, double x_percentile, quamba_qweights *oq, quamba_scales *os, void *ws, size_t ws_bytes,
              hipStream_t st, float *out_f32, float *x_clip_out) {
  const CalPlan p = cal_plan(d, nb, Lc);
  if (ws_bytes < p.total) return fail(QUAMBA_EWORKSPACE, "calibrate: workspace %zu < %zu", ws_bytes, p.total);
  const int Dm = d->d_model, Di = d->d_inner, N = d->d_state, R = d->dt_rank, NX = R + 2 * N;
  const size_t M = (size_t)nb * Lc;
  char *base = static_cast<char *>(ws);
  const CalBufs b = carve(p, ws);
  float *u32 = b.u32, *xz = b.xz, *x = b.x, *dbc = b.dbc, *dtr = b.dtr, *g = b.g, *gH = b.gH, *woh = b.woh, *A = b.A;
  unsigned *slots = b.slots;
  unsigned long long *hist = b.hist;

  {  // observer slots and the histograms behind them
    const size_t words = (p.hist - p.slots) / 4 + 4 * 256 * 2;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(nblk(words)), dim3(256), 0, st, slots, words, 0u);
  }
  QUAMBA_LAUNCH_CHECK();
  int rc;
  if ((rc = fp_forward(d, w, calib_u, nb, Lc, b, st))) return rc;
  if (out_f32 && (rc = sgemm(g, Di, w->W_out, Di, out_f32, (int)M, Dm, Di, st))) return rc;
  if ((rc = launch_hadamard_f32(g, (int)M, Di, gH, st))) return rc;      // y^H = H_n g
  if ((rc = launch_hadamard_f32(w->W_out, Dm, Di, woh, st))) return rc;  // rows of W_out^H

  // observers
  const Obs obs[] = {
      {u32, M, Dm, 0, Dm, S_U},         {xz, M, 2 * Di, 0, Di, S_XPRE},    {xz, M, 2 * Di, Di, 2 * Di, S_Z},
      {dbc, M, NX, 0, R, S_DTL},        {dbc, M, NX, R, R + N, S_B},       {dbc, M, NX, R + N, NX, S_C},
      {dtr, M, Di, 0, Di, S_DT},        {gH, M, Di, 0, Di, S_Y},           {w->W_in, (size_t)2 * Di, Dm, 0, Dm, S_WIN},
      {w->conv_w, (size_t)Di, 4, 0, 4, S_CW}, {w->W_x, (size_t)NX, Di, 0, Di, S_WX},
      {w->W_dt, (size_t)Di, R, 0, R, S_WDT},  {A, (size_t)Di, N, 0, N, S_A},   {w->D, 1, Di, 0, Di, S_D},
      {woh, (size_t)Dm, Di, 0, Di, S_WOH}};
  if ((rc = absmax(obs, sizeof(obs) / sizeof(obs[0]), slots, st))) return rc;

  const size_t nx = M * Di;
  if (x_rule != QUAMBA_X_MSE_CLIP) {
    // percentile maximum of |x| (Section 4.2): value of 1-based rank ceil(p/100 * n)
    size_t rank = (size_t)std::ceil(x_percentile * (double)nx / 100.0);
    if (rank < 1) rank = 1;
    if (rank > nx) rank = nx;
    for (int pass = 0; pass < 4; ++pass)
      hipLaunchKernelGGL(select_hist_kernel, dim3(hist_workgroups(nx)), dim3(256), 0, st, x, nx, pass, (unsigned long long)rank, hist);
    hipLaunchKernelGGL(select_finish_kernel, dim3(1), dim3(256), 0, st, hist, (unsigned long long)rank, slots + S_COUNT);
    QUAMBA_LAUNCH_CHECK();
  }
  // quantize the weights (Eq. 2) and copy the two fp32 bias vectors; with the scales formed on the device, so that the host is waited for once
  const Quant qws[] = {{w->W_in, oq->W_in, (size_t)2 * Di * Dm, slots + S_WIN, 0}, {w->conv_w, oq->conv_w, (size_t)Di * 4, slots + S_CW, 0},
                       {w->W_x, oq->W_x, (size_t)NX * Di, slots + S_WX, 0},        {w->W_dt, oq->W_dt, (size_t)Di * R, slots + S_WDT, 0},
                       {A, oq->A, (size_t)Di * N, slots + S_A, 0},                 {w->D, oq->D, (size_t)Di, slots + S_D, 0},
                       {woh, oq->W_outH, (size_t)Dm * Di, slots + S_WOH, 0},     {w->conv_b, oq->conv_b, (size_t)Di, nullptr, 1},
                       {w->dt_bias, oq->dt_bias, (size_t)Di, nullptr, 1}};
  if ((rc = quantize_f32(qws, sizeof(qws) / sizeof(qws[0]), st))) return rc;
  float mx[S_COUNT + 1];
  QUAMBA_HIP(hipMemcpyAsync(mx, slots, sizeof(mx), hipMemcpyDeviceToHost, st));
  QUAMBA_HIP(hipStreamSynchronize(st));
  float xp = mx[S_COUNT];
  if (x_rule == QUAMBA_X_MSE_CLIP) {
    double clip;
    if ((rc = clip_search(x, nx, 8, 32, &clip, nullptr, base + p.clip, CLIP_WS_BYTES, st))) return rc;
    xp = static_cast<float>(clip);
  }

  if (x_clip_out) *x_clip_out = xp;  // the clipping value of x before it becomes a scale
  auto sc_of = scale_of;
  quamba_scales s{};
  s.s_u = sc_of(mx[S_U]); s.s_xpre = sc_of(mx[S_XPRE]); s.s_z = sc_of(mx[S_Z]); s.s_x = sc_of(xp);
  s.s_dtl = sc_of(mx[S_DTL]); s.s_B = sc_of(mx[S_B]); s.s_C = sc_of(mx[S_C]); s.s_dt = sc_of(mx[S_DT]);
  s.s_y = sc_of(mx[S_Y]); s.s_Win = sc_of(mx[S_WIN]); s.s_cw = sc_of(mx[S_CW]); s.s_Wx = sc_of(mx[S_WX]);
  s.s_Wdt = sc_of(mx[S_WDT]); s.s_A = sc_of(mx[S_A]); s.s_D = sc_of(mx[S_D]); s.s_WoutH = sc_of(mx[S_WOH]);
  const double du = s.s_u, dxp = s.s_xpre, dz = s.s_z, dx = s.s_x, ddtl = s.s_dtl, dB = s.s_B, dC = s.s_C,
               ddt = s.s_dt, dy = s.s_y, dWin = s.s_Win, dcw = s.s_cw, dWx = s.s_Wx, dWdt = s.s_Wdt,
               dWoh = s.s_WoutH;
  s.inv_s_u = (float)(1.0 / du);
  s.m_in_x = (float)(du * dWin / dxp);
  s.m_in_z = (float)(du * dWin / dz);
  s.m_conv = (float)(dcw * dxp);
  s.inv_s_x = (float)(1.0 / dx);
  s.m_x_dt = (float)(dx * dWx / ddtl);
  s.m_x_B = (float)(dx * dWx / dB);
  s.m_x_C = (float)(dx * dWx / dC);
  s.m_dt = (float)(ddtl * dWdt / ddt);
  s.inv_s_y = (float)(1.0 / dy);
  s.m_out = (float)(dy * dWoh / (double)Di);
  *os = s;
  return QUAMBA_OK;
}

// Calibration of the Appendix H comparison variant: Quamba's calibration, then the scale of H_n x
// (absmax over the calibration batch) and the x_proj weight with every row transformed by the same
// H_n, quantized per tensor; (H w) . (H x) = n (w . x) puts 1/n into the multipliers.
int calibrate_hadx(const quamba_dims *d, const quamba_fp_weights *w, const __half *calib_u, int nb, int Lc,
                   double x_percentile, quamba_qweights *oq, quamba_scales *os, quamba_hadx *oh, void *ws,
                   size_t ws_bytes, hipStream_t st) {
  int rc;
  if ((rc = calibrate(d, w, calib_u, nb, Lc, QUAMBA_X_PERCENTILE, x_percentile, oq, os, ws, ws_bytes, st, nullptr)))
    return rc;
  const CalPlan p = cal_plan(d, nb, Lc);
  const CalBufs b = carve(p, ws);
  const int Di = d->d_inner, Dm = d->d_model, NX = d->dt_rank + 2 * d->d_state;
  const size_t M = (size_t)nb * Lc;
  if (NX > Dm) return fail(QUAMBA_EUNSUPPORTED, "calibrate: dt_rank + 2 d_state = %d exceeds d_model = %d", NX, Dm);
  // the forward pass left x in the workspace; gH and woh are free again
  hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, st, b.slots, (size_t)32, 0u);
  QUAMBA_LAUNCH_CHECK();
  if ((rc = launch_hadamard_f32(b.x, (int)M, Di, b.gH, st))) return rc;
  if ((rc = launch_hadamard_f32(w->W_x, NX, Di, b.woh, st))) return rc;
  const Obs obs[] = {{b.gH, M, Di, 0, Di, 0}, {b.woh, (size_t)NX, Di, 0, Di, 1}};
  if ((rc = absmax(obs, 2, b.slots, st))) return rc;
  float mx[2];
  QUAMBA_HIP(hipMemcpyAsync(mx, b.slots, sizeof(mx), hipMemcpyDeviceToHost, st));
  QUAMBA_HIP(hipStreamSynchronize(st));
  auto sc_of = scale_of;
  oh->s_xH = sc_of(mx[0]);
  oh->s_WxH = sc_of(mx[1]);
  const double a = oh->s_xH, c = oh->s_WxH;
  oh->inv_s_xH = (float)(1.0 / a);
  oh->m_xh_dt = (float)(a * c / ((double)Di * (double)os->s_dtl));
  oh->m_xh_B = (float)(a * c / ((double)Di * (double)os->s_B));
  oh->m_xh_C = (float)(a * c / ((double)Di * (double)os->s_C));
  oh->xhat_scale = (float)(a / (double)Di);
  const size_t nw = (size_t)NX * Di;
  const Quant qw{b.woh, oh->W_xH, nw, b.slots + 1, 0};
  if ((rc = quantize_f32(&qw, 1, st))) return rc;
  QUAMBA_HIP(hipStreamSynchronize(st));
  return QUAMBA_OK;
}

// Calibration with an asymmetric grid for the scan input (Appendix K): Quamba's calibration, then
// lo = min(min x, 0), hi = the percentile maximum, s = (hi - lo) / 255, zero point
// clamp(rne(-128 - lo / s)), and the x_proj column term -zp * rowsum(W_x_q).
int calibrate_xasym(const quamba_dims *d, const quamba_fp_weights *w, const __half *calib_u, int nb, int Lc,
                    double x_percentile, quamba_qweights *oq, quamba_scales *os, quamba_xasym *oa, void *ws,
                    size_t ws_bytes, hipStream_t st) {
  int rc;
  float hi = 0.f;
  if ((rc = calibrate(d, w, calib_u, nb, Lc, QUAMBA_X_PERCENTILE, x_percentile, oq, os, ws, ws_bytes, st, nullptr, &hi)))
    return rc;
  const CalPlan p = cal_plan(d, nb, Lc);
  const CalBufs b = carve(p, ws);
  const int Di = d->d_inner, NX = d->dt_rank + 2 * d->d_state;
  const size_t nx = (size_t)nb * Lc * Di;
  hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, st, b.slots, (size_t)32, 0u);
  hipLaunchKernelGGL(negmax_kernel, dim3((unsigned)std::min<size_t>((nx + 255) / 256, 2048)), dim3(256), 0, st, b.x, nx,
                     b.slots);
  QUAMBA_LAUNCH_CHECK();
  float neg;
  QUAMBA_HIP(hipMemcpyAsync(&neg, b.slots, sizeof(neg), hipMemcpyDeviceToHost, st));
  QUAMBA_HIP(hipStreamSynchronize(st));
  const double lo = -(double)neg, span = (double)hi - lo;
  const float s = span > 0.0 ? (float)(span / 255.0) : 1.0f;
  int zp = (int)std::nearbyint(-128.0 - lo / (double)s);
  zp = std::min(127, std::max(-128, zp));
  oa->s_x = s;
  oa->inv_s_x = (float)(1.0 / (double)s);
  oa->zero_point = zp;
  oa->m_x_dt = (float)((double)s * (double)os->s_Wx / (double)os->s_dtl);
  oa->m_x_B = (float)((double)s * (double)os->s_Wx / (double)os->s_B);
  oa->m_x_C = (float)((double)s * (double)os->s_Wx / (double)os->s_C);
  hipLaunchKernelGGL(scaled_rowsum_i8_kernel, dim3(NX), dim3(256), 0, st, oq->W_x, Di, -zp, oa->col_bias);
  QUAMBA_LAUNCH_CHECK();
  QUAMBA_HIP(hipStreamSynchronize(st));
  return QUAMBA_OK;
}

// Calibration with a non-uniform 8-bit format for the scan input (Appendix K): Quamba's calibration,
// then the format's scale (log2: the maximum of |x| over the batch; E4M3: the percentile maximum
// over 448), the multipliers with it, and the int8 codes of W_x as bfloat16 for the matrix units.
int calibrate_xfmt(const quamba_dims *d, const quamba_fp_weights *w, const __half *calib_u, int nb, int Lc, int format,
                   double x_percentile, quamba_qweights *oq, quamba_scales *os, quamba_xfmt *of, void *ws,
                   size_t ws_bytes, hipStream_t st) {
  int rc;
  float hi = 0.f;
  if ((rc = calibrate(d, w, calib_u, nb, Lc, QUAMBA_X_PERCENTILE, x_percentile, oq, os, ws, ws_bytes, st, nullptr, &hi)))
    return rc;
  const CalPlan p = cal_plan(d, nb, Lc);
  const CalBufs b = carve(p, ws);
  const int Di = d->d_inner, NX = d->dt_rank + 2 * d->d_state;
  float s;
  if (format == QUAMBA_XFMT_E4M3) {
    s = hi > 0.f ? (float)((double)hi / 448.0) : 1.0f;
  } else {
    hipLaunchKernelGGL(fill_u32_kernel, dim3(1), dim3(256), 0, st, b.slots, (size_t)32, 0u);
    QUAMBA_LAUNCH_CHECK();
    const Obs obs{b.x, (size_t)nb * Lc, Di, 0, Di, 0};
    if ((rc = absmax(&obs, 1, b.slots, st))) return rc;
    float mx;
    QUAMBA_HIP(hipMemcpyAsync(&mx, b.slots, sizeof(mx), hipMemcpyDeviceToHost, st));
    QUAMBA_HIP(hipStreamSynchronize(st));
    s = mx > 0.f ? mx : 1.0f;
  }
  of->format = format;
  of->s_x = s;
  of->inv_s_x = (float)(1.0 / (double)s);
  of->m_x_dt = (float)((double)s * (double)os->s_Wx / (double)os->s_dtl);
  of->m_x_B = (float)((double)s * (double)os->s_Wx / (double)os->s_B);
  of->m_x_C = (float)((double)s * (double)os->s_Wx / (double)os->s_C);
  if ((rc = launch_i8_to_bf16(oq->W_x, NX, Di, of->W_x_bf16, st))) return rc;
  QUAMBA_HIP(hipStreamSynchronize(st));
  return QUAMBA_OK;
}

}  // namespace quamba

extern "C" int quamba_debug_percentile_workgroups(long long values) { return values > 0 ? quamba::hist_workgroups((size_t)values) : 0; }
