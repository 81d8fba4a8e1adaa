// Fused fast Hadamard transform + int8 quantization of the gated scan output (Section 4.2
// "SSM outputs", Eq. 3; Section 3.3): per token row, yH = H_n g, yH_q = clamp(rne(yH / s_y)).
//
// n = k * 2^m with k in {1, 12, 20} and H_n = H_k (x) H_{2^m} (index = a * 2^m + b): the
// 2^m part is the Sylvester / natural-order Walsh-Hadamard matrix, done as butterflies; the
// k part (Section 3.3: a known Hadamard matrix of non-power-of-two order) is the first Paley
// construction for q = k - 1 prime, applied as a dense +-1 product of order k.
//
// For fp16 input the order-k factor runs on the matrix cores: y[a, w] = sum_b H_k[a, b] x[b, w]
// is a (k x k) by (k x 2^m) product whose operands (+-1 and fp16 values) are exact in fp16 and
// whose sums accumulate in fp32, so only the order of the fp32 additions differs from the
// scalar form.  H_k is zero-padded to 32 x 32.
//
// One workgroup per row.  The row sits in LDS as fp32; each pass gathers 2^r (or k) elements
// per work item at a power-of-two stride, transforms them in registers and scatters them back.
// The last pass covers the lowest four index bits, so every work item ends with 16 adjacent
// outputs, which it scales, rounds, clamps and stores as one 16-byte word.  The LDS row is
// padded by 4 floats every 16 so that this 16-byte-per-lane pass is bank-conflict free.  The passes are
// in hadamard_row.h; the kernel of a whole generation stack runs them too.
#include <atomic>

#include "common.h"
#include "hadamard_row.h"

namespace quamba {
namespace {

// Outputs (any may be null): out = int8 codes of scale * y; out_f32 = y; out_f16 = fp16(scale * y).
// TR applies H_n^T = H_k^T (x) H_{2^m} (the Sylvester factor is symmetric).
template <int K, int LOGM, typename TIn, bool TR>
__global__ __launch_bounds__(threads_for(K << LOGM)) void hadamard_quant_kernel(const TIn *__restrict__ g, float inv_s,
                                                            int8_t *__restrict__ out,
                                                            float *__restrict__ out_f32,
                                                            __half *__restrict__ out_f16, int M, WarmLines warm) {
  if ((int)blockIdx.x >= M) {  // appended workgroups only read ahead
    warm_lines(warm, blockIdx.x - M);
    return;
  }
  constexpr int n = K << LOGM;
  constexpr int HT = threads_for(n);
  extern __shared__ __attribute__((aligned(16))) float row[];
  const size_t r = blockIdx.x;
  transform_row<K, LOGM, TIn, TR>(g + r * n, row);

  // last pass: bits [0, 4), fused with scale / round / clamp / pack
  for (int w = threadIdx.x; w < n / 16; w += HT) {
    float v[16];
    last_pass(row, w, v);
    if (out) {
      unsigned pk[4];
#pragma unroll
      for (int q = 0; q < 4; ++q)
        pk[q] = pack_q8x4(v[4 * q] * inv_s, v[4 * q + 1] * inv_s, v[4 * q + 2] * inv_s, v[4 * q + 3] * inv_s);
      *reinterpret_cast<uint4 *>(out + r * n + (size_t)w * 16) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
    }
    if (out_f32) {
      float *o = out_f32 + r * n + (size_t)w * 16;
#pragma unroll
      for (int q = 0; q < 4; ++q)
        reinterpret_cast<float4 *>(o)[q] = make_float4(v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]);
    }
    if (out_f16) {
      union {
        uint4 u[2];
        __half h[16];
      } o;
#pragma unroll
      for (int e = 0; e < 16; ++e) o.h[e] = __float2half_rn(v[e] * inv_s);
      uint4 *dst = reinterpret_cast<uint4 *>(out_f16 + r * n + (size_t)w * 16);
      dst[0] = o.u[0];
      dst[1] = o.u[1];
    }
  }
}

// Generation with up to three sequences: Hadamard + quantization + out_proj in one launch.  Two launches
// of a few microseconds each, almost all of it latency, become one: every workgroup owns one row and OC
// output columns, asks for its pieces of their weight rows first (one 16-byte piece per thread and column, n / 16
// threads rounded up to whole waves), transforms its row itself while they arrive (redundantly: the row is 10 KB
// and stays in the cache), and multiplies the 16 codes each thread ends up holding with exactly the
// weight pieces it asked for.  The codes and sums are the stand-alone kernels' bit for bit (same passes, same
// order); the workgroups of column group 0 also store them.  out[r, n] = fp16(acc[r, n] * m_out).
constexpr int OC = 16;  // output columns per workgroup (8: +2 %, 4: +3 %, 32: +12 % on the 64-block step)

template <int K, int LOGM>
__global__ __launch_bounds__(threads_for(K << LOGM)) void hadamard_out_proj_kernel(
    const __half *__restrict__ g, int M, float inv_s, const int8_t *__restrict__ W, int Dm, float m_out,
    __half *__restrict__ out, int8_t *__restrict__ codes_out) {
  constexpr int n = K << LOGM;
  constexpr int HT = threads_for(n);
  static_assert(HT >= n / 16, "one item per thread");
  extern __shared__ __attribute__((aligned(16))) float row[];
  __shared__ int red[HT / 64][OC];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // One workgroup per (row, column group).  Workgroups go to the 8 XCDs round-robin by index, so the
  // M workgroups of a column group are spaced 8 apart: same L2, launched together, one HBM read.
  const int ncg = gridDim.x / M, bid = blockIdx.x;
  int cg, r;
  if (ncg % 8 == 0) {
    const int slot = bid >> 3;
    r = slot % M;
    cg = (slot / M) * 8 + (bid & 7);
  } else {
    r = bid % M;
    cg = bid / M;
  }
  const int n0 = cg * OC;
  // n / 16 need not fill the last wave (1536 = 96 items, 2560 = 160): its other threads repeat the last item with zero codes
  const bool live = HT == n / 16 || tid < n / 16;
  const int item = live ? tid : n / 16 - 1;
  v4i wv[OC];
#pragma unroll
  for (int j = 0; j < OC; ++j)  // the clamp only bounds the address of a ragged last group
    wv[j] = *reinterpret_cast<const v4i *>(W + (size_t)min(n0 + j, Dm - 1) * n + (size_t)item * 16);
  transform_row<K, LOGM, __half, false>(g + (size_t)r * n, row);
  float v[16];
  last_pass(row, item, v);
  v4i c;
#pragma unroll
  for (int q = 0; q < 4; ++q)
    c[q] = static_cast<int>(pack_q8x4(v[4 * q] * inv_s, v[4 * q + 1] * inv_s, v[4 * q + 2] * inv_s, v[4 * q + 3] * inv_s));
  if (!live) c = v4i{0, 0, 0, 0};
  if (cg == 0 && codes_out && live) *reinterpret_cast<v4i *>(codes_out + (size_t)r * n + (size_t)tid * 16) = c;
#pragma unroll
  for (int j = 0; j < OC; ++j) {
    int acc = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_sdot4(c[e], wv[j][e], acc, false);
    acc = wave_sum(acc);
    if (lane == 0) red[wave][j] = acc;
  }
  __syncthreads();
  if (tid < OC && n0 + tid < Dm) {
    int a = 0;
#pragma unroll
    for (int w = 0; w < HT / 64; ++w) a += red[w][tid];
    float y = static_cast<float>(a) * m_out;
    // Left alone, the compiler folds product and conversion into one instruction with one rounding (v_fma_mixlo_f16), which
    // differs from the separate kernels' fp32 product where that lands halfway between two halves (one output in 10^4).
    // 1536 and 2560 keep those kernels' bits; the other orders have been rounded once for as long as this launch serves them.
    if constexpr (HT != n / 16) asm volatile("" : "+v"(y));
    out[(size_t)r * Dm + n0 + tid] = __float2half_rn(y);
  }
}

template <int K, int LOGM, typename TIn, bool TR>
int run(const TIn *g, int M, float inv_s, int8_t *out, float *out_f32, __half *out_f16, hipStream_t st, ReadAhead ahead) {
  constexpr int n = K << LOGM;
  constexpr size_t lds = (size_t)(n + n / 4) * sizeof(float);
  if (lds > 64 * 1024) {  // the attribute is per device: one bit per device index
    static std::atomic<unsigned long long> attr_set{0};
    int dev = 0;
    QUAMBA_HIP(hipGetDevice(&dev));
    const unsigned long long bit = 1ull << (dev & 63);
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
      QUAMBA_HIP(hipFuncSetAttribute(reinterpret_cast<const void *>(&hadamard_quant_kernel<K, LOGM, TIn, TR>),
                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
      attr_set.fetch_or(bit, std::memory_order_release);
    }
  }
  const WarmLines warm = warm_lines_of(ahead.ptr, ahead.bytes);
  hipLaunchKernelGGL((hadamard_quant_kernel<K, LOGM, TIn, TR>), dim3(M + warm.blocks), dim3(threads_for(n)), lds, st, g, inv_s, out,
                     out_f32, out_f16, M, warm);
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}

template <int K, typename TIn, bool TR>
int dispatch_m(int m, const TIn *g, int M, float inv_s, int8_t *out, float *out_f32, __half *out_f16, hipStream_t st, ReadAhead ahead) {
  switch (m) {
#define QUAMBA_CASE(LM) \
  case LM:              \
    return run<K, LM, TIn, TR>(g, M, inv_s, out, out_f32, out_f16, st, ahead);
    QUAMBA_CASE(4)
    QUAMBA_CASE(5)
    QUAMBA_CASE(6)
    QUAMBA_CASE(7)
    QUAMBA_CASE(8)
    QUAMBA_CASE(9)
    QUAMBA_CASE(10)
    default:
      break;
  }
  if constexpr (K == 1) {
    switch (m) {
      QUAMBA_CASE(11)
      QUAMBA_CASE(12)
      QUAMBA_CASE(13)
      QUAMBA_CASE(14)
      default:
        break;
    }
  }
#undef QUAMBA_CASE
  return fail(QUAMBA_EUNSUPPORTED, "hadamard: order %d*2^%d is outside the supported range", K, m);
}

}  // namespace

bool hadamard_factor(int n, int *k, int *m) {
  if (n <= 0) return false;
  int odd = n, p = 0;
  while ((odd & 1) == 0) {
    odd >>= 1;
    ++p;
  }
  if (odd == 1) {
    *k = 1;
    *m = p;
    return true;
  }
  if ((odd == 3 || odd == 5) && p >= 2) {
    *k = odd * 4;
    *m = p - 2;
    return true;
  }
  return false;
}

namespace {
template <typename TIn, bool TR>
int dispatch_k(const TIn *g, int M, int n, float inv_s_y, int8_t *yH_q, float *yH_f32, __half *y_f16, hipStream_t st,
               ReadAhead ahead = {}) {
  int k = 0, m = 0;
  if (!hadamard_factor(n, &k, &m) || m < 4)
    return fail(QUAMBA_EUNSUPPORTED, "hadamard: n=%d is not k*2^m with k in (1,12,20) and m >= 4", n);
  if (M == 0) return QUAMBA_OK;
  switch (k) {
    case 1:
      return dispatch_m<1, TIn, false>(m, g, M, inv_s_y, yH_q, yH_f32, y_f16, st, ahead);  // H_{2^m} is symmetric
    case 12:
      return dispatch_m<12, TIn, TR>(m, g, M, inv_s_y, yH_q, yH_f32, y_f16, st, ahead);
    default:
      return dispatch_m<20, TIn, TR>(m, g, M, inv_s_y, yH_q, yH_f32, y_f16, st, ahead);
  }
}
}  // namespace

int launch_hadamard_quant(const __half *g, int M, int n, float inv_s_y, int8_t *yH_q, float *yH_f32,
                          hipStream_t st, ReadAhead ahead) {
  return dispatch_k<__half, false>(g, M, n, inv_s_y, yH_q, yH_f32, nullptr, st, ahead);
}

namespace {
template <int K, int LOGM>
int run_out_proj(const __half *g, int M, float inv_s, const int8_t *W, int Dm, float m_out, __half *out, int8_t *codes,
                 hipStream_t st) {
  constexpr int n = K << LOGM;
  constexpr size_t lds = (size_t)(n + n / 4) * sizeof(float);
  static_assert(lds <= 64 * 1024, "fits the default dynamic LDS limit");
  hipLaunchKernelGGL((hadamard_out_proj_kernel<K, LOGM>), dim3((Dm + OC - 1) / OC * M), dim3(threads_for(n)), lds, st, g, M,
                     inv_s, W, Dm, m_out, out, codes);
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}
}  // namespace

// orders for which one thread per 16 elements is a whole wave or more and the row fits 64 KB of LDS: 1024 to 8192, 1536 to 12288
// and 2560 to 10240, each by powers of two.  The step of a narrow layer is bound by its launches: with three sequences (20 launches
// in a graph, us each) 1536 wide 19.9 -> 17.5, 2560 wide 21.8 -> 18.6; with one or two, quantization in in_proj's launch
// included, 16.2 -> 14.0 and 18.5 -> 15.0, 16.2 -> 13.9 and 18.8 -> 15.2
bool hadamard_fuses_out_proj(int n, int Dm) {
  int k = 0, m = 0;
  if (Dm < 1 || !hadamard_factor(n, &k, &m)) return false;
  return (k == 1 && m >= 10 && m <= 13) || (k == 12 && m >= 7 && m <= 10) || (k == 20 && m >= 7 && m <= 9);
}

// M rows (a few: with four the separate kernels are faster, and two rows per workgroup, the transforms one
// after the other, cost 5-9 us more than they save): out[r, 0..Dm) = fp16(m_out * W codes(H_n g[r])), codes as launch_hadamard_quant's (stored to codes if given)
int launch_hadamard_out_proj(const __half *g, int M, int n, float inv_s_y, const int8_t *W, int Dm, float m_out,
                             __half *out, int8_t *codes, hipStream_t st) {
  if (M < 1 || M > 64) return fail(QUAMBA_EINVAL, "hadamard + out_proj: M=%d", M);
  if (!hadamard_fuses_out_proj(n, Dm)) return fail(QUAMBA_EUNSUPPORTED, "hadamard + out_proj: n=%d Dm=%d", n, Dm);
  int k = 0, m = 0;
  hadamard_factor(n, &k, &m);
#define QUAMBA_CASE(KK, LM) \
  if (k == KK && m == LM) return run_out_proj<KK, LM>(g, M, inv_s_y, W, Dm, m_out, out, codes, st);
  QUAMBA_CASE(1, 10) QUAMBA_CASE(1, 11) QUAMBA_CASE(1, 12) QUAMBA_CASE(1, 13)
  QUAMBA_CASE(12, 7) QUAMBA_CASE(12, 8) QUAMBA_CASE(12, 9) QUAMBA_CASE(12, 10)
  QUAMBA_CASE(20, 7) QUAMBA_CASE(20, 8) QUAMBA_CASE(20, 9)
#undef QUAMBA_CASE
  return fail(QUAMBA_EUNSUPPORTED, "hadamard + out_proj: n=%d", n);
}

// fp32 rows in, fp32 rows out, no quantization (used by calibration)
int launch_hadamard_f32(const float *x, int M, int n, float *y, hipStream_t st) {
  return dispatch_k<float, false>(x, M, n, 1.f, nullptr, y, nullptr, st);
}

// Backward transform of quantized codes (Appendix H, the comparison variant's scan input):
// x_hat = fp16(scale * H_n^T xH_q).  The integer sums are exact in fp32 for n * 128 < 2^24.
int launch_hadamard_inverse(const int8_t *xH_q, int M, int n, float scale, __half *x_hat, hipStream_t st) {
  return dispatch_k<int8_t, true>(xH_q, M, n, scale, nullptr, nullptr, x_hat, st);
}

}  // namespace quamba
