// Device side of the fused Hadamard transform (its layout and passes are described in hadamard.hip): one token row in LDS,
// transformed by the HT threads of a workgroup.
#pragma once

#include "device_util.h"

namespace quamba {
namespace {

// Threads per row: one per 16 elements (every pass then gives each thread one work item), in
// whole waves, at most 1024.
constexpr int threads_for(int n) { return n / 16 >= 1024 ? 1024 : (n / 16 + 63) / 64 * 64; }

struct WholeGroup {  // the barrier between passes where every thread of the workgroup takes part
  __device__ __forceinline__ void operator()() const { __syncthreads(); }
};

__device__ __forceinline__ int pad(int i) { return i + ((i >> 4) << 2); }

// Sign pattern of the Paley-I Hadamard matrix of order Q+1, Q prime, Q = 3 (mod 4):
// H = I + S, S[0][j] = +1, S[i][0] = -1, S[i+1][j+1] = chi(i - j) (Legendre symbol mod Q).
// neg[a] has bit b set when H[a][b] = -1.
template <int Q>
struct Paley {
  unsigned neg[Q + 1];
  constexpr Paley() : neg{} {
    bool residue[Q] = {};
    for (int i = 1; i < Q; ++i) residue[(i * i) % Q] = true;
    for (int a = 0; a <= Q; ++a) {
      unsigned bits = 0;
      for (int b = 0; b <= Q; ++b) {
        bool minus = false;
        if (a == 0) {
          minus = false;
        } else if (b == 0) {
          minus = true;
        } else if (a != b) {
          const int diff = ((a - 1) - (b - 1) + Q) % Q;
          minus = !residue[diff];
        }
        if (minus) bits |= 1u << b;
      }
      neg[a] = bits;
    }
  }
};

// H_k as fp16 bit patterns (+1 = 0x3C00, -1 = 0xBC00), zero-padded to 32 x 32: the A operand of
// the MFMA form, read 16 bytes per lane.
// TR: the table of H_k^T (the Paley matrices are not symmetric; the backward transform needs it).
template <int K, bool TR>
struct PaleyHalf {
  uint16_t h[32][32];
  constexpr PaleyHalf() : h{} {
    constexpr Paley<K - 1> tab{};
    for (int a = 0; a < K; ++a)
      for (int b = 0; b < K; ++b) {
        const bool minus = TR ? ((tab.neg[b] >> a) & 1u) : ((tab.neg[a] >> b) & 1u);
        h[a][b] = minus ? 0xBC00 : 0x3C00;
      }
  }
};
template <int K, bool TR>
__device__ const PaleyHalf<K, TR> g_paley_half{};

template <int K, int HT, bool TR, typename Sync>
__device__ __forceinline__ void order_k_pass(float *row, int logm, int tid, const Sync &sync) {
  if constexpr (K > 1) {
    constexpr Paley<K - 1> tab{};
    const int items = 1 << logm;
    for (int w = tid; w < items; w += HT) {
      float v[K], o[K];
#pragma unroll
      for (int a = 0; a < K; ++a) v[a] = row[pad((a << logm) | w)];
#pragma unroll
      for (int a = 0; a < K; ++a) {
        float s = 0.f;
#pragma unroll
        for (int b = 0; b < K; ++b) s += (TR ? ((tab.neg[b] >> a) & 1u) : ((tab.neg[a] >> b) & 1u)) ? -v[b] : v[b];
        o[a] = s;
      }
#pragma unroll
      for (int a = 0; a < K; ++a) row[pad((a << logm) | w)] = o[a];
    }
    sync();
  }
}

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// fp16 row in global memory -> order-k transform -> fp32 row in LDS (padded layout), using
// v_mfma_f32_32x32x16_f16.  The row is first staged as fp16 [K][2^LOGM + 8] in the same LDS
// bytes (the pitch keeps the two half-waves of a fragment read on different banks).  Operand
// element e of lane l at k step s is b = 16 s + 8 (l / 32) + e for both operands: H_k[l % 32, b]
// on the A side, x[b, 32 t + l % 32] on the B side; register r of the result is row
// a = 8 (r / 4) + 4 (l / 32) + r % 4, column 32 t + l % 32.
// int8 input (the backward transform of quantized codes) is widened to fp16 while staging, which is exact.
template <int K, int LOGM>
__device__ __forceinline__ _Float16 *half_slot(float *row, int i) {  // where element i of the row (i % 8 == 0) is staged
  constexpr int W = 1 << LOGM, PITCH = W + 8;
  return reinterpret_cast<_Float16 *>(row) + (i >> LOGM) * PITCH + (i & (W - 1));
}

// a lane's operands of H_k
struct OrderK {
  h8 f[2];
};
template <int K, bool TR>
__device__ __forceinline__ OrderK order_k_operands(int lane) {
  OrderK r;
#pragma unroll
  for (int s = 0; s < 2; ++s) r.f[s] = *reinterpret_cast<const h8 *>(&g_paley_half<K, TR>.h[lane & 31][16 * s + 8 * (lane >> 5)]);
  return r;
}

// the staged row -> its order-k transform, fp32 (the threads' own staging stores come first)
template <int K, int LOGM, int HT, typename Sync>
__device__ __forceinline__ void order_k_mfma(float *row, int tid, const OrderK &hk, const Sync &sync) {
  static_assert(K > 1 && K <= 32 && LOGM >= 5, "one 32-row tile of H_k, whole 32-column tiles");
  constexpr int W = 1 << LOGM, PITCH = W + 8;
  // Addresses: one per tile, everything else a constant offset from it (LDS pitches are linear in the row).  Formed one by one they were
  // half of this pass's instructions: the Hadamard + out_proj part of the 64-block step with one sequence takes 0.4 us less a block.
  constexpr int PADDED = W + W / 4;  // floats of one row a in the padded layout
  const _Float16 *hx = reinterpret_cast<const _Float16 *>(row);
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int a = lane & 31, upper = lane >> 5;
  sync();
  constexpr int NWAVE = HT / 64, TILES = W / 32, TPW = (TILES + NWAVE - 1) / NWAVE;  // column tiles, per wave
  f32x16 acc[TPW];
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int t = wave + NWAVE * q;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[q][r] = 0.f;
    if (t < TILES) {
      const _Float16 *col = hx + upper * (8 * PITCH) + 32 * t + a;
#pragma unroll
      for (int s = 0; s < 2; ++s) {
        if (16 * s >= K) continue;
        h8 hb;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // rows b = 16 s + 8 upper + e past K are zero; those of the upper lanes alone are read from row 16 s + e instead
          _Float16 v = static_cast<_Float16>(0.f);
          if (16 * s + 8 + e < K) v = col[(16 * s + e) * PITCH];
          else if (16 * s + e < K) v = upper ? static_cast<_Float16>(0.f) : col[(16 * s + e) * PITCH - upper * (8 * PITCH)];
          hb[e] = v;
        }
        acc[q] = __builtin_amdgcn_mfma_f32_32x32x16_f16(hk.f[s], hb, acc[q], 0, 0, 0);
      }
    }
  }
  sync();  // every fragment is in registers: the fp16 staging may be overwritten
#pragma unroll
  for (int q = 0; q < TPW; ++q) {
    const int t = wave + NWAVE * q;
    if (t < TILES) {
      float *col = row + upper * (4 * PADDED) + pad(32 * t + a);
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const int oa = 8 * (r >> 2) + (r & 3);  // + 4 upper
        if (oa + 4 < K) col[oa * PADDED] = acc[q][r];
        else if (oa < K && !upper) col[oa * PADDED] = acc[q][r];
      }
    }
  }
  sync();
}

template <int K, int LOGM, int HT, typename TIn, bool TR>
__device__ __forceinline__ void order_k_load_mfma(const TIn *__restrict__ src, float *row) {
  static_assert(sizeof(TIn) <= 2, "fp16 or int8 rows");
  constexpr int n = K << LOGM;
  for (int i = threadIdx.x * 8; i < n; i += HT * 8) {
    uint4 *dst = reinterpret_cast<uint4 *>(half_slot<K, LOGM>(row, i));
    if constexpr (sizeof(TIn) == 2) {
      *dst = *reinterpret_cast<const uint4 *>(src + i);
    } else {
      const uint2 in = *reinterpret_cast<const uint2 *>(src + i);
      union {
        uint4 u;
        _Float16 h[8];
      } w;
#pragma unroll
      for (int e = 0; e < 8; ++e)
        w.h[e] = static_cast<_Float16>(static_cast<int>(static_cast<int8_t>((e < 4 ? in.x : in.y) >> (8 * (e & 3)))));
      *dst = w.u;
    }
  }
  order_k_mfma<K, LOGM, HT>(row, threadIdx.x, order_k_operands<K, TR>(threadIdx.x & 63), WholeGroup{});
}

template <int R>
__device__ __forceinline__ void butterflies(float (&v)[1 << R]) {
#pragma unroll
  for (int len = 1; len < (1 << R); len <<= 1)
#pragma unroll
    for (int i = 0; i < (1 << R); ++i)
      if ((i & len) == 0) {
        const float a = v[i], b = v[i + len];
        v[i] = a + b;
        v[i + len] = a - b;
      }
}

// Butterflies over index bits [s, s+R) of the whole row.
template <int R, int HT, typename Sync>
__device__ __forceinline__ void radix_pass(float *row, int n, int s, int tid, const Sync &sync) {
  if constexpr (R > 0) {
    const int items = n >> R;
    for (int w = tid; w < items; w += HT) {
      const int low = w & ((1 << s) - 1);
      const int base = ((w >> s) << (s + R)) | low;
      float v[1 << R];
#pragma unroll
      for (int j = 0; j < (1 << R); ++j) v[j] = row[pad(base + (j << s))];
      butterflies<R>(v);
#pragma unroll
      for (int j = 0; j < (1 << R); ++j) row[pad(base + (j << s))] = v[j];
    }
    sync();
  }
}

// index bits [4, LOGM) in up to three passes of at most 5 bits, high bits first; ends with a barrier where there is a pass
template <int K, int LOGM, int HT, typename Sync>
__device__ __forceinline__ void high_passes(float *row, int tid, const Sync &sync) {
  constexpr int n = K << LOGM;
  constexpr int HI = LOGM - 4;
  constexpr int NP = (HI + 4) / 5;
  constexpr int R0 = NP > 0 ? (HI + NP - 1) / NP : 0;
  constexpr int R1 = NP > 1 ? (HI - R0 + NP - 2) / (NP - 1) : 0;
  constexpr int R2 = NP > 2 ? HI - R0 - R1 : 0;
  static_assert(R0 + R1 + R2 == HI && NP <= 3, "pass schedule");
  radix_pass<R0, HT>(row, n, LOGM - R0, tid, sync);
  radix_pass<R1, HT>(row, n, LOGM - R0 - R1, tid, sync);
  radix_pass<R2, HT>(row, n, 4, tid, sync);
}

// One row of n = K 2^LOGM values from global memory through every pass but the last, left in LDS
// (padded fp32 layout); ends with a barrier.
template <int K, int LOGM, typename TIn, bool TR>
__device__ __forceinline__ void transform_row(const TIn *__restrict__ src, float *row) {
  static_assert(LOGM >= 4, "the last pass owns the low four index bits");
  constexpr int n = K << LOGM;
  constexpr int HT = threads_for(n);
  if constexpr (sizeof(TIn) <= 2 && K > 1 && LOGM >= 5) {
    order_k_load_mfma<K, LOGM, HT, TIn, TR>(src, row);
  } else {
    for (int i = threadIdx.x * 8; i < n; i += HT * 8) {
      float *dst = row + pad(i);
      if constexpr (sizeof(TIn) == 2) {
        union {
          uint4 u;
          __half h[8];
        } in;
        in.u = *reinterpret_cast<const uint4 *>(src + i);
        *reinterpret_cast<float4 *>(dst) = make_float4(__half2float(in.h[0]), __half2float(in.h[1]),
                                                       __half2float(in.h[2]), __half2float(in.h[3]));
        *reinterpret_cast<float4 *>(dst + 4) = make_float4(__half2float(in.h[4]), __half2float(in.h[5]),
                                                           __half2float(in.h[6]), __half2float(in.h[7]));
      } else if constexpr (sizeof(TIn) == 1) {
        const uint2 in = *reinterpret_cast<const uint2 *>(src + i);
#pragma unroll
        for (int e = 0; e < 8; ++e)
          dst[e] = static_cast<float>(static_cast<int>(static_cast<int8_t>((e < 4 ? in.x : in.y) >> (8 * (e & 3)))));
      } else {
        *reinterpret_cast<float4 *>(dst) = *reinterpret_cast<const float4 *>(src + i);
        *reinterpret_cast<float4 *>(dst + 4) = *reinterpret_cast<const float4 *>(src + i + 4);
      }
    }
    __syncthreads();
    order_k_pass<K, HT, TR>(row, LOGM, threadIdx.x, WholeGroup{});
  }

  high_passes<K, LOGM, HT>(row, threadIdx.x, WholeGroup{});
}

// last pass of item w: bits [0, 4) of elements [16 w, 16 w + 16)
__device__ __forceinline__ void last_pass(const float *row, int w, float (&v)[16]) {
  const float *p = row + pad(w * 16);
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const float4 f = reinterpret_cast<const float4 *>(p)[q];
    v[4 * q] = f.x;
    v[4 * q + 1] = f.y;
    v[4 * q + 2] = f.z;
    v[4 * q + 3] = f.w;
  }
  butterflies<4>(v);
}

}  // namespace
}  // namespace quamba
