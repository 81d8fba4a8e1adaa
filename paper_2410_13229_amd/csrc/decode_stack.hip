// Generation with one or two sequences: the whole stack of blocks in one launch.
//
// A block of such a step is a chain of four small products (A in_proj + conv step, B x_proj, C scan step with dt_proj, D Hadamard +
// out_proj), each of which needs all of the one before.  As four launches a block, the 64-block step of the 2.8B model
// spends most of its time on launch boundaries and on the first reads of cold weights behind them.  Here one workgroup per CU
// stays for all blocks; eight of its waves have role A (40 columns of in_proj), five role D (10 columns of out_proj), three B or C,
// and each role walks the blocks at its own pace.  A wave asks for its weights of the next block as soon as it is done with the last
// (8 x 15 and 5 x 10 rows of 1 KB, held in registers; with two sequences 18 to 26 registers a lane go to scratch) and then waits for its
// input, so the 40 MB of a block stream in
// under the other roles, and a hand-over costs one trip through the memory side (1.2 to 2 us among 256 workgroups) instead of
// a launch boundary plus the first cold read.  64 blocks of the 2.8B layer: one sequence 1643 -> 1051 us a step, two 1939 -> 1605.  Bound by the
// chain: of 15.4 us a block (one sequence) the four hand-overs take 1.2 to 2.4 each, norm + in_proj + conv 2.0, x_proj 1.0, the scan step 0.6,
// Hadamard + out_proj 3.6 (with two sequences one transform after the other), the spread of the workgroups the rest; the weights are there 9 us early.
//
// The launch takes the CUs for the whole step (all 256 at 2560 x 5120, 77 at 768 x 1536; 16 waves of 128 registers fill one), so
// several users on streams of their own share it only where it leaves CUs: 768 x 1536, one sequence each, one / two / four users 425 / 680 / 1323 us
// launch by launch, 268 / 278 / 564 this way; 2560 x 5120, 64 blocks 1637 / 2073 / 3919 and 1050 / 2270 / 4499, two sequences each 1938 / 2424 /
// 3779 and 1605 / 3190 / 6195.
//
// Hand-over: every 4 bytes of payload (four codes, or two halves) travel in one 8-byte word with a tag, the number of the block
// plus one, written and read by relaxed 64-bit atomics at device scope.  A reader that sees its tag has the payload, so no
// fence (which would write back or drop a whole L2) and no flag is needed.  One buffer per kind of value serves all blocks: a word is
// overwritten for block l + 1 only by a workgroup whose input needs, through the chain, every reader of block l's word to be done.
// How the words lie and are polled decides the speed (the same step 1750 us with every wave polling all its words in lines shared by neighbours): a
// workgroup's words fill lines of their own, readers take whole lines through LDS, and until the first word is there one wave per role
// watches it alone.
//
// Progress does not depend on how many workgroups run at once.  At its start every workgroup signs in; if all of them
// do so within a bounded time they are all resident, and each keeps its own items (the walk above).  If not (another
// kernel holds part of the GPU), the ones that run take the items from a counter, in an order in which an item only waits for
// items with lower numbers, which somebody already holds: any number of workgroups gets through (all resident, that form
// takes 1200 us).  Every wait is bounded (WAIT_TRIES polls, 35 ms and more where no wait of a step that runs takes one); a role's waves that have given up
// hand nothing on any more, so everything behind them gives up as well, down to the outputs, which are NaN.
//
// Arithmetic, operand order and rounding are those of the separate kernels (decode_in_kernel, gemv_i8_kernel, scan_step_kernel,
// hadamard_out_proj_kernel): same bits.
#include <algorithm>
#include <atomic>

#include "common.h"
#include "hadamard_row.h"

namespace quamba {

// 0: on where it is served, 1: off, 2: on, with the work items taken from the counter, 3: on, the first block's input never handed over
std::atomic<int> g_decode_stack_hook{0};

namespace {

typedef unsigned long long u64;
constexpr float LOG2E = 1.44269504088896340736f;
constexpr float LN2 = 0.69314718055994530942f;
constexpr int NS = 16;
constexpr int AC = 5;          // in_proj columns per wave
constexpr int PF = 3;          // rounds of 64 16-byte pieces that cover d_model
// Measured at 64 blocks of the 2.8B layer, one sequence: 3 weight loads in flight per wave 1049 us, 2 1065, 5 1090, all at once 1105; a
// pause of 4 in front of a repeated poll 1049, 1 1056, none 1062 (units of 64 clocks)
constexpr int LOADS_IN_FLIGHT = 3, FRONT_PACE = 20, PACE = 4, RETRY_PACE = 2;
constexpr int WAIT_TRIES = 1 << 18;
constexpr int SIGN_IN_TRIES = 64;

// A workgroup is one per CU, 16 waves: 8 for role A, 5 for D, 3 for B or C (the first workgroups B, the others C).
constexpr int A_WAVES = 8, D_WAVES = 5, BC_WAVES = 3;
constexpr int STACK_THREADS = 64 * (A_WAVES + D_WAVES + BC_WAVES);
constexpr int A_COLS = A_WAVES * AC;  // in_proj columns per workgroup: whole groups of four
constexpr int D_COLS = 10;            // out_proj columns per workgroup
constexpr int D_THREADS = 64 * D_WAVES, BC_THREADS = 64 * BC_WAVES;
static_assert(A_COLS % 4 == 0 && D_COLS % 2 == 0 && A_COLS / 4 <= 16 && D_COLS <= 16 && BC_THREADS / 4 <= 64, "codes leave in fours, halves in pairs");

// What the kernel needs of one block; written to device memory by stack_begin_kernel.
struct StackLayer {
  const int8_t *W_in, *conv_w, *W_x, *W_dt, *A, *D, *W_outH;
  const float *conv_b, *dt_bias;
  const __half *norm_w;
  float inv_s_u, m_in_x, m_in_z, s_cw, s_xpre, inv_s_x, m_x_dt, m_x_B, m_x_C, m_dt;
  float s_x, s_dt, s_z, s_B, s_C, s_A, s_D, inv_s_y, m_out, pad;
};
constexpr int CHUNK_LAYERS = 22;  // descriptors handed over by value in one launch: 3.5 KB of kernel arguments
struct LayerChunk {
  StackLayer layer[CHUNK_LAYERS];
};

struct Words {  // tagged words, [M] rows each: residual stream, x codes, z codes, x_proj codes, gated scan output
  u64 *s, *x, *z, *dbc, *g;
  unsigned *ctrl;  // control words, one per 256 bytes
};
constexpr int CTRL_STRIDE = 64, CTRL_WORDS = 12;
enum { C_SUB = 0 /* 8 sign-in counters */, C_TOP = 8, C_MODE = 9, C_TICKET = 10, C_GAVE_UP = 11 };

struct StackArgs {
  const StackLayer *layers;
  int n_layers, Dm, Di, R;
  float eps;
  float *ssm;
  __half *conv;
  Words w;
  __half *out, *res;  // of the last block, for the final norm
  int nA, nB, nC, nD;
  int x_row, g_row;  // words of one row of x or z, of the gated output
  int from_counter;
};

__device__ __forceinline__ u64 word_load(const u64 *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void word_store(u64 *p, unsigned payload, unsigned tag) {
  __hip_atomic_store(p, (static_cast<u64>(tag) << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ unsigned ctrl_load(const unsigned *p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// A block's descriptor through scalar loads, its pointers as global ones (as generic ones every weight load would also count
// as an LDS access).
typedef __attribute__((address_space(4))) const StackLayer *LayerRef;
__device__ __forceinline__ LayerRef layer_ref(const StackLayer *layers, int l) { return (LayerRef)(layers + l); }
template <typename T>
__device__ __forceinline__ T gload(const void *p) {
  return *(__attribute__((address_space(1))) const T *)p;
}
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Where a word lies.  What one workgroup hands over is in 128-byte lines of its own: a line is written at one moment, so readers that have
// polled it do not have to fetch it again for every neighbour's store.
constexpr int LINE = 16;  // words
__device__ __host__ __forceinline__ int quad_at(int quad) { return quad / (A_COLS / 4) * LINE + quad % (A_COLS / 4); }  // codes of x or z: four columns
__device__ __host__ __forceinline__ int pair_at(int row, int pair) {  // residual stream: two columns
  return pair / (D_COLS / 2) * LINE + row * (D_COLS / 2) + pair % (D_COLS / 2);
}
__device__ __host__ __forceinline__ int gate_at(int d) {  // gated output: channels d, d + 1
  return d / (BC_THREADS / 4) * (2 * LINE) + d % (BC_THREADS / 4) / 2;
}
__device__ __host__ __forceinline__ int dbc_at(int row, int quad) { return quad * LINE + row; }  // x_proj codes: four columns

// The words watched by wait_ahead, spread over the workgroups: item idx of a role first watches a word of the role in front, then one that it awaits.
__device__ __host__ __forceinline__ int in_front(int idx, int nC) { return idx % nC * (2 * LINE); }         // g of the block before
__device__ __host__ __forceinline__ int in_watch(int idx, int nD) { return idx * 37 % nD * LINE; }          // s
__device__ __host__ __forceinline__ int x_front(int idx, int nD) { return idx % nD * LINE; }                // s
__device__ __host__ __forceinline__ int x_watch(int idx, int n) { return quad_at(idx * 37 % (n / 4)); }     // x
__device__ __host__ __forceinline__ int scan_front(int idx) { return quad_at(idx); }                        // x
__device__ __host__ __forceinline__ int scan_watch(int idx, int nB) { return idx % nB * LINE; }             // dbc
__device__ __host__ __forceinline__ int out_front(int idx, int nB) { return idx % nB * LINE; }              // dbc
__device__ __host__ __forceinline__ int out_watch(int idx, int nC) { return idx * 37 % nC * (2 * LINE); }   // g

// How long the waves of a role wait.  A thread that runs out of polls tells the others of its role (an LDS word that is never cleared; they see it behind their next
// barrier) and the control word that the selection of the token reads.  From the next item on the role (`gone`) polls once.
struct Patience {
  unsigned *ctrl, *role_gave_up;
  bool gone;
  __device__ __forceinline__ void give_up() const {
    __hip_atomic_store(ctrl + C_GAVE_UP * CTRL_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(role_gave_up, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
  }
  __device__ __forceinline__ bool gave_up() const { return __hip_atomic_load(role_gave_up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) != 0; }
};

// Polls base[idx[j]] until all N words carry `tag`; the payloads are left in v.
template <int N>
__device__ __forceinline__ void wait_words(const u64 *base, const int (&idx)[N], unsigned tag, unsigned (&v)[N], const Patience &patience) {
  for (int tries = 0;; ++tries) {
    u64 t[N];
#pragma unroll
    for (int j = 0; j < N; ++j) t[j] = word_load(base + idx[j]);
    bool ok = true;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      ok &= static_cast<unsigned>(t[j] >> 32) == tag;
      v[j] = static_cast<unsigned>(t[j]);
    }
    if (ok) break;
    if (patience.gone || tries >= WAIT_TRIES) {
      patience.give_up();
      break;
    }
    __builtin_amdgcn_s_sleep(RETRY_PACE);
  }
}

// Does this tag end a watch?  A later one does as well: nothing keeps the word in front from being overwritten before the watching wave has looked (a gated
// output of the block before may be, by channels whose z codes other columns form).
__device__ __host__ __forceinline__ bool watch_ends(unsigned tag, unsigned wanted) { return tag >= wanted; }

// What one wave of a role does for all of them before wait_words reads every word: it watches one of the awaited words, and before that,
// at a slow pace, one word of the role in front.  All words of all waiting workgroups polled all the time keep the memory
// side so busy that the stores they wait for hardly get through.
__device__ __forceinline__ void wait_ahead(const u64 *front, unsigned front_tag, const u64 *word, unsigned tag, const Patience &patience) {
  int tries = 0;
  if (front)
    for (; !watch_ends(static_cast<unsigned>(word_load(front) >> 32), front_tag) && !patience.gone && tries < WAIT_TRIES; ++tries) __builtin_amdgcn_s_sleep(FRONT_PACE);
  for (; !watch_ends(static_cast<unsigned>(word_load(word) >> 32), tag) && !patience.gone && tries < WAIT_TRIES; ++tries) __builtin_amdgcn_s_sleep(PACE);
}

// A scale read now: left to the compiler, the scalar load of a descriptor field lands where the value is needed, behind the waits.
__device__ __forceinline__ float now(float f) {
  asm volatile("" : "+s"(f));
  return f;
}

// Barrier among the waves of one role: each adds one to an LDS counter that is never reset and waits for its target.
struct RoleBarrier {
  unsigned *count;
  unsigned waves;
  mutable unsigned target;
  __device__ __forceinline__ void operator()() const {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    target += waves;
    if ((threadIdx.x & 63) == 0) __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    while (static_cast<int>(__hip_atomic_load(count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) - target) < 0) {
    }
    asm volatile("" ::: "memory");
  }
};

// Weight loads are kept a few in flight per wave: all at once they queue in front of the hand-overs.
__device__ __forceinline__ void throttle(int issued) {
  if (issued % LOADS_IN_FLIGHT == LOADS_IN_FLIGHT - 1) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// The thread and item index as values of this block only: hoisted out of the walk over the blocks, their addresses
// would take more registers than the weights.
__device__ __forceinline__ int fresh_tid(int first) {
  int t = static_cast<int>(threadIdx.x) - first;
  asm volatile("" : "+v"(t));
  return t;
}
__device__ __forceinline__ int fresh(int i) {
  asm volatile("" : "+s"(i));
  return i;
}

// Sum over the wave in the order of the shuffles lane ^ 32, ^ 16, ^ 8, ^ 4, ^ 2, ^ 1, without a trip through LDS for each.  After the first
// three steps lanes that agree modulo 8 hold the same value, so a rotation by 4 inside a row is lane ^ 4.
__device__ __forceinline__ float butterfly_sum(float v) {
  auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(both[0]) + __uint_as_float(both[1]);
  both = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(both[0]) + __uint_as_float(both[1]);
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, true));  // row_ror 8
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, true));  // row_ror 4
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x4E, 0xf, 0xf, true));   // quad_perm [2, 3, 0, 1]
  v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0xB1, 0xf, 0xf, true));   // quad_perm [1, 0, 3, 2]
  return v;
}

// Sums of N values per lane over the wave: lane j < N returns the sum of value j.
template <int N>
__device__ __forceinline__ int wave_sums(const int (&v)[N], int lane) {
  int t[N];
#pragma unroll
  for (int j = 0; j < N; ++j) t[j] = v[j] + __builtin_amdgcn_update_dpp(0, v[j], 0xB1, 0xf, 0xf, true);  // quad_perm [1, 0, 3, 2]
#pragma unroll
  for (int j = 0; j < N; ++j) t[j] += __builtin_amdgcn_update_dpp(0, t[j], 0x4E, 0xf, 0xf, true);  // quad_perm [2, 3, 0, 1]
#pragma unroll
  for (int j = 0; j < N; ++j) t[j] += __builtin_amdgcn_update_dpp(0, t[j], 0x141, 0xf, 0xf, true);  // row_half_mirror
#pragma unroll
  for (int j = 0; j < N; ++j) t[j] += __builtin_amdgcn_update_dpp(0, t[j], 0x140, 0xf, 0xf, true);  // row_mirror
  int mine = t[0];  // every lane of a row of 16 holds the row's sums
#pragma unroll
  for (int j = 1; j < N; ++j) mine = (lane & 15) == j ? t[j] : mine;
  auto both = __builtin_amdgcn_permlane16_swap(static_cast<unsigned>(mine), static_cast<unsigned>(mine), false, false);
  mine = static_cast<int>(both[0] + both[1]);
  both = __builtin_amdgcn_permlane32_swap(static_cast<unsigned>(mine), static_cast<unsigned>(mine), false, false);
  return static_cast<int>(both[0] + both[1]);
}

template <int MB>
struct InShared {
  __attribute__((aligned(16))) unsigned s[MB * PF * 512];
  float part[4][MB];
  int sums[MB][A_COLS];
};

// ---- role A: residual stream -> norm -> codes -> in_proj for A_COLS columns -> conv step on those of x
template <int MB>
__device__ __forceinline__ void role_in(const StackArgs &p, int l, int idx, int8_t *sA, InShared<MB> &sh, const RoleBarrier &sync,
                                        const Patience &patience) {
  const LayerRef q = layer_ref(p.layers, l);
  idx = fresh(idx);
  const int tid = fresh_tid(0), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int Dm = p.Dm, Di = p.Di, N = 2 * Di, nch = Dm / 16, groups = Dm / 8;
  const int n0 = idx * A_COLS + wave * AC;
  v4i w[PF][AC];
#pragma unroll
  for (int j = 0; j < AC; ++j)
#pragma unroll
    for (int r = 0; r < PF; ++r) {
      w[r][j] = gload<v4i>(q->W_in + (size_t)min(n0 + j, N - 1) * Dm + min(lane + 64 * r, nch - 1) * 16);
      throttle(j * PF + r);
    }
  // thread t of the first wave finishes columns 4 (t % quads) .. of row t / quads
  constexpr int quads = A_COLS / 4;
  const int fm = tid / quads, nq = idx * A_COLS + 4 * (tid % quads);
  const bool fin = tid < MB * quads && nq < N, fin_x = fin && nq < Di;
  v4u cw = {0u, 0u, 0u, 0u};
  v4f cb = {0.f, 0.f, 0.f, 0.f};
  ConvWindow4 win;
  win.u[0] = win.u[1] = win.u[2] = make_uint2(0u, 0u);
  uint2 *cs = reinterpret_cast<uint2 *>(p.conv + (((size_t)l * MB + (fin_x ? fm : 0)) * Di + (fin_x ? nq : 0)) * 3);
  if (fin_x) {
    cw = gload<v4u>(q->conv_w + (size_t)nq * 4);
    cb = gload<v4f>(q->conv_b + nq);
    win.u[0] = cs[0];
    win.u[1] = cs[1];
    win.u[2] = cs[2];
  }
  v4u nw[2] = {};
  if (wave < 4) {
#pragma unroll
    for (int it = 0; it < 2; ++it) nw[it] = gload<v4u>(q->norm_w + (size_t)min(tid + it * 256, groups - 1) * 8);
  }
  const float inv_s_u = now(q->inv_s_u), m_in_x = now(q->m_in_x), m_in_z = now(q->m_in_z), s_cw = now(q->s_cw), s_xpre = now(q->s_xpre),
              inv_s_x = now(q->inv_s_x);
  if (wave == 0) wait_ahead(l ? p.w.g + in_front(idx, p.nC) : nullptr, l, p.w.s + in_watch(idx, p.nD), l + 1, patience);
  sync();
  {  // the rows, as whole lines, into LDS
    constexpr int NWORD = (MB * PF * 512 + 64 * A_WAVES - 1) / (64 * A_WAVES);
    const int per_row = Dm / 2, words = MB * per_row;
    int at[NWORD];
    unsigned v[NWORD];
#pragma unroll
    for (int k = 0; k < NWORD; ++k) {
      const int i = min(tid + 64 * A_WAVES * k, words - 1);
      at[k] = pair_at(MB == 1 ? 0 : i / per_row, MB == 1 ? i : i % per_row);
    }
    wait_words(p.w.s, at, l + 1, v, patience);
#pragma unroll
    for (int k = 0; k < NWORD; ++k)
      if (tid + 64 * A_WAVES * k < words) sh.s[tid + 64 * A_WAVES * k] = v[k];
  }
  sync();
  // the first four waves own groups of 8 halves (tid, tid + 256) of every row (a scalar branch: each wave passes one of the barriers)
  if (wave < 4) {
    uint4 keep[MB][2];
    float ss[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      ss[m] = 0.f;
#pragma unroll
      for (int it = 0; it < 2; ++it) {
        if (tid + it * 256 < groups) {
          union {
            uint4 u;
            __half h[8];
          } r;
          r.u = *reinterpret_cast<const uint4 *>(sh.s + m * (Dm / 2) + (tid + it * 256) * 4);
          keep[m][it] = r.u;
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float f = __half2float(r.h[e]);
            ss[m] += f * f;
          }
        }
      }
    }
#pragma unroll
    for (int m = 0; m < MB; ++m) {
      const float t = butterfly_sum(ss[m]);
      if (lane == 0) sh.part[wave][m] = t;
    }
    sync();
    float rinv[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m)
      rinv[m] = 1.f / sqrtf((sh.part[0][m] + sh.part[1][m] + sh.part[2][m] + sh.part[3][m]) / static_cast<float>(Dm) + p.eps);
#pragma unroll
    for (int it = 0; it < 2; ++it) {
      const int g = tid + it * 256;
      if (g < groups) {
#pragma unroll
        for (int m = 0; m < MB; ++m) {
          union {
            uint4 u;
            __half h[8];
          } r, wv;
          r.u = keep[m][it];
          wv.u = make_uint4(nw[it][0], nw[it][1], nw[it][2], nw[it][3]);
          float v[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) v[e] = __half2float(r.h[e]) * rinv[m] * __half2float(wv.h[e]) * inv_s_u;
          *reinterpret_cast<uint2 *>(sA + (size_t)m * Dm + (size_t)g * 8) =
              make_uint2(pack_q8x4(v[0], v[1], v[2], v[3]), pack_q8x4(v[4], v[5], v[6], v[7]));
        }
      }
    }
  } else {
    sync();
  }
  sync();
  int acc[MB][AC];
#pragma unroll
  for (int m = 0; m < MB; ++m)
#pragma unroll
    for (int j = 0; j < AC; ++j) acc[m][j] = 0;
#pragma unroll
  for (int r = 0; r < PF; ++r)
    if (lane + 64 * r < nch) {
#pragma unroll
      for (int m = 0; m < MB; ++m) {
        const v4i a = *reinterpret_cast<const v4i *>(sA + (size_t)m * Dm + (lane + 64 * r) * 16);
#pragma unroll
        for (int j = 0; j < AC; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) acc[m][j] = __builtin_amdgcn_sdot4(a[e], w[r][j][e], acc[m][j], false);
      }
    }
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int mine = wave_sums<AC>(acc[m], lane);
    if (lane < AC) sh.sums[m][wave * AC + lane] = mine;
  }
  sync();
  if (fin && !patience.gave_up()) {
    int a4[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) a4[j] = sh.sums[fm][4 * (tid % quads) + j];
    if (fin_x) {
      const unsigned xpre = requant_pack4(a4, m_in_x);
      float sv[4];
      conv_step4_core(xpre, make_uint4(cw[0], cw[1], cw[2], cw[3]), make_float4(cb[0], cb[1], cb[2], cb[3]), win, s_cw, s_xpre, sv);
      word_store(p.w.x + fm * p.x_row + quad_at(nq / 4),
                 pack_q8x4(sv[0] * inv_s_x, sv[1] * inv_s_x, sv[2] * inv_s_x, sv[3] * inv_s_x), l + 1);
      cs[0] = win.u[0];
      cs[1] = win.u[1];
      cs[2] = win.u[2];
    } else {
      word_store(p.w.z + fm * p.x_row + quad_at((nq - Di) / 4), requant_pack4(a4, m_in_z), l + 1);
    }
  }
}

// ---- role B: x_proj for four columns; the threads split K in 16-byte pieces
template <int n, int MB>
__device__ __forceinline__ void role_x(const StackArgs &p, int l, int idx, int8_t *sx, int (*red)[MB * 4], const RoleBarrier &sync, const Patience &patience) {
  const LayerRef q = layer_ref(p.layers, l);
  idx = fresh(idx);
  const int tid = fresh_tid(64 * (A_WAVES + D_WAVES)), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int nch = n / 16, ROUNDS = (nch + BC_THREADS - 1) / BC_THREADS;
  const int n0 = idx * 4;
  v4i w[ROUNDS][4];
#pragma unroll
  for (int r = 0; r < ROUNDS; ++r)
#pragma unroll
    for (int j = 0; j < 4; ++j) w[r][j] = gload<v4i>(q->W_x + (size_t)(n0 + j) * n + min(tid + BC_THREADS * r, nch - 1) * 16);
  const float m_x = now(n0 < p.R ? q->m_x_dt : (n0 < p.R + NS ? q->m_x_B : q->m_x_C));
  if (wave == 0) wait_ahead(p.w.s + x_front(idx, p.nD), l + 1, p.w.x + x_watch(idx, n), l + 1, patience);
  sync();
  constexpr int NWORD = (n / 4 + BC_THREADS - 1) / BC_THREADS;
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    int at[NWORD];
    unsigned v[NWORD];
#pragma unroll
    for (int k = 0; k < NWORD; ++k) at[k] = m * p.x_row + quad_at(min(tid + BC_THREADS * k, n / 4 - 1));
    wait_words(p.w.x, at, l + 1, v, patience);
#pragma unroll
    for (int k = 0; k < NWORD; ++k)
      if (tid + BC_THREADS * k < n / 4) reinterpret_cast<unsigned *>(sx)[m * (n / 4) + tid + BC_THREADS * k] = v[k];
  }
  sync();
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    v4i a[ROUNDS];
#pragma unroll
    for (int r = 0; r < ROUNDS; ++r) a[r] = *reinterpret_cast<const v4i *>(sx + m * n + min(tid + BC_THREADS * r, nch - 1) * 16);
    int dots[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      dots[j] = 0;
#pragma unroll
      for (int r = 0; r < ROUNDS; ++r)
        if (tid + BC_THREADS * r < nch) {
#pragma unroll
          for (int e = 0; e < 4; ++e) dots[j] = __builtin_amdgcn_sdot4(a[r][e], w[r][j][e], dots[j], false);
        }
    }
    const int mine = wave_sums<4>(dots, lane);
    if (lane < 4) red[wave][m * 4 + lane] = mine;
  }
  sync();
  if (tid < MB && !patience.gave_up()) {
    int a[4] = {0, 0, 0, 0};
#pragma unroll
    for (int wv = 0; wv < BC_WAVES; ++wv)
#pragma unroll
      for (int j = 0; j < 4; ++j) a[j] += red[wv][tid * 4 + j];
    word_store(p.w.dbc + dbc_at(tid, idx), requant_pack4(a, m_x), l + 1);
  }
}

// softplus and gate as the scan kernels form them
__device__ __forceinline__ float softplus_f(float v) {
  const float e = __builtin_amdgcn_exp2f(-fabsf(v) * LOG2E);
  const float w = 1.f + e;
  const float c = (w - 1.f) - e;
  return fmaxf(v, 0.f) + __builtin_fmaf(__builtin_amdgcn_logf(w), LN2, -c);
}
__device__ __forceinline__ float silu_gate(float y, float z) {
  return y * z * __builtin_amdgcn_rcpf(1.f + __builtin_amdgcn_exp2f(-z * LOG2E));
}

// ---- role C: one step of the scan with dt_proj inside, four lanes per channel, which walk the sequences
template <int Di, int MB>
__device__ __forceinline__ void role_scan(const StackArgs &p, int l, int idx, int8_t *sdbc, const RoleBarrier &sync, const Patience &patience) {
  const LayerRef q = layer_ref(p.layers, l);
  idx = fresh(idx);
  const int tid = fresh_tid(64 * (A_WAVES + D_WAVES));
  const int R = p.R, NX = R + 2 * NS;
  const int gid = idx * BC_THREADS + tid;
  const bool live = gid < Di * 4;
  const int id = live ? gid : Di * 4 - 1;
  const int quad = id & 3, d = id >> 2;
  float *hp = p.ssm + (size_t)l * MB * Di * NS + (size_t)id * 4;
  float4 hv[MB];
#pragma unroll
  for (int m = 0; m < MB; ++m) hv[m] = *reinterpret_cast<const float4 *>(hp + (size_t)m * Di * NS);
  const unsigned aw = gload<unsigned>(q->A + (size_t)d * NS + 4 * quad);
  const float bias = gload<float>(q->dt_bias + d);
  const float Dq = static_cast<float>(gload<signed char>(q->D + d));
  v4i w[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const int kc = 16 * quad + 64 * j;
    w[j] = v4i{0, 0, 0, 0};
    if (kc < R) w[j] = gload<v4i>(q->W_dt + (size_t)d * R + kc);
  }
  const float m_dt = now(q->m_dt), s_x = now(q->s_x), s_dt = now(q->s_dt), s_z = now(q->s_z), s_B = now(q->s_B), s_C = now(q->s_C),
              s_A = now(q->s_A), s_D = now(q->s_D);
  if (tid < 64) wait_ahead(p.w.x + scan_front(idx), l + 1, p.w.dbc + scan_watch(idx, p.nB), l + 1, patience);
  sync();
  unsigned xw[MB], zw[MB];
  {
    int at[MB];
#pragma unroll
    for (int m = 0; m < MB; ++m) at[m] = m * p.x_row + quad_at(d / 4);
    wait_words(p.w.x, at, l + 1, xw, patience);
    wait_words(p.w.z, at, l + 1, zw, patience);
  }
  for (int i = tid; i < MB * (NX / 4); i += BC_THREADS) {
    const int at[1] = {dbc_at(i / (NX / 4), i % (NX / 4))};
    unsigned dw[1];
    wait_words(p.w.dbc, at, l + 1, dw, patience);
    reinterpret_cast<unsigned *>(sdbc)[i] = dw[0];
  }
  sync();
  const bool hand_on = live && !patience.gave_up();
  const int sh = 8 * (d & 3);
#pragma unroll
  for (int m = 0; m < MB; ++m) {
    const int8_t *row = sdbc + m * NX;
    int acc = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int kc = 16 * quad + 64 * j;
      if (kc < R) {
        const v4i a = *reinterpret_cast<const v4i *>(row + kc);
#pragma unroll
        for (int e = 0; e < 4; ++e) acc = __builtin_amdgcn_sdot4(a[e], w[j][e], acc, false);
      }
    }
    const unsigned bw = *reinterpret_cast<const unsigned *>(row + R + 4 * quad);
    const unsigned cw = *reinterpret_cast<const unsigned *>(row + R + NS + 4 * quad);
    acc += __builtin_amdgcn_update_dpp(0, acc, 0xB1, 0xf, 0xf, true);  // quad_perm [1, 0, 3, 2]
    acc += __builtin_amdgcn_update_dpp(0, acc, 0x4E, 0xf, 0xf, true);  // quad_perm [2, 3, 0, 1]
    const int dtq = static_cast<int>(__builtin_rintf(__builtin_amdgcn_fmed3f(static_cast<float>(acc) * m_dt, -128.f, 127.f)));
    const float xv = __builtin_fmaf(s_x, static_cast<float>(static_cast<int8_t>(xw[m] >> sh)), -0.f);
    const float dt = softplus_f(s_dt * static_cast<float>(dtq) + bias);
    const float zv = s_z * static_cast<float>(static_cast<int8_t>(zw[m] >> sh));
    const float u = dt * xv;
    float h[4] = {hv[m].x, hv[m].y, hv[m].z, hv[m].w};
    float y = 0.f;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const float a2 = static_cast<float>(static_cast<int8_t>(aw >> (8 * j))) * (s_A * LOG2E);
      const float Bv = s_B * static_cast<float>(static_cast<int8_t>(bw >> (8 * j)));
      const float Cv = s_C * static_cast<float>(static_cast<int8_t>(cw >> (8 * j)));
      h[j] = __builtin_fmaf(__builtin_amdgcn_exp2f(dt * a2), h[j], u * Bv);
      y = __builtin_fmaf(Cv, h[j], y);
    }
    y += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), 0xB1, 0xf, 0xf, true));
    y += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(y), 0x4E, 0xf, 0xf, true));
    y = __builtin_fmaf(s_D * Dq, xv, y);
    const unsigned g = __half_as_ushort(__float2half_rn(silu_gate(y, zv)));
    // the neighbouring channel's (lane ^ 4, at lanes that are multiples of 8: four lanes up the row)
    const unsigned g1 = static_cast<unsigned>(__builtin_amdgcn_update_dpp(0, static_cast<int>(g), 0x104, 0xf, 0xf, true));  // row_shl 4
    if (hand_on) {
      if ((tid & 7) == 0) word_store(p.w.g + m * p.g_row + gate_at(d), g | (g1 << 16), l + 1);
      *reinterpret_cast<float4 *>(hp + (size_t)m * Di * NS) = make_float4(h[0], h[1], h[2], h[3]);
    }
  }
}

// ---- role D: Hadamard + quantization of every row (each workgroup for itself), out_proj for D_COLS columns, residual add
template <int K, int LOGM, int MB>
__device__ __forceinline__ void role_out(const StackArgs &p, int l, int idx, float *row, int (*red)[MB * D_COLS],
                                         const RoleBarrier &sync, const Patience &patience) {
  const LayerRef q = layer_ref(p.layers, l);
  idx = fresh(idx);
  const int tid = fresh_tid(64 * A_WAVES), lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  constexpr int n = K << LOGM, NT = D_THREADS;
  const int Dm = p.Dm, n0 = idx * D_COLS;
  const bool item_live = n / 16 == NT || tid < n / 16;
  const int item = item_live ? tid : n / 16 - 1;
  v4i wv[D_COLS];
#pragma unroll
  for (int j = 0; j < D_COLS; ++j) {
    wv[j] = gload<v4i>(q->W_outH + (size_t)min(n0 + j, Dm - 1) * n + (size_t)item * 16);
    throttle(j);
  }
  OrderK hk;
  if constexpr (K > 1) {
    hk = order_k_operands<K, false>(lane);
    asm volatile("" : "+v"(hk.f[0]), "+v"(hk.f[1]));  // (read now, not behind the wait)
  }
  const float inv_s_y = now(q->inv_s_y), m_out = now(q->m_out);
  // thread t finishes output n0 + t % D_COLS of row t / D_COLS (Dm and D_COLS are even: a pair of outputs is all in or all out)
  const int fr = tid / D_COLS, fc = n0 + tid % D_COLS;
  const bool fin = tid < MB * D_COLS && fc < Dm;
  const int s_at[1] = {pair_at(fr, fc / 2)};
  unsigned res[1] = {0};
  if (fin) wait_words(p.w.s, s_at, l + 1, res, patience);
  // where this thread's words lie and go: formed now, not behind the wait
  int at[(n / 2 + NT - 1) / NT], to[(n / 2 + NT - 1) / NT];
#pragma unroll
  for (int k = 0; k < (n / 2 + NT - 1) / NT; ++k) {
    const int i = 2 * min(tid + NT * k, n / 2 - 1);
    at[k] = gate_at(i);
    if constexpr (K > 1) to[k] = static_cast<int>(reinterpret_cast<char *>(half_slot<K, LOGM>(row, i)) - reinterpret_cast<char *>(row));
    else to[k] = pad(i) * 4;
    asm volatile("" : "+v"(at[k]), "+v"(to[k]));
  }
  if (wave == 0) wait_ahead(p.w.dbc + out_front(idx, p.nB), l + 1, p.w.g + out_watch(idx, p.nC), l + 1, patience);
  sync();
#pragma unroll
  for (int r = 0; r < MB; ++r) {
    if (r > 0) sync();  // the row in front has been read
    constexpr int NWORD = (n / 2 + NT - 1) / NT;
    unsigned g[NWORD];
#pragma unroll
    for (int k = 0; k < NWORD; ++k) at[k] += r ? p.g_row : 0;
    wait_words(p.w.g, at, l + 1, g, patience);
#pragma unroll
    for (int k = 0; k < NWORD; ++k)
      if (tid + NT * k < n / 2) {
        if constexpr (K > 1) {
          *reinterpret_cast<unsigned *>(reinterpret_cast<char *>(row) + to[k]) = g[k];
        } else {
          float *dst = reinterpret_cast<float *>(reinterpret_cast<char *>(row) + to[k]);
          dst[0] = __half2float(__ushort_as_half(static_cast<unsigned short>(g[k] & 0xffffu)));
          dst[1] = __half2float(__ushort_as_half(static_cast<unsigned short>(g[k] >> 16)));
        }
      }
    if constexpr (K > 1) order_k_mfma<K, LOGM, NT>(row, tid, hk, sync);
    else sync();
    high_passes<K, LOGM, NT>(row, tid, sync);
    float v[16];
    last_pass(row, item, v);
    v4i c;
#pragma unroll
    for (int k = 0; k < 4; ++k)
      c[k] = static_cast<int>(pack_q8x4(v[4 * k] * inv_s_y, v[4 * k + 1] * inv_s_y, v[4 * k + 2] * inv_s_y, v[4 * k + 3] * inv_s_y));
    if (!item_live) c = v4i{0, 0, 0, 0};
    int dots[D_COLS];
#pragma unroll
    for (int j = 0; j < D_COLS; ++j) {
      dots[j] = 0;
#pragma unroll
      for (int e = 0; e < 4; ++e) dots[j] = __builtin_amdgcn_sdot4(c[e], wv[j][e], dots[j], false);
    }
    const int mine = wave_sums<D_COLS>(dots, lane);
    if (lane < D_COLS) red[wave][r * D_COLS + lane] = mine;
  }
  sync();
  const bool gave_up = patience.gave_up();
  if (fin) {
    int a = 0;
#pragma unroll
    for (int w = 0; w < D_WAVES; ++w) a += red[w][tid];
    float y = static_cast<float>(a) * m_out;
    // one rounding from product to half for the orders whose items fill whole waves, two for the others, as
    // hadamard_out_proj_kernel has it
    if constexpr (threads_for(n) != n / 16) asm volatile("" : "+v"(y));
    __half o = __float2half_rn(y);
    const __half rh = __ushort_as_half(static_cast<unsigned short>((fc & 1) ? res[0] >> 16 : res[0] & 0xffffu));
    if (l + 1 == p.n_layers) {
      if (gave_up) o = __ushort_as_half(static_cast<unsigned short>(0x7e00));
      p.out[(size_t)fr * Dm + fc] = o;
      p.res[(size_t)fr * Dm + fc] = rh;
    } else {
      const unsigned t = __half_as_ushort(__float2half_rn(__half2float(o) + __half2float(rh)));
      const unsigned t1 = __shfl_down(t, 1);
      if ((fc & 1) == 0 && !gave_up) word_store(p.w.s + s_at[0], t | (t1 << 16), l + 2);
    }
  }
}

template <int K, int LOGM, int MB>
__global__ __launch_bounds__(STACK_THREADS) void decode_stack_kernel(StackArgs p) {
  constexpr int n = K << LOGM;
  extern __shared__ __attribute__((aligned(16))) float row[];          // role D's row
  __shared__ __attribute__((aligned(16))) int8_t sA[MB * PF * 1024];    // role A's codes
  __shared__ InShared<MB> sIn;
  __shared__ __attribute__((aligned(16))) int8_t sx[MB * n];            // role B's codes
  __shared__ __attribute__((aligned(16))) int8_t sdbc[MB * (256 + 2 * NS)];
  __shared__ int red_x[BC_WAVES][MB * 4], red_out[D_WAVES][MB * D_COLS];
  __shared__ unsigned count[3], gave_up[3];
  __shared__ int s_word;
  const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int G = gridDim.x;
  unsigned *ctrl = p.w.ctrl;
  if (tid < 3) count[tid] = gave_up[tid] = 0;
  if (tid == 0) {
    unsigned mode = 2;
    if (!p.from_counter) {
      // sign in: eight counters by workgroup index, their last arrivals in a ninth
      const int sub = blockIdx.x & 7, members = (G - sub + 7) / 8, subs = min(G, 8);
      if (__hip_atomic_fetch_add(ctrl + (C_SUB + sub) * CTRL_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == (unsigned)members &&
          __hip_atomic_fetch_add(ctrl + C_TOP * CTRL_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1 == (unsigned)subs)
        atomicCAS(ctrl + C_MODE * CTRL_STRIDE, 0u, 1u);
      for (int tries = 0; (mode = ctrl_load(ctrl + C_MODE * CTRL_STRIDE)) == 0; ++tries)
        if (tries >= SIGN_IN_TRIES) {
          const unsigned was = atomicCAS(ctrl + C_MODE * CTRL_STRIDE, 0u, 2u);
          mode = was == 0 ? 2u : was;
          break;
        }
    }
    s_word = (int)mode;
  }
  __syncthreads();
  const bool resident = s_word == 1;
  const int role = wave < A_WAVES ? 0 : (wave < A_WAVES + D_WAVES ? 1 : 2);
  const RoleBarrier sync{&count[role], static_cast<unsigned>(role == 0 ? A_WAVES : (role == 1 ? D_WAVES : BC_WAVES)), 0u};
  const int per_block = p.nA + p.nB + p.nC + p.nD;
  // resident: this workgroup's item of each role for every block, each role's waves at their own pace
  const int blk = blockIdx.x;
  int l = 0, item_a = blk < p.nA ? blk : -1, item_d = blk < p.nD ? blk : -1, item_x = blk < p.nB ? blk : -1,
      item_c = blk >= p.nB && blk < p.nB + p.nC ? blk - p.nB : -1;
  for (;; ++l) {
    if (!resident) {  // one item of one role at a time
      __syncthreads();
      if (tid == 0) s_word = (int)__hip_atomic_fetch_add(ctrl + C_TICKET * CTRL_STRIDE, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __syncthreads();
      const int ticket = __builtin_amdgcn_readfirstlane(s_word);
      l = ticket / per_block;
      int r = ticket % per_block;
      item_a = r < p.nA ? r : -1;
      r -= p.nA;
      item_x = r >= 0 && r < p.nB ? r : -1;
      r -= p.nB;
      item_c = r >= 0 && r < p.nC ? r : -1;
      r -= p.nC;
      item_d = r;
    }
    if (l >= p.n_layers) break;
    const bool gone = __builtin_amdgcn_readfirstlane(gave_up[role]) != 0;
    if (role == 0) {
      if (item_a >= 0) role_in<MB>(p, l, item_a, sA, sIn, sync, Patience{ctrl, &gave_up[0], gone});
    } else if (role == 1) {
      if (item_d >= 0) role_out<K, LOGM, MB>(p, l, item_d, row, red_out, sync, Patience{ctrl, &gave_up[1], gone});
    } else if (item_x >= 0) {
      role_x<n, MB>(p, l, item_x, sx, red_x, sync, Patience{ctrl, &gave_up[2], gone});
    } else if (item_c >= 0) {
      role_scan<n, MB>(p, l, item_c, sdbc, sync, Patience{ctrl, &gave_up[2], gone});
    }
  }
}

// Descriptors of up to CHUNK_LAYERS blocks; the first launch also sets up the words: the residual stream of block 0 is the embedding
// of the token (plus zero, as the first add of the separate kernels has it), all other words (those between the lines among them) and the control
// words zero.
__global__ __launch_bounds__(256) void stack_begin_kernel(LayerChunk chunk, StackLayer *dst, int count, const __half *E,
                                                          const int32_t *tokens, int M, int Dm, int vocab, Words w, unsigned n_words, unsigned first_tag) {
  if (blockIdx.x == 0) {
    // (read through the argument segment: indexing the by-value struct would copy it to scratch first)
    typedef __attribute__((address_space(4))) const unsigned *args_t;
    const args_t src = (args_t)__builtin_amdgcn_kernarg_segment_ptr();
    for (int i = threadIdx.x; i < count * (int)(sizeof(StackLayer) / 4); i += 256) reinterpret_cast<unsigned *>(dst)[i] = src[i];
  }
  if (!E) return;
  // the words of the residual stream come first
  const unsigned i = blockIdx.x * 256 + threadIdx.x;
  if (i >= n_words) return;
  u64 word = 0;
  const int slot = i % LINE, m = slot / (D_COLS / 2), c = i / LINE * (D_COLS / 2) + slot % (D_COLS / 2);
  if (m < M && c < Dm / 2) {  // i = pair_at(m, c)
    const int tok = min(max(tokens[m], 0), vocab - 1);
    const __half2 e = reinterpret_cast<const __half2 *>(E + (size_t)tok * Dm)[c];
    const unsigned lo = __half_as_ushort(__float2half_rn(0.f + __half2float(__low2half(e))));
    const unsigned hi = __half_as_ushort(__float2half_rn(0.f + __half2float(__high2half(e))));
    word = (static_cast<u64>(first_tag) << 32) | lo | (hi << 16);
  }
  w.s[i] = word;
}

struct StackCarve {
  size_t layers, s, x, z, dbc, g, ctrl, total;
};
int stack_x_row(int Di) { return ((Di / 4 + A_COLS / 4 - 1) / (A_COLS / 4)) * LINE; }
int stack_g_row(int Di) { return (Di + BC_THREADS / 4 - 1) / (BC_THREADS / 4) * 2 * LINE; }
StackCarve stack_carve(int n_layers, int M, int Dm, int Di, int R) {
  StackCarve c{};
  size_t off = 0;
  auto take = [&](size_t bytes) {
    const size_t at = off;
    off += align_up(bytes, 256);
    return at;
  };
  c.layers = take((size_t)n_layers * sizeof(StackLayer));
  c.s = take((size_t)((Dm + D_COLS - 1) / D_COLS) * LINE * 8);
  c.x = take((size_t)M * stack_x_row(Di) * 8);
  c.z = take((size_t)M * stack_x_row(Di) * 8);
  c.dbc = take((size_t)(R + 2 * NS) / 4 * LINE * 8);
  c.g = take((size_t)M * stack_g_row(Di) * 8);
  c.ctrl = take((size_t)CTRL_WORDS * CTRL_STRIDE * 4);
  c.total = off;
  return c;
}

// LDS of role D's row
constexpr size_t row_bytes(int n) { return (size_t)(n + n / 4) * sizeof(float); }

// Does the current device hold `groups` workgroups of this kernel at once (as far as the runtime can tell)?
template <int K, int LOGM, int MB>
bool fits(int groups) {
  static std::atomic<int> known[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess) return false;
  std::atomic<int> &slot = known[dev & 63];
  int v = slot.load(std::memory_order_relaxed);
  if (v == 0) {
    int per_cu = 0, cus = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, decode_stack_kernel<K, LOGM, MB>, STACK_THREADS, row_bytes(K << LOGM)) != hipSuccess ||
        hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess)
      return false;
    v = per_cu * cus;
    slot.store(v, std::memory_order_relaxed);
  }
  return groups <= v;
}

// Items of each role in one block.
struct Items {
  int nA, nB, nC, nD;
  int groups() const { return std::max(std::max(nA, nD), nB + nC); }  // workgroups, one item of each role for each
};
Items stack_items(int Dm, int Di, int R) {
  return Items{(2 * Di + A_COLS - 1) / A_COLS, (R + 2 * NS) / 4, (Di * 4 + BC_THREADS - 1) / BC_THREADS, (Dm + D_COLS - 1) / D_COLS};
}

template <int K, int LOGM, int MB, typename Begin>
int run_stack(const StackArgs &args, const Begin &begin, hipStream_t st) {
  constexpr int n = K << LOGM;
  StackArgs p = args;
  const Items items = stack_items(p.Dm, n, p.R);
  p.nA = items.nA;
  p.nB = items.nB;
  p.nC = items.nC;
  p.nD = items.nD;
  p.x_row = stack_x_row(n);
  p.g_row = stack_g_row(n);
  const int rc = begin();
  if (rc != QUAMBA_OK) return rc;
  hipLaunchKernelGGL((decode_stack_kernel<K, LOGM, MB>), dim3(items.groups()), dim3(STACK_THREADS), row_bytes(n), st, p);
  QUAMBA_LAUNCH_CHECK();
  return QUAMBA_OK;
}

// What is built: d_inner = K << LOGM, sequences.  Two sequences of 4096 gain 3 % alone on the GPU (24 blocks 600 -> 582 us; the other widths 11 to
// 20 %) and lose 27 to 46 % where two to four users run a step each at the same time (721 -> 992, 1045 -> 1921): launch by launch.
#define QUAMBA_STACK_WIDTHS(CASE)                                                                                    \
  CASE(12, 7, 1) CASE(12, 7, 2) CASE(1, 11, 1) CASE(1, 11, 2) CASE(20, 7, 1) CASE(20, 7, 2) CASE(12, 8, 1) CASE(12, 8, 2) \
  CASE(1, 12, 1) CASE(20, 8, 1) CASE(20, 8, 2)

// Is a step of this shape served in one launch on the current device?
bool stack_served(int n_layers, int Bt, int Dm, int Di, int R, size_t ws_bytes) {
  // (one block alone: no weights to read ahead)
  if (g_decode_stack_hook.load(std::memory_order_relaxed) == 1 || Bt < 1 || Bt > 2 || n_layers < 2 || Dm > PF * 1024 || R > 256) return false;
  if (stack_carve(n_layers, Bt, Dm, Di, R).total > ws_bytes || (long long)n_layers * 4096 > 0x7fffffffLL) return false;
  const int groups = stack_items(Dm, Di, R).groups();
#define QUAMBA_CASE(K, LM, MB) \
  if (Di == K << LM && Bt == MB) return fits<K, LM, MB>(groups);
  QUAMBA_STACK_WIDTHS(QUAMBA_CASE)
#undef QUAMBA_CASE
  return false;
}

}  // namespace

// All blocks of a generation step from tokens [Bt]; leaves the last block's output and the residual stream before its add in `out`
// and `res`, the states advanced; **gave_up is then nonzero if a wait in it was given up.  *served = false (and nothing launched): the general path has to run.
int launch_decode_stack(const quamba_model *m, const int32_t *tokens, int Bt, float *ssm, __half *conv, __half *out, __half *res,
                        void *ws, size_t ws_bytes, hipStream_t st, bool *served, const unsigned **gave_up) {
  const int Dm = m->dims.d_model, Di = m->dims.d_inner, R = m->dims.dt_rank;
  *served = stack_served(m->n_layers, Bt, Dm, Di, R, ws_bytes);
  if (!*served) return QUAMBA_OK;
  const int hook = g_decode_stack_hook.load(std::memory_order_relaxed);
  const StackCarve c = stack_carve(m->n_layers, Bt, Dm, Di, R);
  char *base = static_cast<char *>(ws);
  StackArgs a{};
  a.layers = reinterpret_cast<const StackLayer *>(base + c.layers);
  a.n_layers = m->n_layers; a.Dm = Dm; a.Di = Di; a.R = R; a.eps = m->eps;
  a.ssm = ssm; a.conv = conv; a.out = out; a.res = res;
  auto words = [&](size_t at) { return reinterpret_cast<u64 *>(base + at); };
  a.w = Words{words(c.s), words(c.x), words(c.z), words(c.dbc), words(c.g), reinterpret_cast<unsigned *>(base + c.ctrl)};
  a.from_counter = hook == 2;
  *gave_up = a.w.ctrl + C_GAVE_UP * CTRL_STRIDE;
  auto begin = [&]() -> int {
    for (int l0 = 0; l0 < m->n_layers; l0 += CHUNK_LAYERS) {
      LayerChunk chunk{};
      const int count = m->n_layers - l0 < CHUNK_LAYERS ? m->n_layers - l0 : CHUNK_LAYERS;
      for (int i = 0; i < count; ++i) {
        const quamba_layer &ly = m->layers[l0 + i];
        const quamba_scales &s = ly.s;
        chunk.layer[i] = StackLayer{ly.q.W_in, ly.q.conv_w, ly.q.W_x, ly.q.W_dt, ly.q.A, ly.q.D, ly.q.W_outH, ly.q.conv_b, ly.q.dt_bias,
                                    reinterpret_cast<const __half *>(ly.norm_w), s.inv_s_u, s.m_in_x, s.m_in_z, s.s_cw, s.s_xpre,
                                    s.inv_s_x, s.m_x_dt, s.m_x_B, s.m_x_C, s.m_dt, s.s_x, s.s_dt, s.s_z, s.s_B, s.s_C, s.s_A, s.s_D,
                                    s.inv_s_y, s.m_out, 0.f};
      }
      const unsigned n_words = l0 ? 0u : (unsigned)((c.total - c.s) / 8);
      hipLaunchKernelGGL(stack_begin_kernel, dim3(std::max(1u, (n_words + 255) / 256)), dim3(256), 0, st, chunk,
                         const_cast<StackLayer *>(a.layers) + l0, count,
                         l0 ? nullptr : reinterpret_cast<const __half *>(m->embedding), tokens, Bt, Dm, m->vocab, a.w, n_words, hook == 3 ? 0u : 1u);
      QUAMBA_LAUNCH_CHECK();
    }
    return QUAMBA_OK;
  };
#define QUAMBA_CASE(K, LM, MB) \
  if (Di == K << LM && Bt == MB) return run_stack<K, LM, MB>(a, begin, st);
  QUAMBA_STACK_WIDTHS(QUAMBA_CASE)
#undef QUAMBA_CASE
  return fail(QUAMBA_EUNSUPPORTED, "decode: d_inner=%d is not served in one launch", Di);
}

// The words one item of a role (0 = A, 1 = B, 2 = C, 3 = D) deals with in a block, as the kernel forms their places; four numbers for each: buffer (0 s, 1 x, 2 z,
// 3 dbc, 4 g), word, tag minus number of the block, how (0 written, 1 awaited with this tag, 2 watched until this tag or a later one).
// Returns how many there are; the first `cap` are stored.
int stack_words(int Dm, int Di, int R, int Bt, int role, int item, int32_t *out, int cap) {
  const Items n = stack_items(Dm, Di, R);
  const int count[4] = {n.nA, n.nB, n.nC, n.nD};
  if (role < 0 || role > 3 || item < 0 || item >= count[role] || Bt < 1 || Bt > 2) return -1;
  const int xr = stack_x_row(Di), gr = stack_g_row(Di);
  int k = 0;
  auto put = [&](int buffer, int word, int tag, int how) {
    if (k < cap) {
      const int32_t e[4] = {buffer, word, tag, how};
      std::copy(e, e + 4, out + 4 * k);
    }
    ++k;
  };
  for (int m = 0; m < Bt; ++m) {
    if (role == 0) {
      for (int i = 0; i < Dm / 2; ++i) put(0, pair_at(m, i), 1, 1);
      for (int c = item * A_COLS; c < std::min((item + 1) * A_COLS, 2 * Di); c += 4)
        put(c < Di ? 1 : 2, m * xr + quad_at((c < Di ? c : c - Di) / 4), 1, 0);
    } else if (role == 1) {
      for (int i = 0; i < Di / 4; ++i) put(1, m * xr + quad_at(i), 1, 1);
      put(3, dbc_at(m, item), 1, 0);
    } else if (role == 2) {
      for (int d = item * (BC_THREADS / 4); d < std::min((item + 1) * (BC_THREADS / 4), Di); ++d) {
        put(1, m * xr + quad_at(d / 4), 1, 1);
        put(2, m * xr + quad_at(d / 4), 1, 1);
        if (d % 2 == 0) put(4, m * gr + gate_at(d), 1, 0);
      }
      for (int i = 0; i < n.nB; ++i) put(3, dbc_at(m, i), 1, 1);
    } else {
      for (int i = 0; i < Di / 2; ++i) put(4, m * gr + gate_at(2 * i), 1, 1);
      for (int c = item * D_COLS; c < std::min((item + 1) * D_COLS, Dm); c += 2) {
        put(0, pair_at(m, c / 2), 1, 1);
        put(0, pair_at(m, c / 2), 2, 0);
      }
    }
  }
  const int watch = watch_ends(2, 1) ? 2 : 1;
  if (role == 0) {
    put(4, in_front(item, n.nC), 0, watch);
    put(0, in_watch(item, n.nD), 1, watch);
  } else if (role == 1) {
    put(0, x_front(item, n.nD), 1, watch);
    put(1, x_watch(item, Di), 1, watch);
  } else if (role == 2) {
    put(1, scan_front(item), 1, watch);
    put(3, scan_watch(item, n.nB), 1, watch);
  } else {
    put(3, out_front(item, n.nB), 1, watch);
    put(4, out_watch(item, n.nC), 1, watch);
  }
  return k;
}

}  // namespace quamba

extern "C" int quamba_debug_decode_stack_words(int d_model, int d_inner, int dt_rank, int batch, int role, int item, int32_t *out, int cap) {
  if (d_model < 16 || d_inner < 16 || dt_rank < 16 || (cap > 0 && !out)) return -1;
  return quamba::stack_words(d_model, d_inner, dt_rank, batch, role, item, out, cap);
}
extern "C" int quamba_debug_decode_stack_served(const quamba_dims *d, int n_layers, int batch) {
  using namespace quamba;
  if (check_model_dims(d) != QUAMBA_OK || batch < 1 || !mixer_decode_norm_available(d, batch) || !mixer_decode_fuses_dt()) return 0;
  return stack_served(n_layers, batch, d->d_model, d->d_inner, d->dt_rank, mixer_workspace_bytes(d, batch, 1));
}
extern "C" void quamba_debug_set_decode_stack(int v) { quamba::g_decode_stack_hook.store(v); }
