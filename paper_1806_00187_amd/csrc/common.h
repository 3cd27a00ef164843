// Internal helpers shared by the gfx950 kernels of the NMT training-step library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include "nmt.h"

typedef _Float16 half_t;
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;

// ---- error handling --------------------------------------------------------------------------
void nmt_set_error(const char* fmt, ...);

#define NMT_HIP_CHECK(expr)                                                                  \
  do {                                                                                       \
    hipError_t e_ = (expr);                                                                  \
    if (e_ != hipSuccess) {                                                                  \
      nmt_set_error("%s failed: %s (%s:%d)", #expr, hipGetErrorString(e_), __FILE__, __LINE__); \
      return NMT_EHIP;                                                                       \
    }                                                                                        \
  } while (0)

#define NMT_REQUIRE(cond, ...)   \
  do {                           \
    if (!(cond)) {               \
      nmt_set_error(__VA_ARGS__); \
      return NMT_EINVAL;         \
    }                            \
  } while (0)

#define NMT_LAUNCH_CHECK() NMT_HIP_CHECK(hipGetLastError())

// ---- the device and the launch-form switches ------------------------------------------------------
// Compute units and XCDs (dies with an L2 of their own) of the current device, asked of the runtime once.
struct DeviceInfo {
  int cus = 256, xcds = 8;
};
const DeviceInfo& device_info();
// More than 64 KB of dynamic LDS has to be asked for: once per device, kernel and size (from any thread), not once per launch.
int allow_lds(const void* kernel, size_t bytes);
// Process-wide switches of launch forms (nmt_tuning): which work-group computes what, never what is computed.
struct Tuning {
  int gemm_group = 4;     // tile rows swept column by column before the next rows
  int gemm_persist = 1;   // 0: never the persistent GEMM form, 1: where it applies (256 x 256 tiles, row-major A, no split, one of its five epilogues)
  int attn_persist = 1;   // 0: one attention work item per work-group
  int worklists = 1;      // 0: attention kernels enumerate every (sentence, tile) instead of taking work lists
  int one_stream = 0;     // 1: forward and backward passes keep to the caller's stream
  int gemm_share = 1;     // products expected to run side by side (callers that keep several passes in flight): large tiles
                          // are chosen as if each product had 1/gemm_share of the compute units
  int row_chain = 1;      // 0: narrow models' operations between two attentions are launches of their own
  int gemm_tile = 0;      // experiments: 0 = chosen per product; 1..5 force 256x256, 128x128, 128x64, 64x128, 64x64 tiles (products not cut along k, no weight-gradient groups)
  int gemm_timing = 0;    // 1: every GEMM product (a weight-gradient group: its launch) is bracketed by HIP events on its launch stream (nmt_gemm_timing reads them)
};
Tuning& tuning();

static inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
static inline int64_t round_up(int64_t x, int64_t m) { return (x + m - 1) / m * m; }
static inline int ceil_div(int64_t a, int64_t b) { return (int)((a + b - 1) / b); }

// ---- wavefront reductions (64 lanes) --------------------------------------------------------
// Every lane gets the result.  The partner's value comes over the vector ALU's own lane crossings (half and row swaps,
// row rotations, quad permutations: a few clocks each) instead of the LDS permute a shuffle turns into (~130 clocks each,
// in a chain of six): the LayerNorm kernels are a chain of two to four of these (260 rows x 64: forward 4.5 -> 3.8 us, backward
// 9.9 -> 8.6, with the row keys requested ahead).  Lane L meets L ^ 32, then 16, 8, 4, 2, 1;
// a rotation by 4 meets L ^ 4 or (L ^ 4) ^ 8, which hold the same value by then.
template <typename Op>
__device__ __forceinline__ float wave_reduce(float v, Op op) {
  auto bits = [](float x) { return __builtin_bit_cast(int, x); };
  auto num = [](int x) { return __builtin_bit_cast(float, x); };
  const auto halves = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
  v = op(__builtin_bit_cast(float, (unsigned)halves[0]), __builtin_bit_cast(float, (unsigned)halves[1]));
  const auto rows = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
  v = op(__builtin_bit_cast(float, (unsigned)rows[0]), __builtin_bit_cast(float, (unsigned)rows[1]));
  v = op(v, num(__builtin_amdgcn_update_dpp(0, bits(v), 0x128, 0xF, 0xF, true)));  // row_ror:8
  v = op(v, num(__builtin_amdgcn_update_dpp(0, bits(v), 0x124, 0xF, 0xF, true)));  // row_ror:4
  v = op(v, num(__builtin_amdgcn_update_dpp(0, bits(v), 0x4E, 0xF, 0xF, true)));   // quad_perm:[2,3,0,1]
  return op(v, num(__builtin_amdgcn_update_dpp(0, bits(v), 0xB1, 0xF, 0xF, true)));  // quad_perm:[1,0,3,2]
}
__device__ __forceinline__ float wave_sum(float v) {
  return wave_reduce(v, [](float a, float b) { return a + b; });
}
__device__ __forceinline__ float wave_max(float v) {
  return wave_reduce(v, [](float a, float b) { return fmaxf(a, b); });
}
// The value of lane L ^ 32 combined with this lane's, for values that differ between the wavefront's halves.
__device__ __forceinline__ float half_sum(float v) {
  const auto h = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
  return __builtin_bit_cast(float, (unsigned)h[0]) + __builtin_bit_cast(float, (unsigned)h[1]);
}
__device__ __forceinline__ float half_max(float v) {
  const auto h = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)h[0]), __builtin_bit_cast(float, (unsigned)h[1]));
}

// ---- Philox4x32-10 counter-based generator (Salmon et al., SC'11) ----------------------------
__device__ __forceinline__ uint4 philox4x32_10(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    if (r) {
      k0 += 0x9E3779B9u;
      k1 += 0xBB67AE85u;
    }
    // one 32 x 32 -> 64 bit multiply per product (a single quarter-rate instruction instead of a high / low pair)
    const uint64_t p0 = (uint64_t)0xD2511F53u * c.x, p1 = (uint64_t)0xCD9E8D57u * c.z;
    const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0, hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
    c = make_uint4(hi1 ^ c.y ^ k0, lo1, hi0 ^ c.w ^ k1, lo0);
  }
  return c;
}

// Device-side dropout description (built on the host from nmt_dropout).  Row r of an activation
// belongs to sentence `uid` at position `pos` of sub-batch `micro`: either r / n_pos, r % n_pos and
// the micro index in c3 (one rectangular batch), or, when `rowkey` is set, rowkey[r] =
// (uid, pos | micro << 16) (several batches of different shapes stacked row-wise).
struct DropDev {
  uint32_t k0, k1;      // Philox key = seed
  uint32_t c3;          // step << 8 | micro
  uint32_t site_hi;     // site << 16
  uint32_t thr;         // keep iff 16-bit uniform >= thr; 0 = dropout off
  float scale;          // 1 / (1 - p)
  int32_t n_pos;        // rows per sentence
  const uint32_t* uid;  // per-sentence ids or nullptr
  const uint2* rowkey;  // per-row (uid, pos | micro << 16) or nullptr
};

DropDev make_drop(const nmt_dropout* d);  // host; d == nullptr or p <= 0 gives thr = 0

// Position within its sentence of row `row`.
__device__ __forceinline__ uint32_t drop_row_pos(const DropDev& dd, uint32_t row) {
  return dd.rowkey ? (dd.rowkey[row].y & 0xFFFFu) : row % (uint32_t)dd.n_pos;
}

// What row `row` puts into the counters, for kernels that fetch it ahead of the draws.
struct DropRow { uint32_t uid, pos, c3; };
__device__ __forceinline__ DropRow drop_row_of(const DropDev& dd, uint2 rk) { return DropRow{rk.x, rk.y & 0xFFFFu, (dd.c3 & 0xFFFFFF00u) | (rk.y >> 16)}; }
__device__ __forceinline__ DropRow drop_row(const DropDev& dd, uint32_t row) {
  if (dd.rowkey) return drop_row_of(dd, dd.rowkey[row]);
  const uint32_t sent = row / (uint32_t)dd.n_pos;
  return DropRow{dd.uid ? dd.uid[sent] : sent, row - sent * (uint32_t)dd.n_pos, dd.c3};
}
// Keep decisions of the 8 columns [8*grp, 8*grp+8) of a row: bit i set = column 8*grp+i kept.
__device__ __forceinline__ uint32_t drop_keep8(const DropDev& dd, const DropRow& r, uint32_t grp) {
  const uint4 w = philox4x32_10(make_uint4(grp, r.uid, dd.site_hi | r.pos, r.c3), dd.k0, dd.k1);
  const uint32_t words[4] = {w.x, w.y, w.z, w.w};
  uint32_t bits = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    bits |= ((words[i] & 0xFFFFu) >= dd.thr ? 1u : 0u) << (2 * i);
    bits |= ((words[i] >> 16) >= dd.thr ? 1u : 0u) << (2 * i + 1);
  }
  return bits;
}
__device__ __forceinline__ uint32_t drop_keep8(const DropDev& dd, uint32_t row, uint32_t grp) { return drop_keep8(dd, drop_row(dd, row), grp); }

// One word of every cache line of a kernel's arguments, asked for together: where the code reads them one after the other, each line's first
// use is a trip to memory of its own (0.4 us).
template <typename Args>
__device__ __forceinline__ void touch(const Args& a) {
  const uint32_t* words = reinterpret_cast<const uint32_t*>(&a);
  uint32_t w[(sizeof(Args) + 63) / 64];
#pragma unroll
  for (size_t i = 0; i < sizeof(Args) / 64; ++i) w[i] = words[16 * i];
  w[sizeof(w) / 4 - 1] = words[sizeof(Args) / 4 - 1];
#pragma unroll
  for (size_t i = 0; i < sizeof(w) / 4; ++i) asm volatile("" ::"s"(w[i]));
}

// The same for a kernel whose arguments, BYTES of them, are no struct.
template <int BYTES>
__device__ __forceinline__ void touch_arguments() {
  const auto* words = (const __attribute__((address_space(4))) uint32_t*)__builtin_amdgcn_kernarg_segment_ptr();
  uint32_t w[(BYTES + 63) / 64];
#pragma unroll
  for (int i = 0; i < (BYTES + 63) / 64; ++i) w[i] = words[i + 1 < (BYTES + 63) / 64 ? 16 * i : BYTES / 4 - 1];
#pragma unroll
  for (int i = 0; i < (BYTES + 63) / 64; ++i) asm volatile("" ::"s"(w[i]));
}
// Division by a number the host knows, without the reciprocal the compiler would form first (100 instructions' time in front of a kernel's first load).
struct Divisor {
  uint32_t d = 1, m = 0xFFFFFFFFu;  // m = floor(2^32 / d): the high word of n m is n / d or one less
};
static inline Divisor divisor(uint32_t d) { return Divisor{d, d == 1 ? 0xFFFFFFFFu : (uint32_t)((1ull << 32) / d)}; }
__device__ __forceinline__ uint32_t div_mod(uint32_t n, const Divisor& by, uint32_t& rest) {
  uint32_t q = __umulhi(n, by.m);
  rest = n - q * by.d;
  if (rest >= by.d) {
    ++q;
    rest -= by.d;
  }
  return q;
}

// Orders one wavefront's LDS accesses: what its other lanes wrote before is visible after (LDS
// instructions of a wavefront execute in order; this keeps the compiler from reordering them).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// ---- small vector helpers ---------------------------------------------------------------------
__device__ __forceinline__ half8_t ld_half8(const half_t* p) { return *reinterpret_cast<const half8_t*>(p); }
__device__ __forceinline__ void st_half8(half_t* p, half8_t v) { *reinterpret_cast<half8_t*>(p) = v; }
// Streaming forms for data that is touched once per kernel and is larger than the caches: no retention asked for.
__device__ __forceinline__ half8_t ld_half8_nt(const half_t* p) { return __builtin_nontemporal_load(reinterpret_cast<const half8_t*>(p)); }
__device__ __forceinline__ void st_half8_nt(half_t* p, half8_t v) { __builtin_nontemporal_store(v, reinterpret_cast<half8_t*>(p)); }
__device__ __forceinline__ floatx4 ld_float4_nt(const float* p) { return __builtin_nontemporal_load(reinterpret_cast<const floatx4*>(p)); }
__device__ __forceinline__ void st_float4_nt(float* p, floatx4 v) { __builtin_nontemporal_store(v, reinterpret_cast<floatx4*>(p)); }
__device__ __forceinline__ half8_t zero_half8() {
  half8_t z = {0, 0, 0, 0, 0, 0, 0, 0};
  return z;
}

// ---- internal launchers (all enqueue on `stream`, return NMT_* codes) -------------------------
struct GemmEpilogue {
  const half_t* bias = nullptr;
  int relu = 0;
  DropDev drop = {};
  const half_t* add = nullptr;
  const half_t* relu_src = nullptr;
  float mask_scale = 1.f;
  int row0 = 0;  // row of the whole activation that row 0 of this product is (dropout counters)
  float out_scale = 1.f;  // the accumulated product is multiplied by this first (weight gradients of a large pass)
};
// partial: optional fp32 scratch of partial_floats floats for cutting the contraction into `splits`
// pieces summed by a second kernel (needs an empty epilogue; splits == 0: the launcher decides, which only the entry point
// nmt_op_gemm_splitk offers).
int launch_gemm(const half_t* A, bool a_t, int lda, const half_t* B, bool b_t, int ldb, half_t* C, int ldc,
                int M, int N, int K, const GemmEpilogue& ep, hipStream_t stream, float* partial = nullptr,
                int64_t partial_floats = 0, int splits = 1);

// One weight gradient: C[M, N] = sum_k A[k, M] B[k, N], and, if colsum is set, colsum[M] = sum_k A[k, M] (the bias gradient).
struct WgradProduct {
  const half_t *A, *B;
  half_t *C, *colsum;
  int lda, ldb, ldc, M, N, K;
};
constexpr int kMaxWgrad = 8;
// Partial sums that a group with `per_split` floats of results and column sums, over up to `rows` positions, can use of `most`.
int64_t wgrad_group_floats(int64_t per_split, int64_t rows, int64_t most);

// fp32 product on the matrix cores, for the benchmark's fp32 comparison leg (not used by the training step)
int launch_gemm_f32(const float* A, bool a_t, int lda, const float* B, bool b_t, int ldb, float* C, int ldc, int M, int N, int K,
                    int splits, hipStream_t stream);

// Sum of the event-bracketed durations of the products launched since the last call (tuning().gemm_timing), their
// number and their algorithmic FLOPs; waits for them to finish.
int gemm_timing_read(double* ms, int64_t* products, double* flops);

// Work lists of one attention kind over a sentence table, made on the device (launch_attention_worklists)
// so that the attention kernels start no work-group for a (sentence, tile) that does not exist:
// counts[c], c = 0..kAttnClasses-1: sentences whose longer side takes c + 1 tiles of 32 positions, [kAttnClasses]: longer ones,
// [kAttnClasses + 1]: query tiles; by_tiles [kAttnClasses][n_sent]: the table entries of the sentences of each class; qsent / qtile:
// per query tile its sentence's table entry and its tile number (entries are copies, so that a work
// item needs one dependent load).
constexpr int kAttnClasses = 8;
struct AttnWork {
  const int32_t* counts = nullptr;
  const int4* by_tiles = nullptr;
  const int4* qsent = nullptr;
  const int32_t* qtile = nullptr;
  int n_k_rows = 0;  // key rows in total; 0 for self-attention (the keys are the queries' rows)
};
int64_t attention_worklist_ints(int n_sent, int n_q_rows);  // int32 words of storage behind one AttnWork (16-byte aligned)
AttnWork attention_work(const int32_t* storage, int n_sent, int n_q_rows, int n_k_rows);
// The lists of up to three tables of n_sent sentences each, in one launch.
int launch_attention_worklists(const int4* const* tabs, const int* n_q_rows, int32_t* const* storage, int n, int n_sent, hipStream_t stream);

int launch_attention_fwd(const half_t* Q, int ldq, const half_t* K, int ldk, const half_t* V, int ldv, half_t* O,
                         int ldo, float* lse, const int32_t* key_ids, int pad_id, int causal, int B, int H,
                         int dh, int Tq, int Tk, const int4* sent_tab, int n_q_rows, const AttnWork* work,
                         hipStream_t stream);
int launch_attention_bwd(const half_t* Q, int ldq, const half_t* K, int ldk, const half_t* V, int ldv,
                         const half_t* O, int ldo, const half_t* dO, int lddo, const float* lse, half_t* dQ,
                         int lddq, half_t* dK, int lddk, half_t* dV, int lddv, const int32_t* key_ids, int pad_id,
                         int causal, int B, int H, int dh, int Tq, int Tk, const int4* sent_tab, int n_q_rows,
                         const AttnWork* work, hipStream_t stream);

// A stretch of weights that products soon after a LayerNorm read.  A pass touches each weight once, and between two passes the activations and the
// optimizer's state push it out of the 256 MB last-level cache: a product of few rows then waits for memory at each k-tile (3100 x 2048 x 512 and the
// 3100 x 512 x 2048 that reads its result: 21.9 us with the weights and that result in the cache, 27.6 with neither).  So the LayerNorm's launch has work-groups of its own,
// behind the rows', that read one word of each 128-byte line and drop it: the compute units are not full then, and memory is nearly idle.  With the
// products' results kept in the same cache (kWriteThrough in the products' file), Transformer-base on 2990 tokens, forward / backward 1196 / 1762 -> 1157 / 1716 us,
// Transformer-big on 380 tokens 956 / 1401 -> 881 / 1302, on 2600 tokens 2230 / 3840 -> 2220 / 3774; 40000 tokens lose nothing (9180 / 16680 -> 9065 / 16615), so
// every number of rows does it.  Activations asked for in the same way cost more than they gave (backward +1 to +3 %: they are read at memory's full rate already).
struct Ahead {
  const half_t* p = nullptr;
  uint32_t lines = 0, first = 0;  // 128-byte lines; the work-groups of rows, which come first (the launcher's)
};
constexpr int kAheadThreads = 256, kAheadLoads = 2;  // of a work-group: 64 KB
static inline Ahead ahead(const half_t* p, int64_t halves) { return Ahead{p, (uint32_t)(halves / 64), 0}; }  // (whole lines: nothing behind the stretch is read)
static inline int ahead_groups(const Ahead& a) { return ceil_div(a.lines, kAheadThreads * kAheadLoads); }
__device__ __forceinline__ void ask_ahead(const Ahead& a, int group) {
  if ((int)threadIdx.x >= kAheadThreads) return;
  uint32_t v[kAheadLoads];
#pragma unroll
  for (int i = 0; i < kAheadLoads; ++i) {
    const uint32_t line = ((uint32_t)group * kAheadLoads + i) * kAheadThreads + threadIdx.x;
    v[i] = *reinterpret_cast<const uint32_t*>(a.p + (size_t)min(line, a.lines - 1) * 64);
  }
#pragma unroll
  for (int i = 0; i < kAheadLoads; ++i) asm volatile("" ::"v"(v[i]));
}
int launch_residual_layernorm_fwd(const half_t* sub, const half_t* resid, const half_t* gamma, const half_t* beta,
                                  half_t* out, float* stats, int rows, int d, float eps, const DropDev& drop,
                                  hipStream_t stream, const Ahead& next = {});
int64_t layernorm_bwd_scratch_floats(int d);                        // partial sums of a call of any number of rows ...
int64_t layernorm_bwd_partial_floats(int most_rows, int d);         // ... of up to `most_rows`
// LayerNorm backward of one element, for every kernel that has one: the gradient of a row is the same bits whichever computes it.  So the operations are
// spelled out; left to the compiler it takes two products of a sum into one v_dot2c_f32_f16 here and not there, which rounds once for both.
// go, gamma: fp16 values (their product is exact); xhat: the normalised element; m1, m2: means of go gamma and go gamma xhat over the row.
__device__ __forceinline__ void ln_bwd_row_sums(float& s1, float& s2, float go, float gamma, float xhat) {
#pragma clang fp contract(off)
  s1 = __builtin_fmaf(go, gamma, s1);
  s2 = __builtin_fmaf(go * gamma, xhat, s2);
}
__device__ __forceinline__ float ln_bwd_dy(float go, float gamma, float xhat, float rstd, float m1, float m2) {
#pragma clang fp contract(off)
  return rstd * __builtin_fmaf(-xhat, m2, __builtin_fmaf(go, gamma, -m1));
}
// Partial rows of column sums as a kernel left them: `rows` rows of up to three quantities, and where their totals go.
struct ColumnSums {
  const float* partial;
  int rows;
  half_t* dst[3];
};
constexpr int kMaxColumnSums = 4;
// dst[k][col] = fp16(scale * sum_b partial[b][k][col]), k = 0..nq-1, for up to kMaxColumnSums buffers of partial rows.
struct FinalizeArgs {
  int nq, cols, pitch;
  float scale;
  ColumnSums in[kMaxColumnSums];
};
// One work-group's share: it owns THREADS / 32 columns of one quantity; its 32 row-lanes stride over the partial rows
// (independent loads, several in flight) and are combined in a fixed order, the same whatever THREADS.  red: 32 * (THREADS / 32 + 1) floats of LDS.
template <int THREADS>
__device__ __forceinline__ void finalize_columns(const FinalizeArgs& a, int block, float* red) {
  constexpr int COLS = THREADS / 32, PITCH = COLS + 1;
  const int cx = threadIdx.x % COLS, ry = threadIdx.x / COLS;
  const int cblocks = (a.cols + COLS - 1) / COLS;
  const int k = (block / cblocks) % a.nq, col = (block % cblocks) * COLS + cx;
  const ColumnSums& in = a.in[block / (cblocks * a.nq)];
  const int nblk = in.rows;
  float s = 0.f;
  if (col < a.cols) {
    const float* p = in.partial + (size_t)k * a.pitch + col;
    const size_t step = (size_t)a.nq * a.pitch;
    int b = ry;
    for (; b + 96 < nblk; b += 128)
      s += (p[b * step] + p[(b + 32) * step]) + (p[(b + 64) * step] + p[(b + 96) * step]);
    for (; b < nblk; b += 32) s += p[b * step];
  }
  red[ry * PITCH + cx] = s;
  __syncthreads();
  if (ry == 0 && col < a.cols) {
    float t = red[cx];
#pragma unroll
    for (int r = 1; r < 32; ++r) t += red[r * PITCH + cx];
    if (in.dst[k]) in.dst[k][col] = (half_t)(t * a.scale);
  }
}
// The row gradients; the gradients of gamma, beta and the bias are left as partial rows described by `sums`, which
// launch_layernorm_param_grads adds up (several calls' in one launch).
int launch_residual_layernorm_bwd(const half_t* dout, const half_t* sub, const half_t* resid, const half_t* gamma,
                                  const float* stats, half_t* dy, half_t* dym, half_t* dgamma, half_t* dbeta,
                                  half_t* dbias, float* partial, int rows, int d, const DropDev& drop,
                                  hipStream_t stream, ColumnSums& sums, const Ahead& next = {});
int launch_layernorm_param_grads(const ColumnSums* sums, int n, int d, float scale, hipStream_t stream);  // scale: factor on all of them
// What lies between two attentions of a narrow model, row by row, in one launch each way (d = 64, 128 or 256; see row_chain_fits).  Rows of
// d columns are contiguous.  Forward: s1 = o wo^T + bo, x1 = LN(x + dropout(s1)); if F: h = relu(x1 w1^T + b1), s2 = h w2^T + b2, x2 = LN(x1 +
// dropout(s2)); then projections of the last of these.
constexpr int kMaxRowChainProj = 4;
struct RowChainLn {
  const half_t *gamma, *beta;
  half_t *sub, *out;  // s and x of the sub-layer
  float* stats;
  DropDev drop;
};
struct RowChainFwd {
  int rows, F, n_proj;
  float eps;
  const half_t *o, *wo, *bo, *x;
  RowChainLn ln1, ln2;
  const half_t *w1, *b1, *w2, *b2;
  half_t* h;
  struct Proj { const half_t *w, *b; half_t* out; int n; } proj[kMaxRowChainProj];
};
// Backward: the gradient at the last LayerNorm's output is dx, or head_a head_w + dy_in if head_k (the columns of head_a); LayerNorm a; if F: the
// feed-forward sub-layer and LayerNorm b; then dO = dsub wo.  `dsub` of a LayerNorm may be where ITS sub-layer's predecessor in the order of the backward pass
// (LayerNorm a for b) has its `sub`, dy_out where dy_in is.  dy_out null: not wanted (without dropout it is dsub).
struct RowChainLnBwd {
  const half_t *sub, *resid, *gamma;
  const float* stats;
  half_t* dsub;
  float* partial;     // row_chain_blocks(rows) partial rows of 3 d
  DropDev drop;
};
struct RowChainBwd {
  int rows, F, head_k;
  const half_t *head_a, *head_w, *dy_in, *dx;
  RowChainLnBwd ln_a, ln_b;
  const half_t *w2, *h, *w1, *wo;
  half_t *dh, *dy_out, *dO;
};
bool row_chain_fits(int d, int F);
int row_chain_blocks(int rows);
int launch_row_chain_fwd(const RowChainFwd& a, int d, hipStream_t stream);
int launch_row_chain_bwd(const RowChainBwd& a, int d, hipStream_t stream);
// All products (1..kMaxWgrad of them, results times out_scale) in one launch, or two if they are cut along k.  partial: fp32 scratch for that
// (may be null: never cut).  tile, splits: 0 = chosen by cost.
// sums: partial rows of d columns (a layer's LayerNorm gradients) that are added up as well, times out_scale: in the same launch where that is one of
// small tiles.
int launch_wgrad_group(const WgradProduct* products, int n, float out_scale, float* partial, int64_t partial_floats, hipStream_t stream,
                       int tile = 0, int splits = 0, const ColumnSums* sums = nullptr, int n_sums = 0, int d = 0);
int launch_embed_fwd(const int32_t* ids, const half_t* E, half_t* x, int rows, int d, int vocab, const DropDev& drop,
                     hipStream_t stream);
int launch_softmax_xent(half_t* logits, const int32_t* targets, float* row_loss, int rows, int V, int pad_id,
                        float eps_ls, float loss_scale, float* loss_sum, int32_t* ntok, hipStream_t stream,
                        float* row_lse = nullptr, int32_t* row_target = nullptr);  // given: the loss alone; logits stay, and the rows'
                                                    // log-sum-exps and targets go there ...
int launch_softmax_grad(half_t* logits, const int32_t* row_target, float* row_lse, int rows, int V, int pad_id, float eps_ls, float loss_scale,
                        hipStream_t stream);                        // ... from which this makes the gradient, in place
int64_t colsum_scratch_floats(int cols);
int launch_colsum(const half_t* src, int ld, half_t* dst, float* partial, int rows, int cols, hipStream_t stream, float scale = 1.f);
int launch_colsum_static(const half_t* src, int ld, half_t* dst, int rows, int cols, hipStream_t stream);  // partial sums in a fixed device array
int64_t embed_bwd_scratch_ints(int vocab, int rows_total, int d);
// Embedding gradient in two parts that share `scratch`: the order of the positions by id (ids alone), then the sums.
int launch_embed_sort(const int32_t* ids_a, int rows_a, const int32_t* ids_b, int rows_b, int d, int vocab, int32_t* scratch, hipStream_t stream);
int launch_embed_sum(const half_t* dx_a, int rows_a, const DropDev& drop_a, const half_t* dx_b, int rows_b, const DropDev& drop_b, half_t* gE,
                     int d, const int32_t* scratch, hipStream_t stream, float scale = 1.f);
// flag (cleared by the caller; null: no check) is raised if a sum is inf or NaN
int launch_accumulate(const half_t* g16, float* acc, int64_t n, int first, hipStream_t stream, float mult = 1.f, int32_t* flag = nullptr);
int launch_last_accumulate_and_adam(const half_t* g16, float mult, int first, float* master, float* m, float* v, float* acc, half_t* w16, int64_t n,
                                    float lr, float b1, float b2, float eps, int t, int32_t* flag, hipStream_t stream, float grad_scale);
// in_place: acc *= inv_scale in the same pass; otherwise acc is only read
int launch_check_overflow(float* acc, int64_t n, float inv_scale, int32_t* flag, hipStream_t stream, bool in_place = true);
// *loss_total (+)= *loss, *ntok_total (+)= *ntok (first: overwrite)
int launch_add_scalars(const float* loss, const int32_t* ntok, float* loss_total, int32_t* ntok_total, int first, hipStream_t stream);
int launch_adam(float* master, float* m, float* v, const float* g, half_t* w16, int64_t n, float lr, float b1,
                float b2, float eps, int t, const int32_t* flag, hipStream_t stream, float grad_scale = 1.f);  // the update uses g * grad_scale
// Shapes of the sub-batches stacked row-wise in one pass (passed to the table kernel by value).
struct SegmentList {
  int n;
  int B[NMT_MAX_SEGMENTS], S[NMT_MAX_SEGMENTS], T[NMT_MAX_SEGMENTS];
  uint32_t micro[NMT_MAX_SEGMENTS];
};
// Row keys (uid, pos | micro << 16) of all source / target rows and the per-sentence attention
// tables (first query row, first key row, Tq, Tk) for encoder self-, decoder self- and
// encoder-decoder attention.  uid == nullptr: a sentence's id is its index within its sub-batch.
int launch_build_tables(const SegmentList& segs, int n_sent, const uint32_t* uid, uint2* rk_src, uint2* rk_tgt, int4* tab_ss,
                        int4* tab_tt, int4* tab_ts, hipStream_t stream);
// The same for sentences packed back to back (no padding): first rows come from a prefix sum of the
// lengths in `sentences`; lengths are clamped to [1, max] and to the row totals, so no table entry
// ever points outside [0, n_src) / [0, n_tgt).  sent_rows: scratch of 2 * n_sent ints.
int launch_build_tables_packed(const nmt_sentence* sentences, int n_sent, int n_src, int n_tgt, int max_src, int max_tgt,
                               int32_t* sent_rows, uint2* rk_src, uint2* rk_tgt, int4* tab_ss, int4* tab_tt, int4* tab_ts,
                               hipStream_t stream);
int launch_dropout_mask(uint8_t* keep, int rows, int n_cols, const DropDev& drop, hipStream_t stream);
