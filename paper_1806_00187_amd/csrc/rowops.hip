// HBM-bound row kernels of the training step: embedding (+positions, dropout), fused
// residual + dropout + LayerNorm forward / backward (one wavefront per token row), column sums
// for bias gradients, fused vocabulary softmax + label-smoothed cross-entropy + gradient, and the
// deterministic embedding-gradient reduction.
#include <math.h>

#include <mutex>

#include "common.h"

namespace {

constexpr int kThreads = 256;
constexpr int kWavesPerBlock = kThreads / kWave;

__device__ __forceinline__ void unpack8(const half8_t h, float (&f)[8]) {
#pragma unroll
  for (int e = 0; e < 8; ++e) f[e] = (float)h[e];
}
__device__ __forceinline__ half8_t pack8(const float (&f)[8]) {
  half8_t h;
#pragma unroll
  for (int e = 0; e < 8; ++e) h[e] = (half_t)f[e];
  return h;
}

// ------------------------------------------------------------------------------------------------
// Embedding forward: x = dropout(sqrt(d) * E[id] + PE(pos)); PE[t,2i] = sin(t / 10000^(2i/d)),
// PE[t,2i+1] = cos(same).  One thread per 8 columns.
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) embed_fwd_kernel(const int32_t* __restrict__ ids, const half_t* __restrict__ E,
                                                             half_t* __restrict__ x, int rows, int d, int vocab,
                                                             DropDev drop) {
  const int chunks = d >> 3;
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (gid >= (int64_t)rows * chunks) return;
  const int row = (int)(gid / chunks), c = (int)(gid % chunks);
  int id = ids[row];
  id = id < 0 ? 0 : (id >= vocab ? vocab - 1 : id);
  float v[8];
  unpack8(ld_half8(E + (size_t)id * d + c * 8), v);
  const float pos = (float)drop_row_pos(drop, (uint32_t)row);
  const float sq = sqrtf((float)d);
  const float k = -logf(10000.f) / (float)d;
#pragma unroll
  for (int e = 0; e < 8; e += 2) {
    const float ang = pos * expf(k * (float)(c * 8 + e));
    v[e] = v[e] * sq + sinf(ang);
    v[e + 1] = v[e + 1] * sq + cosf(ang);
  }
  if (drop.thr) {
    const uint32_t bits = drop_keep8(drop, (uint32_t)row, (uint32_t)c);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[e] = ((bits >> e) & 1u) ? v[e] * drop.scale : 0.f;
  }
  st_half8(x + (size_t)row * d + c * 8, pack8(v));
}

// ------------------------------------------------------------------------------------------------
// out = LayerNorm(resid + dropout(sub)); one wavefront per row, NCH chunks of 8 columns per lane.
// Plain loads and stores, here and backward: what these kernels read the product before has just written, and the next one reads
// what they write.  With streaming forms (no retention asked for) whole updates took, start / now in us: 2 x 1400 positions x 256
// 1370 / 1295, 3000 x 512 3830 / 3780; 3000 to 17700 x 1024 the same within 0.5 %.  (The kernels themselves, on one stream, take up to 10 % longer at
// 3000 to 30000 rows -- 6000 x 512, five calls forward: 28.5 / 30.2 us --; of whole passes of 550 sizes and widths on one stream none was slower by more than 0.3 %.)
// ------------------------------------------------------------------------------------------------
// kKeyedRows: there are row keys (passes of a model have them; without, a branch stands between a row's key and its other loads).  kFullRows: and rows
// of 512 NCH columns (no branch around any load, so that the draws run while the row is on its way, and divisions by a power of two).  With that,
// and the arguments asked for together, forward passes, us: 3100 x 512 1225 -> 1185, 380 x 1024 985 -> 947, 3000 x 1024 2277 -> 2229.
enum RowForm { kAnyRows, kKeyedRows, kFullRows };
RowForm row_form(const DropDev& drop, int d, int nch) { return !drop.rowkey ? kAnyRows : d == 512 * nch ? kFullRows : kKeyedRows; }

template <int NCH, RowForm FORM>
__device__ __forceinline__ void load_presum(float (&y)[NCH][8], const half_t* __restrict__ sub,
                                            const half_t* __restrict__ resid, int row, int d, int lane,
                                            const DropDev& drop) {
  constexpr bool KEYED = FORM != kAnyRows, FULL = FORM == kFullRows;
  const int chunks = d >> 3;
  half8_t hs[NCH], hr[NCH];  // everything the row needs is requested before anything is used, its key first, which the draws begin with
  uint2 rk = {};
  if constexpr (KEYED) rk = drop.rowkey[row];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + kWave * i;
    hs[i] = FULL || c < chunks ? ld_half8(sub + (size_t)row * d + c * 8) : zero_half8();
    hr[i] = FULL || c < chunks ? ld_half8(resid + (size_t)row * d + c * 8) : zero_half8();
  }
  DropRow key = {};
  if constexpr (KEYED) key = drop_row_of(drop, rk);
  else if (drop.thr) key = drop_row(drop, (uint32_t)row);
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const uint32_t bits = drop.thr ? drop_keep8(drop, key, (uint32_t)(lane + kWave * i)) : 0xFFu;
#pragma unroll
    for (int e = 0; e < 8; ++e) y[i][e] = (float)hr[i][e] + (((bits >> e) & 1u) ? (float)hs[i][e] * drop.scale : 0.f);
  }
}

template <int NCH, RowForm FORM>
__global__ void __launch_bounds__(kThreads) res_ln_fwd_kernel(const half_t* __restrict__ sub, const half_t* __restrict__ resid,
                                                              const half_t* __restrict__ gamma, const half_t* __restrict__ beta,
                                                              half_t* __restrict__ out, float* __restrict__ stats, int rows,
                                                              int d_in, float eps, DropDev drop, Ahead next) {
  constexpr bool FULL = FORM == kFullRows;
  const int d = FULL ? 512 * NCH : d_in;
  touch_arguments<64 + sizeof(DropDev) + sizeof(Ahead)>();
  if (blockIdx.x >= next.first) {
    ask_ahead(next, (int)(blockIdx.x - next.first));
    return;
  }
  const int lane = threadIdx.x & 63;
  const int row = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int chunks = d >> 3;
  float y[NCH][8];
  half8_t gam[NCH], bet[NCH];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + kWave * i;
    gam[i] = FULL || c < chunks ? ld_half8(gamma + c * 8) : zero_half8();
    bet[i] = FULL || c < chunks ? ld_half8(beta + c * 8) : zero_half8();
  }
  load_presum<NCH, FORM>(y, sub, resid, row, d, lane, drop);
  float s = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
#pragma unroll
    for (int e = 0; e < 8; ++e) s += y[i][e];
  const float mean = wave_sum(s) / (float)d;
  float q = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i)
    if (FULL || lane + kWave * i < chunks) {
#pragma unroll
      for (int e = 0; e < 8; ++e) q += (y[i][e] - mean) * (y[i][e] - mean);
    }
  const float rstd = 1.0f / sqrtf(wave_sum(q) / (float)d + eps);
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = lane + kWave * i;
    if (FULL || c < chunks) {
      float o[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (y[i][e] - mean) * rstd * (float)gam[i][e] + (float)bet[i][e];
      st_half8(out + (size_t)row * d + c * 8, pack8(o));
    }
  }
  if (lane == 0) {
    stats[2 * row] = mean;
    stats[2 * row + 1] = rstd;
  }
}

// Backward.  Each wavefront walks groups of ROWS rows (their loads are all issued before anything is
// computed), keeps per-lane column sums for dgamma, dbeta and the bias gradient in registers, and the block
// writes one partial row of d floats per quantity.  The three inputs of a row stay in
// registers as the fp16 values they were loaded as and are widened where they are used (twice: row statistics,
// then the result), which keeps the kernel at four wavefronts per SIMD.
constexpr int kLnBwdMaxBlocks = 1024;

template <int NCH, int ROWS, int WAVES, RowForm FORM>
__global__ void __launch_bounds__(64 * WAVES) res_ln_bwd_kernel(const half_t* __restrict__ dout, const half_t* __restrict__ sub,
                                                              const half_t* __restrict__ resid, const half_t* __restrict__ gamma,
                                                              const float* __restrict__ stats, half_t* __restrict__ dy_out,
                                                              half_t* __restrict__ dym_out, float* __restrict__ partial, int rows,
                                                              int d_in, DropDev drop, Ahead next) {
  constexpr bool KEYED = FORM != kAnyRows, FULL = FORM == kFullRows;
  const int d = FULL ? 512 * NCH : d_in;
  extern __shared__ __align__(16) float red[];  // [WAVES][NCH][2][64 lanes][4]
  touch_arguments<72 + sizeof(DropDev) + sizeof(Ahead)>();
  if (blockIdx.x >= next.first) {
    ask_ahead(next, (int)(blockIdx.x - next.first));
    return;
  }
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int chunks = d >> 3;
  float sg[NCH][8], sb[NCH][8], sbias[NCH][8];
  half8_t gam[NCH];
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    gam[i] = FULL || lane + kWave * i < chunks ? ld_half8(gamma + (lane + kWave * i) * 8) : zero_half8();
#pragma unroll
    for (int e = 0; e < 8; ++e) sg[i][e] = sb[i][e] = sbias[i][e] = 0.f;
  }
  for (int row0 = (blockIdx.x * WAVES + wave) * ROWS; row0 < rows; row0 += next.first * WAVES * ROWS) {
    half8_t hs[ROWS][NCH], hr[ROWS][NCH], hg[ROWS][NCH];
    uint32_t bits[ROWS][NCH];
    DropRow key[ROWS] = {};
    uint2 rk[ROWS];
    if constexpr (KEYED) {
#pragma unroll
      for (int u = 0; u < ROWS; ++u) rk[u] = drop.rowkey[min(row0 + u, rows - 1)];
    }
    float mean[ROWS], rstd[ROWS], s1[ROWS], s2[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int row = min(row0 + u, rows - 1);  // a row past the end repeats the last one and is not written
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int c = lane + kWave * i;
        const bool in = FULL || c < chunks;
        hs[u][i] = in ? ld_half8(sub + (size_t)row * d + c * 8) : zero_half8();
        hr[u][i] = in ? ld_half8(resid + (size_t)row * d + c * 8) : zero_half8();
        hg[u][i] = in ? ld_half8(dout + (size_t)row * d + c * 8) : zero_half8();
      }
      mean[u] = stats[2 * row];
      rstd[u] = stats[2 * row + 1];
      if (!KEYED && drop.thr) key[u] = drop_row(drop, (uint32_t)row);
    }
    if constexpr (KEYED) {
#pragma unroll
      for (int u = 0; u < ROWS; ++u) key[u] = drop_row_of(drop, rk[u]);
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
#pragma unroll
      for (int i = 0; i < NCH; ++i) bits[u][i] = drop.thr ? drop_keep8(drop, key[u], (uint32_t)(lane + kWave * i)) : 0xFFu;
    // normalised value of element e of chunk i of row u (the pre-normalisation sum is formed in fp32, as in the forward pass)
    auto xhat = [&](int u, int i, int e) {
      const float y = (float)hr[u][i][e] + (((bits[u][i] >> e) & 1u) ? (float)hs[u][i][e] * drop.scale : 0.f);
      return (y - mean[u]) * rstd[u];
    };
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const bool live = row0 + u < rows;
      s1[u] = s2[u] = 0.f;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        if (FULL || lane + kWave * i < chunks) {
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float xh = xhat(u, i, e), go = (float)hg[u][i][e];
            ln_bwd_row_sums(s1[u], s2[u], go, (float)gam[i][e], xh);
            if (live) {
              sg[i][e] += go * xh;
              sb[i][e] += go;
            }
          }
        }
      }
    }
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      s1[u] = wave_sum(s1[u]);
      s2[u] = wave_sum(s2[u]);
    }
    // (the widened copies of the first pass are not kept: the inputs are widened again from their fp16 registers)
#pragma unroll
    for (int u = 0; u < ROWS; ++u)
#pragma unroll
      for (int i = 0; i < NCH; ++i) asm volatile("" : "+v"(hs[u][i]), "+v"(hr[u][i]), "+v"(hg[u][i]));
#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
      const int row = row0 + u;
      if (row >= rows) break;
      const float m1 = s1[u] / (float)d, m2 = s2[u] / (float)d;
#pragma unroll
      for (int i = 0; i < NCH; ++i) {
        const int c = lane + kWave * i;
        if (FULL || c < chunks) {
          float dy[8], dm[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            dy[e] = ln_bwd_dy((float)hg[u][i][e], (float)gam[i][e], xhat(u, i, e), rstd[u], m1, m2);
            dm[e] = ((bits[u][i] >> e) & 1u) ? dy[e] * drop.scale : 0.f;
            sbias[i][e] += dm[e];
          }
          st_half8(dy_out + (size_t)row * d + c * 8, pack8(dy));
          if (dym_out) st_half8(dym_out + (size_t)row * d + c * 8, pack8(dm));
        }
      }
    }
  }
  // block reduction, one quantity after the other: every wavefront leaves its sums in LDS, then each thread adds four columns up over the
  // wavefronts, in their order.  (All three at a time would take LDS that the other stream's products do not leave.)
  floatx4 *red4 = reinterpret_cast<floatx4*>(red), *dst = reinterpret_cast<floatx4*>(partial + (size_t)blockIdx.x * 3 * d);
  const int quads = d >> 2;
  constexpr int SHARE = (NCH * 128 + 64 * WAVES - 1) / (64 * WAVES);  // groups of four columns to a thread
  floatx4 total[3][SHARE];
#pragma unroll
  for (int q = 0; q < 3; ++q) {
    if (q) __syncthreads();
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      const float(&src)[8] = q == 0 ? sg[i] : (q == 1 ? sb[i] : sbias[i]);
      floatx4* at = red4 + (wave * NCH + i) * 128 + lane;  // (the low and the high four columns of the lanes apart: every bank once)
      at[0] = floatx4{src[0], src[1], src[2], src[3]};
      at[64] = floatx4{src[4], src[5], src[6], src[7]};
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < SHARE; ++r) {
      const int i = (int)threadIdx.x + r * 64 * WAVES;
      const floatx4* at = red4 + (i >> 7) * 128 + (i & 1) * 64 + ((i >> 1) & 63);
      if (i >= quads) continue;
      total[q][r] = at[0];
#pragma unroll
      for (int w = 1; w < WAVES; ++w) total[q][r] += at[w * NCH * 128];
    }
  }
#pragma unroll
  for (int q = 0; q < 3; ++q)  // (stored at the end: a barrier waits for the stores before it)
#pragma unroll
    for (int r = 0; r < SHARE; ++r)
      if (const int i = (int)threadIdx.x + r * 64 * WAVES; i < quads) dst[q * quads + i] = total[q][r];
}

// A layer's LayerNorm gradients are leaves like its weight gradients, so their two or three sums wait for the layer's
// end and run on the second stream in place of a 3-6 us launch each in the chain of input gradients (whole updates of
// 3000 positions x 512: 4.31 -> 4.18 ms); beside small weight gradients they are part of those' launch.
constexpr int kFinThreads = 1024;
__global__ void __launch_bounds__(kFinThreads) finalize_partials_kernel(const FinalizeArgs a) {
  __shared__ float red[32 * 33];
  finalize_columns<kFinThreads>(a, blockIdx.x, red);
}
int launch_finalize(const ColumnSums* in, int n, int nq, int cols, int pitch, float scale, hipStream_t stream) {
  NMT_REQUIRE(in && n >= 1 && n <= kMaxColumnSums, "column sums: %d buffers outside [1, %d]", n, kMaxColumnSums);
  FinalizeArgs a = {};
  a.nq = nq;
  a.cols = cols;
  a.pitch = pitch;
  a.scale = scale;
  for (int i = 0; i < n; ++i) a.in[i] = in[i];
  hipLaunchKernelGGL(finalize_partials_kernel, dim3(n * nq * ceil_div(cols, 32)), dim3(kFinThreads), 0, stream, a);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

// ------------------------------------------------------------------------------------------------
// Column sums of an fp16 matrix (bias gradients): grid (column blocks of 512, row splits).
// ------------------------------------------------------------------------------------------------
constexpr int kColsumMaxSplits = 512;

__global__ void __launch_bounds__(kThreads) colsum_kernel(const half_t* __restrict__ src, int ld, float* __restrict__ partial,
                                                          int rows, int cols) {
  __shared__ float red[kWavesPerBlock][512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int col = blockIdx.x * 512 + lane * 8;
  const int nsplit = gridDim.y;
  const int per = (rows + nsplit - 1) / nsplit;
  const int r0 = blockIdx.y * per, r1 = min(rows, r0 + per);
  float s[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  if (col < cols) {
    int r = r0 + wave;
    for (; r + 3 * kWavesPerBlock < r1; r += 4 * kWavesPerBlock) {  // four independent loads in flight
      half8_t h[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) h[u] = ld_half8_nt(src + (size_t)(r + u * kWavesPerBlock) * ld + col);
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        float v[8];
        unpack8(h[u], v);
#pragma unroll
        for (int e = 0; e < 8; ++e) s[e] += v[e];
      }
    }
    for (; r < r1; r += kWavesPerBlock) {
      float v[8];
      unpack8(ld_half8(src + (size_t)r * ld + col), v);
#pragma unroll
      for (int e = 0; e < 8; ++e) s[e] += v[e];
    }
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) red[wave][lane * 8 + e] = s[e];
  __syncthreads();
  if (wave == 0 && col < cols) {
#pragma unroll
    for (int e = 0; e < 8; ++e)
      partial[(size_t)blockIdx.y * cols + col + e] = red[0][lane * 8 + e] + red[1][lane * 8 + e] + red[2][lane * 8 + e] + red[3][lane * 8 + e];
  }
}

// ------------------------------------------------------------------------------------------------
// Fused softmax + label-smoothed cross-entropy + gradient; one block per row, the row held in
// registers (NCH chunks of 8 logits per thread).  A pass without training needs the loss alone: the row is read and not
// written back (26000 x 32768: 591 -> 297 us; the written half was the gradient), and its log-sum-exp and target are kept in case a
// backward pass is asked for after all, which then forms the same gradient from them (the caller's targets may be gone by then).
// ------------------------------------------------------------------------------------------------
__device__ __forceinline__ float block_reduce(float v, bool is_max, float* sh) {
  v = is_max ? wave_max(v) : wave_sum(v);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  __syncthreads();
  if (lane == 0) sh[wave] = v;
  __syncthreads();
  float r = sh[0];
#pragma unroll
  for (int w = 1; w < kWavesPerBlock; ++w) r = is_max ? fmaxf(r, sh[w]) : r + sh[w];
  return r;
}

enum XentForm { kLossAndGrad, kLossOnly, kGradOnly };
template <int NCH, XentForm FORM>
__global__ void __launch_bounds__(kThreads) softmax_xent_kernel(half_t* __restrict__ logits, const int32_t* __restrict__ targets,
                                                                float* __restrict__ row_loss, float* __restrict__ row_lse,
                                                                int32_t* __restrict__ row_target, int V, int pad_id, float eps_ls,
                                                                float loss_scale) {
  __shared__ float sh[kWavesPerBlock];
  const int row = blockIdx.x;
  const int chunks = V >> 3;
  half_t* z = logits + (size_t)row * V;
  const int y = targets[row];
  if constexpr (FORM == kLossOnly)
    if (threadIdx.x == 0) row_target[row] = y;
  if (y == pad_id) {  // padding positions contribute neither loss nor gradient
    if constexpr (FORM != kLossOnly)
      for (int c = threadIdx.x; c < chunks; c += kThreads) st_half8(z + c * 8, zero_half8());
    if constexpr (FORM != kGradOnly)
      if (threadIdx.x == 0) row_loss[row] = 0.f;
    return;
  }
  // The row stays in registers as fp16.  Pass 1 (maximum, plain sum) runs on pairs of halfs; the two
  // exponential passes fold the shift and the scale into one fused multiply-add in front of the base-2
  // exponential: exp(z - m) = 2^(z log2e - m log2e), loss_scale * exp(z - lse) = 2^(z log2e - lse log2e + log2 loss_scale).
  typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
  struct Pairs { half2_t p[4]; };
  constexpr float kLog2e = 1.4426950408889634f;
  half8_t reg[NCH];
  half2_t mx2 = {(_Float16)-INFINITY, (_Float16)-INFINITY};
  const half2_t ones = {(_Float16)1.f, (_Float16)1.f};
  float sz = 0.f;
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = threadIdx.x + kThreads * i;
    if (c < chunks) {
      reg[i] = ld_half8_nt(z + c * 8);
      const Pairs h = __builtin_bit_cast(Pairs, reg[i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        mx2 = __builtin_elementwise_max(mx2, h.p[e]);
        sz = __builtin_amdgcn_fdot2(h.p[e], ones, sz, false);
      }
    }
  }
  const int yc = min(max(y, 0), V - 1);
  float lse;
  if constexpr (FORM == kGradOnly) {
    lse = row_lse[row];
  } else {
    const float zy = (float)z[yc];
    const float mx = block_reduce(fmaxf((float)mx2[0], (float)mx2[1]), true, sh);
    const float shift = -mx * kLog2e;
    float se = 0.f;
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
      if (threadIdx.x + kThreads * i < chunks) {
#pragma unroll
        for (int e = 0; e < 8; ++e) se += __builtin_amdgcn_exp2f(fmaf((float)reg[i][e], kLog2e, shift));
      }
    }
    se = block_reduce(se, false, sh);
    sz = block_reduce(sz, false, sh);
    lse = mx + logf(se);
    if (threadIdx.x == 0) row_loss[row] = lse - (1.f - eps_ls) * zy - (eps_ls / (float)V) * sz;
    if constexpr (FORM == kLossOnly) {
      if (threadIdx.x == 0) row_lse[row] = lse;
      return;
    }
  }
  const float q_scaled = loss_scale * eps_ls / (float)V, hit = loss_scale * (1.f - eps_ls);
  const float shift2 = -lse * kLog2e + log2f(loss_scale);
#pragma unroll
  for (int i = 0; i < NCH; ++i) {
    const int c = threadIdx.x + kThreads * i;
    if (c < chunks) {
      float g[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) g[e] = __builtin_amdgcn_exp2f(fmaf((float)reg[i][e], kLog2e, shift2)) - q_scaled;
      if (c == (yc >> 3)) {
#pragma unroll
        for (int e = 0; e < 8; ++e)
          if (e == (yc & 7)) g[e] -= hit;
      }
      half8_t o;
#pragma unroll
      for (int e = 0; e < 8; ++e) o[e] = (half_t)g[e];
      st_half8_nt(z + c * 8, o);
    }
  }
}

// loss_sum = sum of row losses (fixed order), ntok = number of non-pad targets; single block.
__global__ void __launch_bounds__(1024) loss_reduce_kernel(const float* __restrict__ row_loss, const int32_t* __restrict__ targets,
                                                           int rows, int pad_id, float* loss_sum, int32_t* ntok) {
  __shared__ float sl[1024];
  __shared__ int sn[1024];
  float s = 0.f;
  int n = 0;
  for (int r = threadIdx.x; r < rows; r += 1024) {
    s += row_loss[r];
    n += targets[r] != pad_id;
  }
  sl[threadIdx.x] = s;
  sn[threadIdx.x] = n;
  __syncthreads();
  for (int o = 512; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      sl[threadIdx.x] += sl[threadIdx.x + o];
      sn[threadIdx.x] += sn[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *loss_sum = sl[0];
    *ntok = sn[0];
  }
}

// ------------------------------------------------------------------------------------------------
// Embedding backward.  The token positions of both id streams are sorted by id with a stable two-pass
// radix sort (8 bits per pass), so every vocabulary row's positions are contiguous and in increasing
// order.  The sorted list is cut into segments of kEmbSeg entries; one block per segment sums the
// gradient rows of each run of equal ids.  A run that holds all positions of its id is added to the
// row of the shared matrix at once; runs of ids that spill over segment borders leave fp32 partial
// sums, which a second kernel adds up in a fixed order.  The order of every sum is fixed, so results
// do not depend on scheduling.  Where a run begins and ends is read off the sorted ids themselves.
// The sort needs the ids alone: the backward pass enqueues it beside its first products, and only the
// two summing kernels are left for the end.
// ------------------------------------------------------------------------------------------------
constexpr int kEmbSeg = 16;          // sorted entries per block of the row-summing kernel
constexpr int kSortPerBlock = 1024;  // entries per block of a radix pass

__device__ __forceinline__ int clamp_id(int id, int vocab) { return id < 0 ? 0 : (id >= vocab ? vocab - 1 : id); }
__device__ __forceinline__ int id_at(const int32_t* a, int na, const int32_t* b, int i, int vocab) {
  return clamp_id(i < na ? a[i] : b[i - na], vocab);
}
// Exclusive scan over the block's 1024 threads; `total` is the sum of all.
__device__ __forceinline__ int block_scan_1024(int v, int* sh, int& total) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  int s = v;
#pragma unroll
  for (int o = 1; o < kWave; o <<= 1) {
    const int u = __shfl_up(s, o, kWave);
    if (lane >= o) s += u;
  }
  if (lane == 63) sh[wave] = s;
  __syncthreads();
  int before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < 16; ++w) {
    const int x = sh[w];
    before += w < wave ? x : 0;
    total += x;
  }
  __syncthreads();
  return before + s - v;
}
// exclusive scan of cnt[0..n) in place, n a multiple of 4; single block of 1024 threads, 4 entries per thread at a time
__global__ void __launch_bounds__(1024) radix_scan_kernel(int32_t* cnt, int n) {
  __shared__ int sh[16];
  int run = 0;
  for (int base = 0; base < n; base += 4096) {
    const int i = base + (int)threadIdx.x * 4;
    int4 c = make_int4(0, 0, 0, 0);
    if (i < n) c = *reinterpret_cast<const int4*>(cnt + i);
    int total;
    const int at = run + block_scan_1024(c.x + c.y + c.z + c.w, sh, total);
    if (i < n) *reinterpret_cast<int4*>(cnt + i) = make_int4(at, at + c.x, at + c.x + c.y, at + c.x + c.y + c.z);
    run += total;
  }
}

// Lanes of the wavefront that hold the same 8-bit digit as this one (among those with `valid`).
__device__ __forceinline__ unsigned long long same_digit(int digit, bool valid) {
  unsigned long long peers = __ballot(valid);
#pragma unroll
  for (int bit = 0; bit < 8; ++bit) {
    const unsigned long long set = __ballot((digit >> bit) & 1);
    peers &= ((digit >> bit) & 1) ? set : ~set;
  }
  return peers;
}
// The whole sort in one block, for lists that fit its LDS as (id << 16 | position) words: six launches
// of about 4 us each, whatever their work, become one (5 us at 260 entries, 23 us at 6000).  Each of
// the sixteen wavefronts owns a contiguous run of the list and its own counters, so it ranks its entries
// without waiting for the others; counters are scanned digit by digit, wavefront by wavefront, which keeps
// the sort stable.
constexpr int kSmallSort = 16384;
constexpr size_t kSmallSortLds = (size_t)2 * kSmallSort * sizeof(uint32_t) + 16 * 256 * sizeof(int);
__global__ void __launch_bounds__(1024) emb_sort_small_kernel(const int32_t* a, int na, const int32_t* b, int vocab, int n,
                                                              int32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out) {
  extern __shared__ __align__(16) uint32_t sort_lds[];
  __shared__ int sh[16];
  uint32_t *from = sort_lds, *to = sort_lds + kSmallSort;
  int* hist = reinterpret_cast<int*>(sort_lds + 2 * kSmallSort);  // [256 digits][16 wavefronts]
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int per = ((n + 16 * kWave - 1) / (16 * kWave)) * kWave, lo = min(n, wave * per), hi = min(n, lo + per);
  for (int i = threadIdx.x; i < n; i += 1024) from[i] = (uint32_t)id_at(a, na, b, i, vocab) << 16 | (uint32_t)i;
  for (int pass = 0; pass < 2; ++pass) {
    const int shift = 16 + 8 * pass;
    for (int i = threadIdx.x; i < 4096; i += 1024) hist[i] = 0;
    __syncthreads();
    for (int i = lo + lane; i < hi; i += kWave) atomicAdd(&hist[((from[i] >> shift) & 255u) * 16 + wave], 1);
    __syncthreads();
    int4* h4 = reinterpret_cast<int4*>(hist) + threadIdx.x;
    const int4 c = *h4;
    int total;
    const int at = block_scan_1024(c.x + c.y + c.z + c.w, sh, total);
    *h4 = make_int4(at, at + c.x, at + c.x + c.y, at + c.x + c.y + c.z);
    __syncthreads();
    for (int i0 = lo; i0 < hi; i0 += kWave) {
      const bool valid = i0 + lane < hi;
      const uint32_t e = valid ? from[i0 + lane] : 0u;
      const int digit = (int)((e >> shift) & 255u);
      const unsigned long long peers = same_digit(digit, valid);
      if (valid) {
        const int rank = __popcll(peers & ((1ull << lane) - 1ull));
        const int first = hist[digit * 16 + wave];
        to[first + rank] = e;
        if (rank == 0) hist[digit * 16 + wave] = first + __popcll(peers);  // (every peer has read it: lock-step)
      }
    }
    __syncthreads();
    uint32_t* t = from;
    from = to;
    to = t;
  }
  for (int i = threadIdx.x; i < n; i += 1024) {
    keys_out[i] = (int32_t)(from[i] >> 16);
    vals_out[i] = (int32_t)(from[i] & 0xFFFFu);
  }
}

// One radix pass over (key, value) pairs; pass 0 takes key = id of position i, value = i.
// Histogram: hist[digit * nblk + block] = number of the block's entries with that digit, so that an
// exclusive scan of the whole array gives each (digit, block) its first output slot.
__global__ void __launch_bounds__(kThreads) radix_hist_kernel(const int32_t* a, int na, const int32_t* b, int vocab,
                                                              const int32_t* __restrict__ keys, int n, int shift, int nblk,
                                                              int32_t* __restrict__ hist) {
  __shared__ int h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  const int base = blockIdx.x * kSortPerBlock;
  for (int r = 0; r < kSortPerBlock / kThreads; ++r) {
    const int i = base + r * kThreads + threadIdx.x;
    if (i < n) atomicAdd(&h[((keys ? keys[i] : id_at(a, na, b, i, vocab)) >> shift) & 255], 1);
  }
  __syncthreads();
  hist[threadIdx.x * nblk + blockIdx.x] = h[threadIdx.x];
}
// Stable scatter: entries keep their order within a digit.  The block's four wavefronts take turns;
// within a wavefront the lanes holding the same digit are found with eight ballots.
__global__ void __launch_bounds__(kThreads) radix_scatter_kernel(const int32_t* a, int na, const int32_t* b, int vocab,
                                                                 const int32_t* __restrict__ keys, const int32_t* __restrict__ vals,
                                                                 int n, int shift, int nblk, const int32_t* __restrict__ offs,
                                                                 int32_t* __restrict__ keys_out, int32_t* __restrict__ vals_out) {
  __shared__ int next[256];
  next[threadIdx.x] = offs[threadIdx.x * nblk + blockIdx.x];
  __syncthreads();
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int base = blockIdx.x * kSortPerBlock;
  for (int r = 0; r < kSortPerBlock / kThreads; ++r) {
    const int i = base + r * kThreads + threadIdx.x;
    const bool valid = i < n;
    const int key = valid ? (keys ? keys[i] : id_at(a, na, b, i, vocab)) : 0;
    const int val = valid ? (vals ? vals[i] : i) : 0;
    const int digit = (key >> shift) & 255;
    for (int w = 0; w < kThreads / kWave; ++w) {
      if (wave == w) {
        const unsigned long long peers = same_digit(digit, valid);
        if (valid) {
          const int rank = __popcll(peers & ((1ull << lane) - 1ull));
          const int slot = next[digit] + rank;
          keys_out[slot] = key;
          vals_out[slot] = val;
          if (rank == 0) next[digit] += __popcll(peers);   // every peer has read next[digit] (lock-step) before this write
        }
      }
      __syncthreads();
    }
  }
}

__device__ __forceinline__ void emb_add(half_t* __restrict__ dst, const half8_t row, int d, const float (&tot)[8], float scale) {
  float cur[8];
  unpack8(row, cur);
  const float sq = sqrtf((float)d) * scale;
#pragma unroll
  for (int e = 0; e < 8; ++e) cur[e] += sq * tot[e];
  st_half8(dst, pack8(cur));
}

// One block per segment of kEmbSeg sorted entries.
// part[(2 * seg + 0) * d ..]: sum of the segment's first run if that run began in an earlier segment;
// part[(2 * seg + 1) * d ..]: sum of its last run if that run began here and goes on in the next one.
// Bound by latency (a few hundred thousand columns in all): a position, its gradient row and row key, the dropout draws, the sum.
// The draws are ten rounds of dependent multiplies for eight columns, so the entries of a segment are shared out: a group of d / 8
// threads takes every groups-th entry (AHEAD of them, all requested together) and leaves the row after dropout in LDS; then
// the first group adds the entries up in the order of the list, a thread per eight columns.  The ids are the same for the whole
// block and come with one load; EARLY: the table rows of runs that end here are asked for beside the gradient rows.
// emb_segment_columns_kernel (a thread per eight columns draws for all sixteen entries) and this one, us: 260 entries x 64 16.2 / 6.5,
// 2800 x 256 16.7 / 6.8, 6600 x 512 15.0 / 8.0, 27000 x 512 18.6 / 16.9.
template <int THREADS, int AHEAD, bool EARLY>
__global__ void __launch_bounds__(THREADS) emb_segment_kernel(const half_t* __restrict__ dxa, int na, DropDev da,
                                                           const half_t* __restrict__ dxb, DropDev db, half_t* __restrict__ gE, int n,
                                                           int d, const int32_t* __restrict__ keys, const int32_t* __restrict__ perm,
                                                           float* __restrict__ part, float scale) {
  extern __shared__ __align__(16) half_t s_row[];  // [kEmbSeg][d]
  __shared__ float s_scale[kEmbSeg];
  const int e0 = blockIdx.x * kEmbSeg, cnt = min(kEmbSeg, n - e0);
  const int chunks = d >> 3, groups = THREADS / chunks, g = (int)threadIdx.x / chunks, c = (int)threadIdx.x - g * chunks;
  const int lane = (int)threadIdx.x & 63, before = keys[max(0, min(e0 - 1 + min(lane, kEmbSeg + 1), n - 1))];
  int pos[AHEAD];
  half8_t x[AHEAD];
  uint2 rk[AHEAD];
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) pos[u] = perm[min(e0 + min(g + u * groups, kEmbSeg - 1), n - 1)];  // (one past the end repeats another)
  const bool keyed = da.rowkey && db.rowkey;  // (in a pass of the training step; without row keys: rows of one rectangular batch)
  auto row_of = [&](int u) { return pos[u] < na ? pos[u] : pos[u] - na; };
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
    x[u] = ld_half8((pos[u] < na ? dxa : dxb) + (size_t)row_of(u) * d + c * 8);
  }
  if (keyed) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) rk[u] = (pos[u] < na ? da.rowkey : db.rowkey)[row_of(u)];
  } else {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const DropDev& dd = pos[u] < na ? da : db;
      const DropRow row = dd.thr ? drop_row(dd, (uint32_t)row_of(u)) : DropRow{};
      rk[u] = make_uint2(row.uid, row.pos | (row.c3 & 0xFFu) << 16);
    }
  }
  // the ids of the entries before, in and behind the segment (-1: none), the same in every lane
  int key[kEmbSeg + 2];
#pragma unroll
  for (int u = 0; u < kEmbSeg + 2; ++u) {
    const int i = e0 - 1 + u, k = __builtin_amdgcn_readlane(before, u);
    key[u] = i >= 0 && i < n ? k : -1;
  }
  // the table's rows of runs that end here (of runs that began earlier the next kernel takes care); the others' requests lie outside the extent
  const __amdgpu_buffer_rsrc_t to = __builtin_amdgcn_make_buffer_rsrc(gE, 0, 0x7FFFFFFF, 0x00020000);
  const bool sums = g == 0;  // (the threads of the first group add up, eight columns each: c is their chunk)
  auto table_row = [&](int u) {
    const bool ends = key[u + 1] != key[u + 2] && key[u + 1] != key[0] && key[u + 1] >= 0;
    const uint32_t at = ((uint32_t)key[u + 1] * (uint32_t)d + (uint32_t)c * 8u) * 2u;
    return __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(to, (int)(ends && sums ? at : 0x80000000u), 0, 0));
  };
  half8_t table[kEmbSeg];
  if constexpr (EARLY) {
#pragma unroll
    for (int u = 0; u < kEmbSeg; ++u) table[u] = table_row(u);
  }
  if (da.thr || db.thr) {
#pragma unroll
    for (int u = 0; u < AHEAD; ++u) {
      const DropDev& dd = pos[u] < na ? da : db;
      const uint32_t bits = drop_keep8(dd, drop_row_of(dd, rk[u]), (uint32_t)c);  // (a threshold of 0 keeps all)
#pragma unroll
      for (int e = 0; e < 8; ++e) x[u][e] = (bits >> e) & 1u ? x[u][e] : (half_t)0;
    }
  }
#pragma unroll
  for (int u = 0; u < AHEAD; ++u) {
    const int k = g + u * groups;
    if (g < groups && k < kEmbSeg) {
      st_half8(s_row + (size_t)k * d + c * 8, x[u]);
      if (c == 0) s_scale[k] = pos[u] < na ? (da.thr ? da.scale : 1.f) : (db.thr ? db.scale : 1.f);
    }
  }
  __syncthreads();
  if (!sums) return;
  if constexpr (!EARLY) {
#pragma unroll
    for (int u = 0; u < kEmbSeg; ++u) table[u] = table_row(u);
  }
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
  for (int u = 0; u < kEmbSeg; ++u) {
    if (u < cnt) {
      const half8_t in = ld_half8(s_row + (size_t)u * d + c * 8);
      const float sc = s_scale[u];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += (float)in[e] * sc;
      const bool goes_on = key[u + 2] == key[u + 1], came_in = key[u + 1] == key[0];
      if (!goes_on || u + 1 == cnt) {
        if (!came_in && !goes_on) {
          emb_add(gE + (size_t)key[u + 1] * d + c * 8, table[u], d, acc, scale);
        } else {
          floatx4* dst = reinterpret_cast<floatx4*>(part + ((size_t)2 * blockIdx.x + (came_in ? 0 : 1)) * d + c * 8);
          dst[0] = floatx4{acc[0], acc[1], acc[2], acc[3]};
          dst[1] = floatx4{acc[4], acc[5], acc[6], acc[7]};
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] = 0.f;
      }
    }
  }
}
// The same for lists so long that the blocks no longer share the chip's compute units a few at a time: one thread per 8 columns, no rows in
// LDS.  Then not the chain of one segment counts but how many are on their way at once, and a block of d / 8 threads and no LDS leaves
// room for more of them.  The gradient rows, row keys and table rows of kEmbAhead entries are requested together before any is used (94 -> 16 us at
// 6000 entries x 512 columns, 113 -> 81 us at 107000 x 1024, against a chain of dependent loads per entry).
constexpr int kEmbAhead = 8;
static_assert(kEmbSeg % kEmbAhead == 0 && kEmbSeg + 2 <= kWave, "a block's first wavefront stages the segment's ids");
__global__ void __launch_bounds__(kThreads) emb_segment_columns_kernel(const half_t* __restrict__ dxa, int na, DropDev da,
                                                               const half_t* __restrict__ dxb, DropDev db, half_t* __restrict__ gE, int n,
                                                               int d, const int32_t* __restrict__ keys, const int32_t* __restrict__ perm,
                                                               float* __restrict__ part, float scale) {
  __shared__ int s_pos[kEmbSeg], s_key[kEmbSeg + 2];  // s_key: with the entries before and after the segment (-1: none)
  __shared__ DropRow s_drop[kEmbSeg];
  const int e0 = blockIdx.x * kEmbSeg, cnt = min(kEmbSeg, n - e0);
  if (threadIdx.x < kEmbSeg + 2) {
    const int i = e0 - 1 + (int)threadIdx.x;
    s_key[threadIdx.x] = i >= 0 && i < n ? keys[i] : -1;
    if (threadIdx.x < kEmbSeg) {
      const int pos = i + 1 < n ? perm[i + 1] : 0;
      s_pos[threadIdx.x] = pos;
      if (pos < na ? da.thr : db.thr) s_drop[threadIdx.x] = drop_row(pos < na ? da : db, (uint32_t)(pos < na ? pos : pos - na));
    }
  }
  __syncthreads();
  const int c = threadIdx.x;
  if (c >= (d >> 3)) return;
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int run_begin = 0;
  for (int k0 = 0; k0 < cnt; k0 += kEmbAhead) {
    half8_t x[kEmbAhead], row[kEmbAhead];
    uint32_t bits[kEmbAhead];
    int pos[kEmbAhead], key[kEmbAhead + 1];  // the same in every lane: kept in scalar registers
#pragma unroll
    for (int u = 0; u <= kEmbAhead; ++u) key[u] = __builtin_amdgcn_readfirstlane(s_key[min(k0 + u, cnt) + 1]);
#pragma unroll
    for (int u = 0; u < kEmbAhead; ++u) {
      pos[u] = __builtin_amdgcn_readfirstlane(s_pos[min(k0 + u, cnt - 1)]);  // (an entry past the end repeats the last one and is not added)
      x[u] = ld_half8((pos[u] < na ? dxa + (size_t)pos[u] * d : dxb + (size_t)(pos[u] - na) * d) + c * 8);
      row[u] = zero_half8();
      if (key[u + 1] != key[u] && key[u] >= 0) row[u] = ld_half8(gE + (size_t)key[u] * d + c * 8);  // the run ends here: its row is needed
    }
#pragma unroll
    for (int u = 0; u < kEmbAhead; ++u) {
      const bool in_a = pos[u] < na;
      bits[u] = (in_a ? da.thr : db.thr) ? drop_keep8(in_a ? da : db, s_drop[min(k0 + u, cnt - 1)], (uint32_t)c) : 0xFFu;
    }
#pragma unroll
    for (int u = 0; u < kEmbAhead; ++u) {
      const int k = k0 + u;
      if (k >= cnt) break;
      const float sc = pos[u] < na ? (da.thr ? da.scale : 1.f) : (db.thr ? db.scale : 1.f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += ((bits[u] >> e) & 1u) ? (float)x[u][e] * sc : 0.f;
      const bool goes_on = key[u + 1] == key[u];
      if (goes_on && k + 1 < cnt) continue;
      const bool came_in = run_begin == 0 && __builtin_amdgcn_readfirstlane(s_key[0]) == key[u];
      if (!came_in && !goes_on) {
        emb_add(gE + (size_t)key[u] * d + c * 8, row[u], d, acc, scale);
      } else {
        float* dst = part + ((size_t)2 * blockIdx.x + (came_in ? 0 : 1)) * d + c * 8;
#pragma unroll
        for (int e = 0; e < 8; ++e) dst[e] = acc[e];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] = 0.f;
      run_begin = k + 1;
    }
  }
}
// Block s finishes the id whose run began in an earlier segment and ends in segment s: kEmbFinish / (d / 8)
// groups of threads stride over the run's partial sums and are added up in a fixed order.
constexpr int kEmbFinish = 1024;
__global__ void __launch_bounds__(kEmbFinish) emb_finish_kernel(half_t* __restrict__ gE, int n, int d, const int32_t* __restrict__ keys,
                                                                const float* __restrict__ part, float scale) {
  const int e0 = blockIdx.x * kEmbSeg;
  const int v = keys[e0];
  if (e0 == 0 || keys[e0 - 1] != v) return;                          // no run carried in
  if (e0 + kEmbSeg < n && keys[e0 + kEmbSeg] == v) return;           // it goes on: a later block finishes it
  // the first segment whose first entry is v, by sixty-four probes at a time (every wavefront for itself)
  int lo = 0, hi = blockIdx.x;  // keys[lo - 1 segments] < v <= keys[hi segments]; hi's first entry is v
  while (lo < hi) {
    const int step = (hi - lo + kWave - 1) / kWave, at = min(hi, lo + (int)(threadIdx.x & 63) * step);
    const int below = __popcll(__ballot(keys[at * kEmbSeg] < v));     // probes are increasing: the first `below` lie before v
    if (below == 0) { hi = lo; break; }
    const int last = lo + (below - 1) * step;                         // (a probe clamped to hi is not below v)
    hi = min(hi, last + step);
    lo = last + 1;
  }
  const int first = hi > 0 && keys[hi * kEmbSeg - 1] == v ? hi - 1 : hi;  // where the run began
  __shared__ __align__(16) float red[kEmbFinish * 8];
  const int chunks = d >> 3, groups = kEmbFinish / chunks, r = threadIdx.x / chunks, c = threadIdx.x % chunks;
  const int count = (int)blockIdx.x - first + 1;
  if (r < groups) {
    float tot[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    for (int i = r; i < count; i += groups) {
      const float* p = part + ((size_t)2 * (first + i) + (i == 0 ? 1 : 0)) * d + c * 8;
#pragma unroll
      for (int e = 0; e < 8; ++e) tot[e] += p[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) red[threadIdx.x * 8 + e] = tot[e];
  }
  __syncthreads();
  if (r != 0) return;
  float tot[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) tot[e] = red[c * 8 + e];
  for (int g = 1; g < min(groups, count); ++g) {
#pragma unroll
    for (int e = 0; e < 8; ++e) tot[e] += red[(g * chunks + c) * 8 + e];
  }
  half_t* dst = gE + (size_t)v * d + c * 8;
  emb_add(dst, ld_half8(dst), d, tot, scale);
}

__global__ void __launch_bounds__(kThreads) dropout_mask_kernel(uint8_t* keep, int rows, int n_cols, DropDev drop) {
  const int groups = (n_cols + 7) >> 3;
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (gid >= (int64_t)rows * groups) return;
  const int row = (int)(gid / groups), grp = (int)(gid % groups);
  const uint32_t bits = drop.thr ? drop_keep8(drop, (uint32_t)row, (uint32_t)grp) : 0xFFu;
  for (int e = 0; e < 8; ++e) {
    const int col = grp * 8 + e;
    if (col < n_cols) keep[(size_t)row * n_cols + col] = (bits >> e) & 1u;
  }
}

int ln_nch(int d) { return d <= 512 ? 1 : (d <= 1024 ? 2 : 4); }

}  // namespace

// ------------------------------------------------------------------------------------------------
// Row keys and sentence tables of a group of sub-batches: one wavefront per sentence, its lanes write the row keys (one thread
// per sentence wrote them one after the other: about 900 packed sentences 14 -> 4.5 us).
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) build_tables_kernel(const SegmentList sl, int n_sent, const uint32_t* __restrict__ uid,
                                                               uint2* __restrict__ rk_src, uint2* __restrict__ rk_tgt,
                                                               int4* __restrict__ tab_ss, int4* __restrict__ tab_tt,
                                                               int4* __restrict__ tab_ts) {
  const int sb = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (sb >= n_sent) return;
  int seg = 0, first = 0, src0 = 0, tgt0 = 0;  // first sentence / source row / target row of the segment
  while (seg + 1 < sl.n && sb >= first + sl.B[seg]) {
    first += sl.B[seg];
    src0 += sl.B[seg] * sl.S[seg];
    tgt0 += sl.B[seg] * sl.T[seg];
    ++seg;
  }
  const int b = sb - first, S = sl.S[seg], T = sl.T[seg];
  const int srow = src0 + b * S, trow = tgt0 + b * T;
  const uint32_t id = uid ? uid[sb] : (uint32_t)b;
  const uint32_t hi = sl.micro[seg] << 16;
  if (lane == 0) {
    tab_ss[sb] = make_int4(srow, srow, S, S);
    tab_tt[sb] = make_int4(trow, trow, T, T);
    tab_ts[sb] = make_int4(trow, srow, T, S);
  }
  for (int t = lane; t < S; t += kWave) rk_src[srow + t] = make_uint2(id, hi | (uint32_t)t);
  for (int t = lane; t < T; t += kWave) rk_tgt[trow + t] = make_uint2(id, hi | (uint32_t)t);
}

// Packed sentences: exclusive prefix sums of the clamped lengths (one block of 1024 threads) ...
__global__ void __launch_bounds__(1024) packed_rows_kernel(const nmt_sentence* __restrict__ sent, int n_sent, int max_src, int max_tgt,
                                                           int32_t* __restrict__ rows) {
  __shared__ int sh_s[1024], sh_t[1024];
  const int per = (n_sent + 1023) / 1024;
  const int lo = min(n_sent, (int)threadIdx.x * per), hi = min(n_sent, lo + per);
  int ss = 0, tt = 0;
  for (int i = lo; i < hi; ++i) {
    ss += min(max(sent[i].src_len, 1), max_src);
    tt += min(max(sent[i].tgt_len, 1), max_tgt);
  }
  sh_s[threadIdx.x] = ss;
  sh_t[threadIdx.x] = tt;
  __syncthreads();
  for (int o = 1; o < 1024; o <<= 1) {
    const int vs = (int)threadIdx.x >= o ? sh_s[threadIdx.x - o] : 0, vt = (int)threadIdx.x >= o ? sh_t[threadIdx.x - o] : 0;
    __syncthreads();
    sh_s[threadIdx.x] += vs;
    sh_t[threadIdx.x] += vt;
    __syncthreads();
  }
  int rs = sh_s[threadIdx.x] - ss, rt = sh_t[threadIdx.x] - tt;
  for (int i = lo; i < hi; ++i) {
    rows[2 * i] = rs;
    rows[2 * i + 1] = rt;
    rs += min(max(sent[i].src_len, 1), max_src);
    rt += min(max(sent[i].tgt_len, 1), max_tgt);
  }
}
// ... then one wavefront per sentence writes its table entries and row keys.
__global__ void __launch_bounds__(kThreads) packed_tables_kernel(const nmt_sentence* __restrict__ sent, int n_sent, int n_src, int n_tgt,
                                                                int max_src, int max_tgt, const int32_t* __restrict__ rows,
                                                                uint2* __restrict__ rk_src, uint2* __restrict__ rk_tgt,
                                                                int4* __restrict__ tab_ss, int4* __restrict__ tab_tt,
                                                                int4* __restrict__ tab_ts) {
  const int sb = blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (sb >= n_sent) return;
  const nmt_sentence se = sent[sb];
  // rows past the totals the host sized everything for do not exist: a sentence is cut there
  const int srow = min(rows[2 * sb], n_src - 1), trow = min(rows[2 * sb + 1], n_tgt - 1);
  const int S = min(min(max(se.src_len, 1), max_src), n_src - srow), T = min(min(max(se.tgt_len, 1), max_tgt), n_tgt - trow);
  const uint32_t hi = (se.micro_idx & 0xFFu) << 16;
  if (lane == 0) {
    tab_ss[sb] = make_int4(srow, srow, S, S);
    tab_tt[sb] = make_int4(trow, trow, T, T);
    tab_ts[sb] = make_int4(trow, srow, T, S);
  }
  for (int t = lane; t < S; t += kWave) rk_src[srow + t] = make_uint2(se.uid, hi | (uint32_t)t);
  for (int t = lane; t < T; t += kWave) rk_tgt[trow + t] = make_uint2(se.uid, hi | (uint32_t)t);
}

// ================================================================================================
// launchers
// ================================================================================================
int launch_embed_fwd(const int32_t* ids, const half_t* E, half_t* x, int rows, int d, int vocab, const DropDev& drop,
                     hipStream_t stream) {
  NMT_REQUIRE(rows > 0 && d > 0 && d % 8 == 0 && vocab > 0, "embed_fwd: bad shape rows=%d d=%d", rows, d);
  NMT_REQUIRE(ids && E && x && aligned16(E) && aligned16(x), "embed_fwd: null or misaligned pointer");
  NMT_REQUIRE(drop.n_pos > 0, "embed_fwd: positions per sentence must be positive");
  const int64_t n = (int64_t)rows * (d / 8);
  hipLaunchKernelGGL(embed_fwd_kernel, dim3(ceil_div(n, kThreads)), dim3(kThreads), 0, stream, ids, E, x, rows, d, vocab, drop);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

// The kernel of the form the rows have.
#define NMT_ROW_FORM(run, kernel, ...)                                \
  switch (row_form(drop, d, ln_nch(d))) {                             \
    case kFullRows: run(kernel<__VA_ARGS__, kFullRows>); break;       \
    case kKeyedRows: run(kernel<__VA_ARGS__, kKeyedRows>); break;     \
    default: run(kernel<__VA_ARGS__, kAnyRows>);                      \
  }
int launch_residual_layernorm_fwd(const half_t* sub, const half_t* resid, const half_t* gamma, const half_t* beta,
                                  half_t* out, float* stats, int rows, int d, float eps, const DropDev& drop,
                                  hipStream_t stream, const Ahead& next) {
  NMT_REQUIRE(rows > 0 && d >= 8 && d % 8 == 0 && d <= 2048, "layernorm: d=%d must be a multiple of 8 in [8, 2048]", d);
  NMT_REQUIRE(sub && resid && gamma && beta && out && stats, "layernorm: null pointer");
  NMT_REQUIRE(aligned16(sub) && aligned16(resid) && aligned16(gamma) && aligned16(beta) && aligned16(out), "layernorm: misaligned pointer");
  NMT_REQUIRE(!drop.thr || drop.n_pos > 0, "layernorm: positions per sentence must be positive");
  Ahead a = next;
  a.first = (uint32_t)ceil_div(rows, kWavesPerBlock);
  const dim3 grid(a.first + ahead_groups(a)), block(kThreads);
  auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, sub, resid, gamma, beta, out, stats, rows, d, eps, drop, a); };
  switch (ln_nch(d)) {
    case 1: NMT_ROW_FORM(run, res_ln_fwd_kernel, 1); break;
    case 2: NMT_ROW_FORM(run, res_ln_fwd_kernel, 2); break;
    default: NMT_ROW_FORM(run, res_ln_fwd_kernel, 4); break;
  }
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

int64_t layernorm_bwd_scratch_floats(int d) { return (int64_t)kLnBwdMaxBlocks * 3 * ln_nch(d) * 512; }

namespace {
// One row per wavefront while that is at most one work-group per compute unit (half the code to fetch and a shorter chain: 380 rows x
// 1024, whole update 4370 -> 4304 us; 260 x 64: 560 -> 540), of four wavefronts and then, up to 512 columns, of eight: every work-group leaves a partial row of
// sums (1400 x 256, two rows on four / one on eight: 6.5 / 5.6 us; 3100 x 512: 9.0 / 9.2).
struct LnBwdForm { int rows_per_wave, waves; };
LnBwdForm ln_bwd_form(int rows, int d) {
  const int cus = device_info().cus;
  if (ceil_div(rows, 4) <= cus) return {1, 4};
  return ceil_div(rows, 8) <= cus && ln_nch(d) == 1 ? LnBwdForm{1, 8} : LnBwdForm{2, 4};
}
// a grid that is resident at once (3 or 4 work-groups per compute unit fit, by registers): no second, partly filled round
int ln_bwd_blocks(int rows, int d) {
  const int resident = (ln_nch(d) >= 2 ? 3 : 4) * device_info().cus;
  const LnBwdForm f = ln_bwd_form(rows, d);
  return min(min(kLnBwdMaxBlocks, resident), ceil_div(rows, f.waves * f.rows_per_wave));
}
}  // namespace

int64_t layernorm_bwd_partial_floats(int most_rows, int d) {
  const int one_row = kWavesPerBlock * device_info().cus;  // (the most rows that go one to a wavefront: they leave the most partial rows for their number)
  return (int64_t)max(ln_bwd_blocks(most_rows, d), ln_bwd_blocks(min(most_rows, one_row), d)) * 3 * d;
}

int launch_residual_layernorm_bwd(const half_t* dout, const half_t* sub, const half_t* resid, const half_t* gamma,
                                  const float* stats, half_t* dy, half_t* dym, half_t* dgamma, half_t* dbeta,
                                  half_t* dbias, float* partial, int rows, int d, const DropDev& drop,
                                  hipStream_t stream, ColumnSums& sums, const Ahead& next) {
  NMT_REQUIRE(rows > 0 && d >= 8 && d % 8 == 0 && d <= 2048, "layernorm_bwd: d=%d must be a multiple of 8 in [8, 2048]", d);
  NMT_REQUIRE(dout && sub && resid && gamma && stats && dy && partial, "layernorm_bwd: null pointer");
  NMT_REQUIRE(aligned16(dout) && aligned16(sub) && aligned16(resid) && aligned16(gamma) && aligned16(dy) && aligned16(dym),
              "layernorm_bwd: misaligned pointer");
  NMT_REQUIRE(!drop.thr || (drop.n_pos > 0 && dym), "layernorm_bwd: dropout needs the masked output and positions per sentence");
  const int nch = ln_nch(d);
  const LnBwdForm form = ln_bwd_form(rows, d);
  const int nblk = ln_bwd_blocks(rows, d);
  Ahead a = next;
  a.first = (uint32_t)nblk;
  const dim3 grid(a.first + ahead_groups(a)), block(kWave * form.waves);
  const size_t smem = (size_t)form.waves * nch * 512 * sizeof(float);
  auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, smem, stream, dout, sub, resid, gamma, stats, dy, dym, partial, rows, d, drop, a); };
#define NMT_LN_BWD(N, R, W) NMT_ROW_FORM(run, res_ln_bwd_kernel, N, R, W)
  switch (nch * 4 + (form.waves == 8 ? 2 : form.rows_per_wave - 1)) {
    case 4: NMT_LN_BWD(1, 1, 4); break;
    case 5: NMT_LN_BWD(1, 2, 4); break;
    case 6: NMT_LN_BWD(1, 1, 8); break;
    case 8: NMT_LN_BWD(2, 1, 4); break;
    case 9: NMT_LN_BWD(2, 2, 4); break;
    case 16: NMT_LN_BWD(4, 1, 4); break;
    default: NMT_LN_BWD(4, 2, 4); break;
  }
#undef NMT_LN_BWD
  NMT_LAUNCH_CHECK();
  sums = ColumnSums{partial, nblk, {dgamma, dbeta, dbias}};
  return NMT_OK;
}
int launch_layernorm_param_grads(const ColumnSums* sums, int n, int d, float scale, hipStream_t stream) {
  return launch_finalize(sums, n, 3, d, d, scale, stream);
}

int64_t colsum_scratch_floats(int cols) { return (int64_t)kColsumMaxSplits * cols; }

// ------------------------------------------------------------------------------------------------
// Column sums for callers that cannot allocate (code under graph capture, serving loops): the partial
// sums live in a fixed device array instead of a caller-provided buffer.  Each GPU holds its own copy of
// the array at its own address, looked up once per device; every call on a GPU shares that copy.
// ------------------------------------------------------------------------------------------------
constexpr int kStaticColsumMaxCols = 4096;
static __device__ __align__(256) float scratch[(size_t)kColsumMaxSplits * kStaticColsumMaxCols];  // 8 MiB per GPU

namespace {
constexpr int kMaxDevices = 64;
float* g_scratch_ptr[kMaxDevices] = {};
std::mutex g_scratch_mutex;
// Device address of `scratch` on the current device (its name is only a host-side stand-in for it).
int static_scratch(float** out) {
  int dev = 0;
  NMT_HIP_CHECK(hipGetDevice(&dev));
  NMT_REQUIRE(dev >= 0 && dev < kMaxDevices, "colsum_static: device index %d outside [0, %d)", dev, kMaxDevices);
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    NMT_HIP_CHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
    NMT_REQUIRE(p, "colsum_static: the scratch array has no device address");
    g_scratch_ptr[dev] = static_cast<float*>(p);
  }
  *out = g_scratch_ptr[dev];
  return NMT_OK;
}
}  // namespace

int launch_colsum_static(const half_t* src, int ld, half_t* dst, int rows, int cols, hipStream_t stream) {
  NMT_REQUIRE(cols > 0 && cols <= kStaticColsumMaxCols, "colsum_static: cols=%d outside [1, %d], the width the fixed scratch array holds", cols,
              kStaticColsumMaxCols);
  float* partial = nullptr;
  if (int rc = static_scratch(&partial)) return rc;
  // every partial sum the second kernel reads is written by the first one of the same call: nothing to clear
  return launch_colsum(src, ld, dst, partial, rows, cols, stream, 1.f);
}

int launch_colsum(const half_t* src, int ld, half_t* dst, float* partial, int rows, int cols, hipStream_t stream, float scale) {
  NMT_REQUIRE(rows > 0 && cols > 0 && cols % 8 == 0 && ld % 8 == 0 && ld >= cols, "colsum: bad shape rows=%d cols=%d ld=%d", rows, cols, ld);
  NMT_REQUIRE(src && dst && partial && aligned16(src), "colsum: null or misaligned pointer");
  const int cb = ceil_div(cols, 512);
  int splits = 2048 / cb;  // enough blocks to keep every compute unit streaming
  splits = splits > kColsumMaxSplits ? kColsumMaxSplits : splits;
  splits = splits > rows / 16 ? rows / 16 : splits;
  splits = splits < 1 ? 1 : splits;
  hipLaunchKernelGGL(colsum_kernel, dim3(cb, splits), dim3(kThreads), 0, stream, src, ld, partial, rows, cols);
  NMT_LAUNCH_CHECK();
  const ColumnSums sums = {partial, splits, {dst, nullptr, nullptr}};
  return launch_finalize(&sums, 1, 1, cols, cols, scale, stream);
}

namespace {
template <XentForm FORM>
int launch_xent_rows(half_t* logits, const int32_t* targets, float* row_loss, float* row_lse, int32_t* row_target, int rows, int V, int pad_id,
                     float eps_ls, float loss_scale, hipStream_t stream) {
  const dim3 grid(rows), block(kThreads);
  const int nch = ceil_div(V / 8, kThreads);
#define NMT_XENT(N) \
  hipLaunchKernelGGL((softmax_xent_kernel<N, FORM>), grid, block, 0, stream, logits, targets, row_loss, row_lse, row_target, V, pad_id, eps_ls, \
                     loss_scale)
  if (nch <= 1) NMT_XENT(1);
  else if (nch <= 4) NMT_XENT(4);
  else if (nch <= 16) NMT_XENT(16);
  else if (nch <= 20) NMT_XENT(20);
  else NMT_XENT(32);
#undef NMT_XENT
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}
}  // namespace

int launch_softmax_xent(half_t* logits, const int32_t* targets, float* row_loss, int rows, int V, int pad_id, float eps_ls,
                        float loss_scale, float* loss_sum, int32_t* ntok, hipStream_t stream, float* row_lse, int32_t* row_target) {
  NMT_REQUIRE(rows > 0 && V >= 8 && V % 8 == 0 && V <= 65536, "softmax_xent: V=%d must be a multiple of 8 in [8, 65536]", V);
  NMT_REQUIRE(logits && targets && row_loss && loss_sum && ntok && aligned16(logits), "softmax_xent: null or misaligned pointer");
  NMT_REQUIRE(!row_lse == !row_target, "softmax_xent: the loss alone needs room for both the log-sum-exps and the targets");
  if (int rc = row_lse ? launch_xent_rows<kLossOnly>(logits, targets, row_loss, row_lse, row_target, rows, V, pad_id, eps_ls, loss_scale, stream)
                       : launch_xent_rows<kLossAndGrad>(logits, targets, row_loss, nullptr, nullptr, rows, V, pad_id, eps_ls, loss_scale, stream))
    return rc;
  hipLaunchKernelGGL(loss_reduce_kernel, dim3(1), dim3(1024), 0, stream, row_loss, targets, rows, pad_id, loss_sum, ntok);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}
int launch_softmax_grad(half_t* logits, const int32_t* row_target, float* row_lse, int rows, int V, int pad_id, float eps_ls, float loss_scale,
                        hipStream_t stream) {
  NMT_REQUIRE(rows > 0 && V >= 8 && V % 8 == 0 && V <= 65536 && logits && row_target && row_lse && aligned16(logits), "softmax_grad: bad arguments");
  return launch_xent_rows<kGradOnly>(logits, row_target, nullptr, row_lse, nullptr, rows, V, pad_id, eps_ls, loss_scale, stream);
}

namespace {
struct EmbScratch {
  int64_t k1, v1, keys, perm, hist, part, total;  // offsets in int32 units
  int nblk, nseg;
};
EmbScratch emb_scratch(int n, int d) {
  EmbScratch e;
  e.nblk = ceil_div(n, kSortPerBlock);
  e.nseg = ceil_div(n, kEmbSeg);
  int64_t cur = 0;
  auto take = [&](int64_t ints) {
    const int64_t off = cur;
    cur += round_up(ints, 4);
    return off;
  };
  e.k1 = take(n);
  e.v1 = take(n);
  e.keys = take(n);
  e.perm = take(n);
  e.hist = take((int64_t)256 * e.nblk);
  e.part = take((int64_t)2 * e.nseg * d);
  e.total = cur;
  return e;
}
int check_embed(const int32_t* ids_a, int rows_a, const int32_t* ids_b, int rows_b, int d, int vocab, const int32_t* scratch) {
  NMT_REQUIRE(rows_a >= 0 && rows_b >= 0 && rows_a + rows_b > 0, "embed_bwd: no rows");
  NMT_REQUIRE(d >= 8 && d % 8 == 0 && d / 8 <= kThreads && vocab > 0 && vocab <= 65536, "embed_bwd: bad d=%d or vocab=%d", d, vocab);
  NMT_REQUIRE((rows_a == 0 || ids_a) && (rows_b == 0 || ids_b) && scratch && aligned16(scratch), "embed_bwd: null or misaligned pointer");
  return NMT_OK;
}
}  // namespace

int64_t embed_bwd_scratch_ints(int /*vocab*/, int rows_total, int d) { return emb_scratch(rows_total, d).total; }

int launch_embed_sort(const int32_t* ids_a, int rows_a, const int32_t* ids_b, int rows_b, int d, int vocab, int32_t* scratch, hipStream_t stream) {
  if (int rc = check_embed(ids_a, rows_a, ids_b, rows_b, d, vocab, scratch)) return rc;
  const int n = rows_a + rows_b;
  const EmbScratch e = emb_scratch(n, d);
  int32_t *k1 = scratch + e.k1, *v1 = scratch + e.v1, *keys = scratch + e.keys, *perm = scratch + e.perm, *hist = scratch + e.hist;
  if (n <= kSmallSort) {
    NMT_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(emb_sort_small_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kSmallSortLds));
    hipLaunchKernelGGL(emb_sort_small_kernel, dim3(1), dim3(1024), kSmallSortLds, stream, ids_a, rows_a, ids_b, vocab, n, keys, perm);
    NMT_LAUNCH_CHECK();
    return NMT_OK;
  }
  // stable sort of the positions by id: low byte, then high byte
  const int nh = 256 * e.nblk;
  for (int pass = 0; pass < 2; ++pass) {
    const int32_t *kin = pass ? k1 : nullptr, *vin = pass ? v1 : nullptr;
    hipLaunchKernelGGL(radix_hist_kernel, dim3(e.nblk), dim3(kThreads), 0, stream, ids_a, rows_a, ids_b, vocab, kin, n, 8 * pass, e.nblk, hist);
    NMT_LAUNCH_CHECK();
    hipLaunchKernelGGL(radix_scan_kernel, dim3(1), dim3(1024), 0, stream, hist, nh);
    NMT_LAUNCH_CHECK();
    hipLaunchKernelGGL(radix_scatter_kernel, dim3(e.nblk), dim3(kThreads), 0, stream, ids_a, rows_a, ids_b, vocab, kin, vin, n, 8 * pass,
                       e.nblk, hist, pass ? keys : k1, pass ? perm : v1);
    NMT_LAUNCH_CHECK();
  }
  return NMT_OK;
}

int launch_embed_sum(const half_t* dx_a, int rows_a, const DropDev& drop_a, const half_t* dx_b, int rows_b, const DropDev& drop_b, half_t* gE,
                     int d, const int32_t* scratch, hipStream_t stream, float scale) {
  NMT_REQUIRE((rows_a == 0 || (dx_a && aligned16(dx_a))) && (rows_b == 0 || (dx_b && aligned16(dx_b))) && gE && aligned16(gE),
              "embed_bwd: null or misaligned pointer");
  NMT_REQUIRE((!drop_a.thr || drop_a.n_pos > 0) && (!drop_b.thr || drop_b.n_pos > 0), "embed_bwd: positions per sentence must be positive");
  const int n = rows_a + rows_b;
  const EmbScratch e = emb_scratch(n, d);
  const int32_t *keys = scratch + e.keys, *perm = scratch + e.perm;
  float* part = const_cast<float*>(reinterpret_cast<const float*>(scratch + e.part));
  const size_t lds = (size_t)kEmbSeg * d * sizeof(half_t);
  auto segments = [&](auto kernel, int threads) -> int {
    if (lds > 48 * 1024) NMT_HIP_CHECK(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds));
    hipLaunchKernelGGL(kernel, dim3(e.nseg), dim3(threads), lds, stream, dx_a, rows_a, drop_a, dx_b, drop_b, gE, n, d, keys, perm, part, scale);
    return NMT_OK;
  };
  // Entries shared out while the segments are few to a compute unit: one where a block takes 1024 threads, three where it takes 512, ten where a row is
  // a wavefront wide; at any number up to 256 columns.  By entries, shared out / a thread per eight columns, us, on 256 compute units: 2048 wide 2800 12.1 /
  // 15.6, 5000 21.7 / 18.0, 105000 165 / 121; 1024 wide 10000 16.1 / 17.9, 14000 20.2 / 18.7, 105000 77 / 67 (beside the last weight gradients 311 /
  // 251); 512 wide 35700 20.1 / 20.6, 42000 22.1 / 21.7, 200000 72.8 / 64.9; 256 wide 200000 49.6 / 60.2.
  const int chunks = d / 8, cus = device_info().cus, few = (chunks > 128 ? 1 : chunks > 64 ? 3 : 10) * cus;
  if (chunks > 32 && e.nseg > few) {
    hipLaunchKernelGGL(emb_segment_columns_kernel, dim3(e.nseg), dim3((int)round_up(chunks, kWave)), 0, stream, dx_a, rows_a, drop_a, dx_b, drop_b, gE, n, d,
                       keys, perm, part, scale);
  } else {
    // THREADS / (d / 8) groups times AHEAD entries are a segment or more.  From four segments per compute unit on the table's rows are asked for late: what
    // counts then is how many blocks share a compute unit, not the length of one (6600 x 512, all beside the last weight gradients: 14 late, 9.7 early).
    auto form = [&](auto early) -> int {
      constexpr bool E = decltype(early)::value;
      if (chunks <= 256 / kEmbSeg) return segments(emb_segment_kernel<256, 1, E>, 256);
      if (chunks <= 512 / kEmbSeg) return segments(emb_segment_kernel<256, 2, E>, 256);
      if (chunks <= 1024 / kEmbSeg) return segments(emb_segment_kernel<256, 4, E>, 256);
      return chunks <= 2048 / kEmbSeg ? segments(emb_segment_kernel<512, 4, true>, 512) : segments(emb_segment_kernel<1024, 4, true>, 1024);
    };
    if (int rc = e.nseg < 4 * cus ? form(std::true_type{}) : form(std::false_type{})) return rc;
  }
  NMT_LAUNCH_CHECK();
  hipLaunchKernelGGL(emb_finish_kernel, dim3(e.nseg), dim3(kEmbFinish), 0, stream, gE, n, d, keys, part, scale);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

int launch_dropout_mask(uint8_t* keep, int rows, int n_cols, const DropDev& drop, hipStream_t stream) {
  NMT_REQUIRE(keep && rows > 0 && n_cols > 0, "dropout_mask: bad arguments");
  NMT_REQUIRE(!drop.thr || drop.n_pos > 0, "dropout_mask: positions per sentence must be positive");
  const int64_t n = (int64_t)rows * ((n_cols + 7) / 8);
  hipLaunchKernelGGL(dropout_mask_kernel, dim3(ceil_div(n, kThreads)), dim3(kThreads), 0, stream, keep, rows, n_cols, drop);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

int launch_build_tables(const SegmentList& segs, int n_sent, const uint32_t* uid, uint2* rk_src, uint2* rk_tgt, int4* tab_ss,
                        int4* tab_tt, int4* tab_ts, hipStream_t stream) {
  NMT_REQUIRE(segs.n >= 1 && segs.n <= NMT_MAX_SEGMENTS && n_sent > 0, "build_tables: bad segment list");
  NMT_REQUIRE(rk_src && rk_tgt && tab_ss && tab_tt && tab_ts, "build_tables: null pointer");
  hipLaunchKernelGGL(build_tables_kernel, dim3(ceil_div(n_sent, kWavesPerBlock)), dim3(kThreads), 0, stream, segs, n_sent, uid, rk_src, rk_tgt,
                     tab_ss, tab_tt, tab_ts);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

int launch_build_tables_packed(const nmt_sentence* sentences, int n_sent, int n_src, int n_tgt, int max_src, int max_tgt,
                               int32_t* sent_rows, uint2* rk_src, uint2* rk_tgt, int4* tab_ss, int4* tab_tt, int4* tab_ts,
                               hipStream_t stream) {
  NMT_REQUIRE(sentences && n_sent > 0 && n_src >= n_sent && n_tgt >= n_sent && max_src > 0 && max_tgt > 0, "build_tables: bad packed batch");
  NMT_REQUIRE(sent_rows && rk_src && rk_tgt && tab_ss && tab_tt && tab_ts, "build_tables: null pointer");
  hipLaunchKernelGGL(packed_rows_kernel, dim3(1), dim3(1024), 0, stream, sentences, n_sent, max_src, max_tgt, sent_rows);
  NMT_LAUNCH_CHECK();
  hipLaunchKernelGGL(packed_tables_kernel, dim3(ceil_div(n_sent, kWavesPerBlock)), dim3(kThreads), 0, stream, sentences, n_sent, n_src, n_tgt,
                     max_src, max_tgt, sent_rows, rk_src, rk_tgt, tab_ss, tab_tt, tab_ts);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}
