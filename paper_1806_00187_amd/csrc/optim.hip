// HBM-bound update kernels: fp32 gradient accumulation, single-pass unscale + inf/NaN detection,
// Adam on fp32 master weights with fp16 weight refresh.  All are grid-stride loops whose wavefronts read and
// write whole contiguous kilobytes (16 bytes of fp32 per lane).  A large copy reaches 5.0-5.5 TB/s on this card.
#include "common.h"

#include <type_traits>

namespace {

constexpr int kThreads = 256;
constexpr int kMaxBlocks = 256 * 8;  // 8 work-groups per CU keeps enough loads in flight
constexpr int kAdamMaxBlocks = 65536;
constexpr int64_t kStreamFrom = 16 << 20;  // parameters from which accumulator, master weights and moments exceed 256 MB of last-level cache
constexpr int kAccumulateAhead = 4;

template <bool STREAM>
__device__ __forceinline__ floatx4 ld_state(const float* p) { return STREAM ? ld_float4_nt(p) : *reinterpret_cast<const floatx4*>(p); }
template <bool STREAM>
__device__ __forceinline__ void st_state(float* p, floatx4 v) {
  if (STREAM) st_float4_nt(p, v);
  else *reinterpret_cast<floatx4*>(p) = v;
}

__device__ __forceinline__ bool non_finite(float x) { return (__float_as_uint(x) & 0x7F800000u) == 0x7F800000u; }

// acc (+)= mult * float(g16); mult undoes the power-of-two factor a pass applied before rounding to fp16.
// Four fp32 values per lane and access, so that a store instruction covers a contiguous kilobyte (with eight per lane
// it covered every other 16 bytes of two), four of them in flight per thread: 289 -> 223 us at 219 million parameters (5.9 TB/s),
// 84 -> 63 at 63 million.
// CHECK: also raises the flag if a sum is inf or NaN (the last sub-batch of an update: no pass of its own over acc).
template <bool STREAM, bool CHECK = false>
__global__ void __launch_bounds__(kThreads) accumulate_kernel(const half_t* __restrict__ g16, float* __restrict__ acc, int64_t n,
                                                              int first, float mult, int32_t* __restrict__ flag) {
  const int64_t nvec = n >> 2;
  bool bad = false;
  const int64_t block = (int64_t)kAccumulateAhead * kThreads, stride = (int64_t)gridDim.x * block;
  for (int64_t i0 = (int64_t)blockIdx.x * block + threadIdx.x; i0 < nvec; i0 += stride) {
    half4_t g[kAccumulateAhead];
    floatx4 a[kAccumulateAhead];
#pragma unroll
    for (int u = 0; u < kAccumulateAhead; ++u) {
      const int64_t i = min(i0 + u * kThreads, nvec - 1);  // (past the end: the last vector again, not stored)
      g[u] = *reinterpret_cast<const half4_t*>(g16 + i * 4);
      a[u] = first ? floatx4{0, 0, 0, 0} : ld_state<STREAM>(acc + i * 4);
    }
#pragma unroll
    for (int u = 0; u < kAccumulateAhead; ++u) {
#pragma unroll
      for (int e = 0; e < 4; ++e) a[u][e] += mult * (float)g[u][e];
      if (i0 + u * kThreads < nvec) {  // (a lane past the end holds the last vector, which its owner may have stored already: no sum to check)
#pragma unroll
        for (int e = 0; CHECK && e < 4; ++e) bad |= non_finite(a[u][e]);
        st_state<STREAM>(acc + (i0 + u * kThreads) * 4, a[u]);
      }
    }
  }
  // tail (n not a multiple of 4)
  for (int64_t i = (nvec << 2) + (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads) {
    const float a = (first ? 0.f : acc[i]) + mult * (float)g16[i];
    if (CHECK) bad |= non_finite(a);
    acc[i] = a;
  }
  if (CHECK && __any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

// Whether a pass's fp16 gradient holds an inf or NaN: the overflow check of an update of one pass, whose accumulator it becomes
// (times a power of two not above 256, which keeps finite halves finite).  Sixteen bytes a lane, four in flight.
__global__ void __launch_bounds__(kThreads) check_half_kernel(const half_t* __restrict__ g16, int64_t n, int32_t* __restrict__ flag) {
  const int64_t nvec = n >> 3;
  const int64_t block = (int64_t)kAccumulateAhead * kThreads, stride = (int64_t)gridDim.x * block;
  bool bad = false;
  for (int64_t i0 = (int64_t)blockIdx.x * block + threadIdx.x; i0 < nvec; i0 += stride) {
    uint4 g[kAccumulateAhead];
#pragma unroll
    for (int u = 0; u < kAccumulateAhead; ++u) g[u] = reinterpret_cast<const uint4*>(g16)[min(i0 + u * kThreads, nvec - 1)];
#pragma unroll
    for (int u = 0; u < kAccumulateAhead; ++u)
      for (uint32_t w : {g[u].x, g[u].y, g[u].z, g[u].w}) bad |= (w & 0x7C00u) == 0x7C00u || (w & 0x7C000000u) == 0x7C000000u;
  }
  for (int64_t i = (nvec << 3) + (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += (int64_t)gridDim.x * kThreads)
    bad |= non_finite((float)g16[i]);
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

__global__ void set_flag_kernel(int32_t* flag, int32_t v) { *flag = v; }
__global__ void add_scalars_kernel(const float* loss, const int32_t* ntok, float* loss_total, int32_t* ntok_total, int first) {
  *loss_total = (first ? 0.f : *loss_total) + *loss;
  *ntok_total = (first ? 0 : *ntok_total) + *ntok;
}

// IN_PLACE: acc *= inv_scale in the same pass; otherwise the buffer is only read (the caller applies the factor later)
template <bool IN_PLACE>
__global__ void __launch_bounds__(kThreads) check_overflow_kernel(float* __restrict__ acc, int64_t n, float inv_scale,
                                                                  int32_t* __restrict__ flag) {
  const int64_t nvec = n >> 2;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  bool bad = false;
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec; i += stride) {
    floatx4 v = ld_float4_nt(acc + i * 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      bad |= non_finite(v[e]);
      v[e] *= inv_scale;
    }
    if (IN_PLACE) st_float4_nt(acc + i * 4, v);
  }
  for (int64_t i = (nvec << 2) + (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) {
    bad |= non_finite(acc[i]);
    if (IN_PLACE) acc[i] *= inv_scale;
  }
  if (__any(bad) && (threadIdx.x & 63) == 0) atomicOr(flag, 1);
}

// One vector per thread in all but the largest models, and streamed past the caches where they could not hold the state
// until the next update anyway: of grids of 1024 to 65536 work-groups, one to four vectors at a time, streamed or not, this was the
// fastest at 63 and 219 million parameters: 388 -> 313 us and 1410 -> 1184 (5.6 TB/s).  A model whose state the caches do hold
// gains nothing from it (two layers 64 wide, two layers 256 wide: the same within the runs' spread).
// FROM_HALF: an update of one pass.  acc is mult * float(g16), written here on the way (whatever the flag) instead of written by one
// pass and read by two: 34 bytes a parameter for the update instead of 40.  Whole updates of one pass: 3000 positions x 512 wide, 63 million
// parameters, -3.3 %; 219 million, 380 and 3000 positions, -3.3 and -3.6 %.
template <bool STREAM, bool FROM_HALF = false>
__global__ void __launch_bounds__(kThreads) adam_kernel(float* __restrict__ master, float* __restrict__ m, float* __restrict__ v,
                                                        std::conditional_t<FROM_HALF, float, const float>* __restrict__ acc, half_t* __restrict__ w16,
                                                        int64_t n, float lr, float b1, float b2, float eps, float inv_bc1, float inv_bc2,
                                                        float gscale, const int32_t* __restrict__ flag, const half_t* __restrict__ g16, float mult) {
  const bool skip = flag && *flag != 0;  // overflow: skip the update, every buffer stays bit-identical
  if (!FROM_HALF && skip) return;
  const int64_t nvec = n >> 2;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  auto accumulated = [&](half_t g) { return 0.f + mult * (float)g; };
  if (FROM_HALF && skip) {
    for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride)
      if constexpr (FROM_HALF) acc[i] = accumulated(g16[i]);
    return;
  }
  for (int64_t i = (int64_t)blockIdx.x * kThreads + threadIdx.x; i < nvec; i += stride) {
    floatx4 w = ld_state<STREAM>(master + i * 4);
    floatx4 mm = ld_state<STREAM>(m + i * 4);
    floatx4 vv = ld_state<STREAM>(v + i * 4);
    floatx4 a;
    if constexpr (FROM_HALF) {
      const half4_t g = *reinterpret_cast<const half4_t*>(g16 + i * 4);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] = accumulated(g[e]);
      st_state<STREAM>(acc + i * 4, a);
    } else {
      a = ld_state<STREAM>(acc + i * 4);
    }
    const floatx4 gg = a * gscale;   // the gradient in its original scale
    half4_t h;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      mm[e] = b1 * mm[e] + (1.f - b1) * gg[e];
      vv[e] = b2 * vv[e] + (1.f - b2) * gg[e] * gg[e];
      w[e] -= lr * (mm[e] * inv_bc1) / (sqrtf(vv[e] * inv_bc2) + eps);
      h[e] = (half_t)w[e];
    }
    st_state<STREAM>(master + i * 4, w);
    st_state<STREAM>(m + i * 4, mm);
    st_state<STREAM>(v + i * 4, vv);
    *reinterpret_cast<half4_t*>(w16 + i * 4) = h;  // (the next forward pass reads these)
  }
  for (int64_t i = (nvec << 2) + (int64_t)blockIdx.x * kThreads + threadIdx.x; i < n; i += stride) {
    if constexpr (FROM_HALF) acc[i] = accumulated(g16[i]);
    const float gg = acc[i] * gscale;
    const float mm = b1 * m[i] + (1.f - b1) * gg;
    const float vv = b2 * v[i] + (1.f - b2) * gg * gg;
    const float w = master[i] - lr * (mm * inv_bc1) / (sqrtf(vv * inv_bc2) + eps);
    m[i] = mm;
    v[i] = vv;
    master[i] = w;
    w16[i] = (half_t)w;
  }
}

int grid_for(int64_t nvec, int most = kMaxBlocks) {
  int64_t b = (nvec + kThreads - 1) / kThreads;
  return (int)(b < 1 ? 1 : (b > most ? most : b));
}

}  // namespace

int launch_accumulate(const half_t* g16, float* acc, int64_t n, int first, hipStream_t stream, float mult, int32_t* flag) {
  NMT_REQUIRE(g16 && acc && n > 0, "accumulate: bad arguments");
  NMT_REQUIRE(aligned16(g16) && aligned16(acc), "accumulate: buffers must be 16-byte aligned");
  const bool big = n >= kStreamFrom;
  hipLaunchKernelGGL(flag ? (big ? accumulate_kernel<true, true> : accumulate_kernel<false, true>)
                          : (big ? accumulate_kernel<true, false> : accumulate_kernel<false, false>),
                     dim3(grid_for(ceil_div(n, 4 * kAccumulateAhead), 4 * kMaxBlocks)), dim3(kThreads), 0, stream, g16, acc, n, first, mult, flag);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

int launch_add_scalars(const float* loss, const int32_t* ntok, float* loss_total, int32_t* ntok_total, int first, hipStream_t stream) {
  hipLaunchKernelGGL(add_scalars_kernel, dim3(1), dim3(1), 0, stream, loss, ntok, loss_total, ntok_total, first);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

int launch_check_overflow(float* acc, int64_t n, float inv_scale, int32_t* flag, hipStream_t stream, bool in_place) {
  NMT_REQUIRE(acc && flag && n > 0, "check_overflow: bad arguments");
  NMT_REQUIRE(aligned16(acc), "check_overflow: buffer must be 16-byte aligned");
  hipLaunchKernelGGL(set_flag_kernel, dim3(1), dim3(1), 0, stream, flag, 0);
  NMT_LAUNCH_CHECK();
  if (in_place) hipLaunchKernelGGL(check_overflow_kernel<true>, dim3(grid_for(n >> 2)), dim3(kThreads), 0, stream, acc, n, inv_scale, flag);
  else hipLaunchKernelGGL(check_overflow_kernel<false>, dim3(grid_for(n >> 2)), dim3(kThreads), 0, stream, acc, n, 1.f, flag);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

int launch_adam(float* master, float* m, float* v, const float* g, half_t* w16, int64_t n, float lr, float b1, float b2,
                float eps, int t, const int32_t* flag, hipStream_t stream, float grad_scale) {
  NMT_REQUIRE(master && m && v && g && w16 && n > 0 && t >= 1, "adam: bad arguments");
  NMT_REQUIRE(aligned16(master) && aligned16(m) && aligned16(v) && aligned16(g) && aligned16(w16), "adam: buffers must be 16-byte aligned");
  const double bc1 = 1.0 - pow((double)b1, (double)t), bc2 = 1.0 - pow((double)b2, (double)t);
  hipLaunchKernelGGL(n >= kStreamFrom ? adam_kernel<true> : adam_kernel<false>, dim3(grid_for(n >> 2, kAdamMaxBlocks)), dim3(kThreads), 0, stream, master,
                     m, v, g, w16, n, lr, b1, b2, eps, (float)(1.0 / bc1), (float)(1.0 / bc2), grad_scale, flag, nullptr, 1.f);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

// What is left of an update when its last pass's gradient g16 is there: accumulation, overflow check and Adam, to the same bits as
// launch_accumulate, launch_check_overflow and launch_adam one after the other.
int launch_last_accumulate_and_adam(const half_t* g16, float mult, int first, float* master, float* m, float* v, float* acc, half_t* w16, int64_t n,
                                    float lr, float b1, float b2, float eps, int t, int32_t* flag, hipStream_t stream, float grad_scale) {
  NMT_REQUIRE(g16 && master && m && v && acc && w16 && flag && n > 0 && t >= 1, "last accumulate and adam: bad arguments");
  NMT_REQUIRE(aligned16(g16) && aligned16(master) && aligned16(m) && aligned16(v) && aligned16(acc) && aligned16(w16),
              "last accumulate and adam: buffers must be 16-byte aligned");
  hipLaunchKernelGGL(set_flag_kernel, dim3(1), dim3(1), 0, stream, flag, 0);
  NMT_LAUNCH_CHECK();
  if (!first) {
    if (const int rc = launch_accumulate(g16, acc, n, 0, stream, mult, flag); rc != NMT_OK) return rc;
    return launch_adam(master, m, v, acc, w16, n, lr, b1, b2, eps, t, flag, stream, grad_scale);
  }
  hipLaunchKernelGGL(check_half_kernel, dim3(grid_for(ceil_div(n, 8 * kAccumulateAhead), 4 * kMaxBlocks)), dim3(kThreads), 0, stream, g16, n, flag);
  NMT_LAUNCH_CHECK();
  const double bc1 = 1.0 - pow((double)b1, (double)t), bc2 = 1.0 - pow((double)b2, (double)t);
  hipLaunchKernelGGL((n >= kStreamFrom ? adam_kernel<true, true> : adam_kernel<false, true>), dim3(grid_for(n >> 2, kAdamMaxBlocks)), dim3(kThreads), 0,
                     stream, master, m, v, acc, w16, n, lr, b1, b2, eps, (float)(1.0 / bc1), (float)(1.0 / bc2), grad_scale, flag, g16, mult);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}
