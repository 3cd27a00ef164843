// Everything between two attentions of a narrow model in one kernel.  Between an attention and the next there are only operations
// that work on a token's row by itself: output projection, residual + dropout + LayerNorm, feed-forward sub-layer, the next
// attention's projections; backward the same in reverse.  As launches of their own they are six kernels of 4 to 7 us
// for a few hundred rows -- each a launch, a trip to memory for its operands and one for its results --, whatever little they compute.  Here a
// work-group takes 16 rows through all of them: activations stay in LDS, the weights stream past once per work-group.
//
// What bounds it: 64 wide the chain of dependent steps (7 us a layer forward, 9 backward), 256 wide the weights' way into the compute unit: 1.5 MB
// a layer, 64 bytes a clock from L2 at most, forward through LDS (20 of 25 us at 80 GB/s), backward straight into registers (16 of 23).  So it pays
// where the weights of a layer are few, and is not offered above 256 columns; the widest feed-forward layer is four times the width.  Sixteen rows are the least a matrix instruction takes: more work-groups, each
// with the same weights to read, cost nothing while compute units are idle.  Whole passes of 2 + 2 layers, forward and backward, a launch for each operation / chains, us:
// 64 wide 32 rows 301 / 212, 2048 419 / 306, 16384 703 / 565; 128 wide 326 / 245, 436 / 303, 859 / 814; 256 wide 512 rows 423 / 402, 2048 497 / 444, 4096 594 / 568, 8192 (two
// rounds of work-groups) 991 / 1005.  The GPU's time alone: a pass of up to 128 rows 256 wide with 1024 hidden units takes 5 to 9 % longer in chains than in today's
// general kernels (6 + 6 layers, 128 rows 1115 / 1210); so does an update of several such passes one
// after the other (eight of 128 rows, 3 + 3 layers, 4.88 / 5.15 ms; 5.68 before either).  A single one's is bound by the host, which enqueues half as many launches (1270 to 1470 / 1370), as are
// passes in flight (four at a time 4.16 / 3.04 ms), so no line is drawn there.
//
// No product is cut along k among the wavefronts: backward 64 wide a product with 64 columns is two tiles, and six of the eight wavefronts wait for them.
//
// Every product adds up in the order of the general kernels (32 k at a time, increasing), every tensor is rounded where they round it,
// and a row's LayerNorm is computed lane by lane as they do, so activations and their gradients are the same bits as theirs.  (The sums over rows for the
// gradients of gains, shifts and output biases are taken in another order.)
#include <type_traits>

#include "common.h"

namespace {

constexpr int kRows = 16;            // rows of a work-group: the row count of one matrix instruction
constexpr int kWaves = 8, kThreads = 64 * kWaves;
static_assert(kRows == 2 * kWaves, "a wavefront takes two rows of a LayerNorm");
constexpr int kPad = 8;              // halves behind every row in LDS: 16 rows at one column lie on 64 different banks

typedef _Float16 half4v_t __attribute__((ext_vector_type(4)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef uint32_t uint4v_t __attribute__((ext_vector_type(4)));

// Work-group barrier for data in LDS alone: what is on its way to or from memory stays on its way.
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// (Results are rounded to fp32 first, as in the general kernels: element by element the compiler would form the last sum in fp16's own instruction.)
__device__ __forceinline__ half8_t to_half8(const floatx8& v) { return __builtin_convertvector(v, half8_t); }

// A tile of kRows rows in LDS.
struct LdsTile {
  half_t* p;
  int pitch;
  __device__ __forceinline__ half_t* at(int row, int col) const { return p + row * pitch + col; }
};

// Rows row0 .. row0 + 15 of a [rows, N] matrix (N at most MOST) -> LDS and back, 16 bytes a thread, 32 threads a row.  (Rows past the end repeat the
// last one.)
template <int MOST>
struct TileRegs {
  static constexpr int NV = (MOST + 255) / 256;
  half8_t v[NV];
  __device__ __forceinline__ void request(const half_t* __restrict__ src, int N, int row0, int rows) {
    const half_t* from = src + (size_t)min(row0 + (int)(threadIdx.x >> 5), rows - 1) * N;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = ((threadIdx.x & 31) + 32 * i) * 8;
      v[i] = ld_half8(from + (c < N ? c : 0));  // (a thread without a piece reads the row's first)
    }
  }
  __device__ __forceinline__ void store(const LdsTile& t, int N) const {
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int c = ((threadIdx.x & 31) + 32 * i) * 8;
      if (c < N) *reinterpret_cast<half8_t*>(t.at(threadIdx.x >> 5, c)) = v[i];
    }
  }
};
__device__ __forceinline__ void store_tile(const LdsTile& t, half_t* __restrict__ dst, int N, int row0, int rows) {
  const int r = threadIdx.x >> 5;
  if (row0 + r >= rows) return;
  half_t* to = dst + (size_t)(row0 + r) * N;
  for (int c = (threadIdx.x & 31) * 8; c < N; c += 256) st_half8(to + c, *reinterpret_cast<const half8_t*>(t.at(r, c)));
}

// A wavefront's way through its tiles of a product, eight apart, and the pieces of k (its units of work) of each.
struct Cursor {
  int tile, piece;
  __device__ __forceinline__ void next(int pieces) {
    if (++piece == pieces) {
      piece = 0;
      tile += kWaves;
    }
  }
};
__device__ __forceinline__ int tiles_of(int N, int width, int wave) { return max(0, (N / width - wave + kWaves - 1) / kWaves); }

// ---- x W^T: weights [N, K], k contiguous ----------------------------------------------------------
// Tiles of 16 columns.  A unit is loaded as it lies in memory and turned into operands in LDS of the wavefront's own.  (Asked for in operand order
// -- 16 rows, 64 bytes of each -- an instruction takes the 64 clocks of its 64 addresses: 38 GB/s to a compute unit instead of 145; an
// encoder layer 256 wide 52 us.)  Two units are on their way while one is multiplied, also over the end of a product: the first units of the next one do
// not depend on anything before it.  There is an even number of units to each wavefront, so that the two sets of registers take turns.
template <int D>
struct FwdUnit {
  static constexpr int U = D == 256 ? 256 : D / 2, CH = U / 8;  // k of a unit, 16-byte pieces of a row
  half8_t w[U / 32];
};
struct FwdProduct {
  const half_t* w;
  const half_t* b;  // in LDS
  int K, N;
};
template <int D>
__device__ __forceinline__ void load_unit(FwdUnit<D>& u, const FwdProduct& p, int lane, const Cursor& c) {
  using F = FwdUnit<D>;
  const half_t* at = p.w + (size_t)(c.tile * 16 + lane / F::CH) * p.K + c.piece * F::U + lane % F::CH * 8;
#pragma unroll
  for (int s = 0; s < F::U / 32; ++s) u.w[s] = ld_half8(at + (size_t)(s * (64 / F::CH)) * p.K);
}
template <int D>
__device__ __forceinline__ void load_first(FwdUnit<D> (&u)[2], const FwdProduct& p, int wave, int lane) {
  if (wave * 16 >= p.N) return;
  Cursor c{wave, 0};
  load_unit<D>(u[0], p, lane, c);
  c.next(p.K / FwdUnit<D>::U);
  load_unit<D>(u[1], p, lane, c);
}
// out = x W^T + b into LDS; `u`: its first two units, on their way; on return those of `next`.  DEEP: K is more than a unit (else the wavefront keeps x in
// registers).
template <int D, bool RELU, bool DEEP>
__device__ __forceinline__ void product(FwdUnit<D> (&u)[2], const FwdProduct& p, const LdsTile& x, const LdsTile& out, const LdsTile& own,
                                        const FwdProduct& next, int wave, int lane) {
  using F = FwdUnit<D>;
  constexpr int KS = F::U / 32;
  const int row = lane & 15, q = lane >> 4, pieces = DEEP ? p.K / F::U : 1;
  half8_t xf[KS];
  auto operands = [&](int piece) {
#pragma unroll
    for (int s = 0; s < KS; ++s) xf[s] = *reinterpret_cast<const half8_t*>(x.at(row, piece * F::U + 32 * s + q * 8));
  };
  const int n = tiles_of(p.N, 16, wave) * pieces;
  if (!DEEP && n) operands(0);
  floatx4 acc = {0.f, 0.f, 0.f, 0.f};
  Cursor at{wave, 0}, ahead{wave, 0};
  ahead.next(pieces);
  ahead.next(pieces);
  auto step = [&](const F& f, auto refill) {
    wave_sync();  // the unit before has been read
#pragma unroll
    for (int s = 0; s < KS; ++s) *reinterpret_cast<half8_t*>(own.at(s * (64 / F::CH) + lane / F::CH, lane % F::CH * 8)) = f.w[s];
    refill();
    wave_sync();  // this one is in LDS
    if (DEEP) operands(at.piece);
#pragma unroll
    for (int s = 0; s < KS; ++s)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_f16(*reinterpret_cast<const half8_t*>(own.at(row, 32 * s + q * 8)), xf[s], acc, 0, 0, 0);
    if (at.piece + 1 == pieces) {
      const half4v_t bias = *reinterpret_cast<const half4v_t*>(p.b + at.tile * 16 + q * 4);
      floatx4 y;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        y[e] = acc[e] + (float)bias[e];
        if (RELU) y[e] = fmaxf(y[e], 0.f);
      }
      *reinterpret_cast<half4v_t*>(out.at(row, at.tile * 16 + q * 4)) = __builtin_convertvector(y, half4v_t);
      acc = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    at.next(pieces);
  };
  for (int left = n; left > 2; left -= 2) {
    step(u[0], [&] { load_unit<D>(u[0], p, lane, ahead); ahead.next(pieces); });
    step(u[1], [&] { load_unit<D>(u[1], p, lane, ahead); ahead.next(pieces); });
  }
  if (n) {
    step(u[0], [] {});
    step(u[1], [] {});
  }
  load_first<D>(u, next, wave, lane);
}

// ---- dy W: weights [K, N], n contiguous -----------------------------------------------------------
// A lane loads C consecutive columns of eight consecutive k rows and turns them into C operands of eight k in its registers, so a wavefront's tile
// is 16 C columns wide, MFMA t of a step holding every C-th of them from t on, and a result lane ends up with 4 C consecutive columns of its
// row.  Loads of 16 bytes (C = 8) and of 4 (C = 2, 64 bytes of each row) come at 145 and 120 GB/s to a compute unit, of 8 bytes at 75.  As above, two units
// are on their way while one is multiplied.
template <int C, int KS>
struct BwdUnit {
  typedef uint32_t Words __attribute__((ext_vector_type(C / 2)));
  Words w[8 * KS];
  __device__ __forceinline__ uint32_t word(int i, int t) const { return w[i][t >> 1]; }
};
template <int KS>
struct BwdUnit<2, KS> {
  typedef uint32_t Words;
  Words w[8 * KS];
  __device__ __forceinline__ uint32_t word(int i, int) const { return w[i]; }
};
struct BwdProduct {
  const half_t* w;
  int K, N;
};
template <int C, int KS>
__device__ __forceinline__ void load_unit(BwdUnit<C, KS>& u, const BwdProduct& p, int lane, const Cursor& c) {
  const half_t* at = p.w + (size_t)(c.piece * 32 * KS + (lane >> 4) * 8) * p.N + c.tile * 16 * C + (lane & 15) * C;
#pragma unroll
  for (int s = 0; s < KS; ++s)
#pragma unroll
    for (int e = 0; e < 8; ++e) u.w[8 * s + e] = *reinterpret_cast<const typename BwdUnit<C, KS>::Words*>(at + (size_t)(32 * s + e) * p.N);
}
template <int C, int KS>
__device__ __forceinline__ void load_first(BwdUnit<C, KS> (&u)[2], const BwdProduct& p, int wave, int lane) {
  if (wave * 16 * C >= p.N) return;
  Cursor c{wave, 0};
  load_unit(u[0], p, lane, c);
  c.next(p.K / (32 * KS));
  load_unit(u[1], p, lane, c);
}
template <int C, int KS>
__device__ __forceinline__ half8_t operand(const BwdUnit<C, KS>& u, int s, int t) {
  const uint32_t sel = t & 1 ? 0x07060302u : 0x05040100u;
  uint4v_t d;
#pragma unroll
  for (int j = 0; j < 4; ++j) d[j] = __builtin_amdgcn_perm(u.word(8 * s + 2 * j + 1, t), u.word(8 * s + 2 * j, t), sel);
  return __builtin_bit_cast(half8_t, d);
}
enum SideUse { kNoSide, kSideAdd, kSideMask };
template <SideUse USE>
__device__ __forceinline__ float with_side(float v, half_t s) {
  if constexpr (USE == kSideAdd) return v + (float)s;
  if constexpr (USE == kSideMask) return (float)s > 0.f ? v : 0.f;
  return v;
}
// out = dy W (+ side, or masked by it) into LDS; `side` may be `out` itself.  `u`: the first two units, on their way.
template <int C, int KS, SideUse USE>
__device__ __forceinline__ void product_t(BwdUnit<C, KS> (&u)[2], const BwdProduct& p, const LdsTile& dy, const LdsTile& out, const LdsTile& side, int wave,
                                          int lane) {
  const int row = lane & 15, q = lane >> 4, pieces = p.K / (32 * KS), n = tiles_of(p.N, 16 * C, wave) * pieces;
  floatx4 acc[C];
#pragma unroll
  for (int t = 0; t < C; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
  Cursor at{wave, 0}, ahead{wave, 0};
  ahead.next(pieces);
  ahead.next(pieces);
  auto step = [&](const BwdUnit<C, KS>& f) {
    const half_t* a = dy.at(row, at.piece * 32 * KS + q * 8);
#pragma unroll
    for (int s = 0; s < KS; ++s) {
      const half8_t af = *reinterpret_cast<const half8_t*>(a + 32 * s);
#pragma unroll
      for (int t = 0; t < C; ++t) acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_f16(operand<C, KS>(f, s, t), af, acc[t], 0, 0, 0);
    }
    if (at.piece + 1 == pieces) {
      const int col = at.tile * 16 * C + q * 4 * C;
#pragma unroll
      for (int i = 0; i < C / 2; ++i) {
        const half8_t sd = USE == kNoSide ? zero_half8() : *reinterpret_cast<const half8_t*>(side.at(row, col + 8 * i));
        floatx8 o;
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] = with_side<USE>(acc[e % C][(8 * i + e) / C], sd[e]);
        *reinterpret_cast<half8_t*>(out.at(row, col + 8 * i)) = to_half8(o);
      }
#pragma unroll
      for (int t = 0; t < C; ++t) acc[t] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
    at.next(pieces);
  };
  for (int left = n; left > 2; left -= 2) {
    step(u[0]);
    load_unit(u[0], p, lane, ahead);
    ahead.next(pieces);
    step(u[1]);
    load_unit(u[1], p, lane, ahead);
    ahead.next(pieces);
  }
  if (n) {
    step(u[0]);
    step(u[1]);
  }
}

// ---- LayerNorm of a wavefront's two rows (wave and wave + 8) side by side, eight columns a lane -------------------
// Lane group u = lane / G has row wave + 8 u.  A row's sums are those of the row kernels: they meet the other half of a wavefront (and of 32
// lanes) first, which for a row of so few columns holds zeros, and then in the order below.
template <int D>
struct LnLane {
  static constexpr int G = D == 256 ? 32 : 16;
  int row, col, key;      // row of the tile, first column, row of the matrix (a row past the end: the last one)
  bool in, live;          // whether the lane has columns; whether the row is one to write
  __device__ __forceinline__ LnLane(int row0, int rows, int wave, int lane) {
    const int c = lane % G;
    row = wave + kWaves * (lane / G & 1);
    in = lane < 2 * G && c < D / 8;
    col = c < D / 8 ? c * 8 : 0;
    live = in && row0 + row < rows;
    key = min(row0 + row, rows - 1);
  }
  __device__ __forceinline__ half8_t only(half8_t v) const { return in ? v : zero_half8(); }
  __device__ __forceinline__ static float sum(float v) {
    auto bits = [](float x) { return __builtin_bit_cast(int, x); };
    auto num = [](int x) { return __builtin_bit_cast(float, x); };
    if constexpr (G == 32) {
      const auto h = __builtin_amdgcn_permlane16_swap(__builtin_bit_cast(unsigned, v), __builtin_bit_cast(unsigned, v), false, false);
      v = __builtin_bit_cast(float, (unsigned)h[0]) + __builtin_bit_cast(float, (unsigned)h[1]);
    }
    v += num(__builtin_amdgcn_update_dpp(0, bits(v), 0x128, 0xF, 0xF, true));  // row_ror:8
    v += num(__builtin_amdgcn_update_dpp(0, bits(v), 0x124, 0xF, 0xF, true));  // row_ror:4
    v += num(__builtin_amdgcn_update_dpp(0, bits(v), 0x4E, 0xF, 0xF, true));   // quad_perm:[2,3,0,1]
    return v + num(__builtin_amdgcn_update_dpp(0, bits(v), 0xB1, 0xF, 0xF, true));  // quad_perm:[1,0,3,2]
  }
  // the two rows' values added up
  __device__ __forceinline__ static float both(float v) {
    const unsigned x = __builtin_bit_cast(unsigned, v);
    const auto h = G == 32 ? __builtin_amdgcn_permlane32_swap(x, x, false, false) : __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return __builtin_bit_cast(float, (unsigned)h[0]) + __builtin_bit_cast(float, (unsigned)h[1]);
  }
};
template <int D>
__device__ __forceinline__ half8_t ln_forward(const LnLane<D>& L, const LdsTile& sub, const half8_t& resid, const uint2& key, const half8_t& gamma,
                                              const half8_t& beta, const RowChainLn& ln, const LdsTile& out, float eps) {
  const half8_t hs = L.only(*reinterpret_cast<const half8_t*>(sub.at(L.row, L.col)));
  const uint32_t bits = ln.drop.thr ? drop_keep8(ln.drop, drop_row_of(ln.drop, key), (uint32_t)(L.col >> 3)) : 0xFFu;
  float y[8], s = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) y[e] = (float)resid[e] + (((bits >> e) & 1u) ? (float)hs[e] * ln.drop.scale : 0.f);
#pragma unroll
  for (int e = 0; e < 8; ++e) s += y[e];
  const float mean = LnLane<D>::sum(s) / (float)D;
  float q = 0.f;
#pragma unroll
  for (int e = 0; e < 8; ++e) q += (y[e] - mean) * (y[e] - mean);
  const float rstd = 1.0f / sqrtf(LnLane<D>::sum(L.in ? q : 0.f) / (float)D + eps);
  floatx8 o;
#pragma unroll
  for (int e = 0; e < 8; ++e) o[e] = (y[e] - mean) * rstd * (float)gamma[e] + (float)beta[e];
  const half8_t result = to_half8(o);
  if (L.in) *reinterpret_cast<half8_t*>(out.at(L.row, L.col)) = result;
  if (L.live) {
    st_half8(ln.sub + (size_t)L.key * D + L.col, hs);
    st_half8(ln.out + (size_t)L.key * D + L.col, result);
    if (L.col == 0) *reinterpret_cast<float2*>(ln.stats + 2 * L.key) = make_float2(mean, rstd);
  }
  return result;
}

// LDS of a forward chain: three tiles of D columns, a unit of every wavefront, a tile of the widest product's columns and the biases of all of them.
template <int D>
__global__ void __launch_bounds__(kThreads) row_chain_fwd_kernel(const RowChainFwd a, int wide_pitch) {
  extern __shared__ __align__(16) half_t chain_lds[];
  touch(a);
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = blockIdx.x * kRows, rows = a.rows;
  constexpr int kPitch = D + kPad, kTile = kRows * kPitch, kUnitPitch = FwdUnit<D>::U + kPad;
  const LdsTile in{chain_lds, kPitch}, sub{chain_lds + kTile, kPitch}, x1{chain_lds + 2 * kTile, kPitch},
      own{chain_lds + 3 * kTile + wave * kRows * kUnitPitch, kUnitPitch}, wide{chain_lds + 3 * kTile + kWaves * kRows * kUnitPitch, wide_pitch};
  half_t* const biases = wide.p + kRows * wide_pitch;
  const FwdProduct attn_out{a.wo, biases, D, D}, ffn1{a.w1, biases + D, D, a.F}, ffn2{a.w2, biases + D + a.F, a.F, D};
  half_t* const proj_biases = biases + D + (a.F ? a.F + D : 0);
  auto proj = [&](int i) { return i < a.n_proj ? FwdProduct{a.proj[i].w, proj_biases + i * 3 * D, D, a.proj[i].n} : FwdProduct{nullptr, nullptr, 0, 0}; };
  constexpr bool kDeep = FwdUnit<D>::U < D;

  // everything that does not depend on what is computed here, the tile and the weights that come first first
  FwdUnit<D> unit[2];
  TileRegs<D> o;
  o.request(a.o, D, row0, rows);
  load_first<D>(unit, attn_out, wave, lane);
  const LnLane<D> L(row0, rows, wave, lane);
  const RowChainLn& second = a.F ? a.ln2 : a.ln1;
  const half8_t x = ld_half8(a.x + (size_t)L.key * D + L.col);
  const uint2 key = a.ln1.drop.rowkey[L.key];
  const half8_t gamma1 = ld_half8(a.ln1.gamma + L.col), beta1 = ld_half8(a.ln1.beta + L.col);
  const half8_t gamma2 = ld_half8(second.gamma + L.col), beta2 = ld_half8(second.beta + L.col);
  const int piece = threadIdx.x * 8;  // (no bias has more than the 4096 columns the threads take at once)
  half8_t bias[3 + kMaxRowChainProj];
  bias[0] = ld_half8(a.bo + (piece < D ? piece : 0));
  if (a.F) {
    bias[1] = ld_half8(a.b1 + (piece < a.F ? piece : 0));
    bias[2] = ld_half8(a.b2 + (piece < D ? piece : 0));
  }
#pragma unroll
  for (int i = 0; i < kMaxRowChainProj; ++i)
    if (i < a.n_proj) bias[3 + i] = ld_half8(a.proj[i].b + (piece < a.proj[i].n ? piece : 0));
  o.store(in, D);
  if (piece < D) *reinterpret_cast<half8_t*>(biases + piece) = bias[0];
  if (a.F) {
    if (piece < a.F) *reinterpret_cast<half8_t*>(biases + D + piece) = bias[1];
    if (piece < D) *reinterpret_cast<half8_t*>(biases + D + a.F + piece) = bias[2];
  }
#pragma unroll
  for (int i = 0; i < kMaxRowChainProj; ++i)
    if (i < a.n_proj && piece < a.proj[i].n) *reinterpret_cast<half8_t*>(proj_biases + i * 3 * D + piece) = bias[3 + i];
  lds_barrier();

  product<D, false, kDeep>(unit, attn_out, in, sub, own, a.F ? ffn1 : proj(0), wave, lane);
  lds_barrier();
  const half8_t y = ln_forward<D>(L, sub, L.only(x), key, gamma1, beta1, a.ln1, x1, a.eps);
  lds_barrier();
  if (a.F) {
    product<D, true, kDeep>(unit, ffn1, x1, wide, own, ffn2, wave, lane);
    lds_barrier();
    store_tile(wide, a.h, a.F, row0, rows);
    product<D, false, true>(unit, ffn2, wide, sub, own, proj(0), wave, lane);
    lds_barrier();
    ln_forward<D>(L, sub, L.only(y), key, gamma2, beta2, a.ln2, x1, a.eps);
    lds_barrier();
  }
  for (int i = 0; i < a.n_proj; ++i) {
    if (i) lds_barrier();  // (the tile before has been read)
    product<D, false, kDeep>(unit, proj(i), x1, wide, own, proj(i + 1), wave, lane);
    lds_barrier();
    store_tile(wide, a.proj[i].out, a.proj[i].n, row0, rows);
  }
}

// ---- backward -------------------------------------------------------------------------------------
// LayerNorm backward of a wavefront's rows: dout from LDS; the gradient at the sum goes to `dy` (LDS) and / or a.dy (memory), the
// gradient at the sub-layer's output to `dsub` and ln.dsub.  Column sums over the wavefront's rows are left in `sums` ([wavefront][3][D]).
struct LnBwdRow {
  half8_t sub, resid, gamma;
  float2 stats;
  uint2 key;
};
template <int D>
__device__ __forceinline__ void ln_request(LnBwdRow& r, const RowChainLnBwd& ln, const LnLane<D>& L) {
  r.sub = ld_half8(ln.sub + (size_t)L.key * D + L.col);
  r.resid = ld_half8(ln.resid + (size_t)L.key * D + L.col);
  r.gamma = ld_half8(ln.gamma + L.col);
  r.stats = *reinterpret_cast<const float2*>(ln.stats + 2 * L.key);
  r.key = ln.drop.rowkey[L.key];
}
template <int D>
__device__ __forceinline__ void ln_backward(const LnBwdRow& r, const RowChainLnBwd& ln, const LnLane<D>& L, const LdsTile& dout, const LdsTile* dy,
                                            half_t* dy_out, const LdsTile& dsub, float* sums, int wave, int lane) {
  const half8_t hg = L.only(*reinterpret_cast<const half8_t*>(dout.at(L.row, L.col)));
  const uint32_t bits = ln.drop.thr ? drop_keep8(ln.drop, drop_row_of(ln.drop, r.key), (uint32_t)(L.col >> 3)) : 0xFFu;
  float s1 = 0.f, s2 = 0.f, sums3[3][8];
  auto xhat = [&](int e) {
    const float y = (float)r.resid[e] + (((bits >> e) & 1u) ? (float)r.sub[e] * ln.drop.scale : 0.f);
    return (y - r.stats.x) * r.stats.y;
  };
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const float xh = xhat(e), go = (float)hg[e];
    ln_bwd_row_sums(s1, s2, go, (float)r.gamma[e], xh);
    sums3[0][e] = L.live ? go * xh : 0.f;
    sums3[1][e] = L.live ? go : 0.f;
  }
  const float m1 = LnLane<D>::sum(L.in ? s1 : 0.f) / (float)D, m2 = LnLane<D>::sum(L.in ? s2 : 0.f) / (float)D;
  floatx8 df, mf;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    df[e] = ln_bwd_dy((float)hg[e], (float)r.gamma[e], xhat(e), r.stats.y, m1, m2);
    mf[e] = ((bits >> e) & 1u) ? df[e] * ln.drop.scale : 0.f;
    sums3[2][e] = L.live ? mf[e] : 0.f;
  }
  const half8_t d8 = to_half8(df), m8 = to_half8(mf);
  if (L.in) {
    if (dy) *reinterpret_cast<half8_t*>(dy->at(L.row, L.col)) = d8;
    *reinterpret_cast<half8_t*>(dsub.at(L.row, L.col)) = m8;
  }
  if (L.live) {
    if (dy_out) st_half8(dy_out + (size_t)L.key * D + L.col, d8);
    st_half8(ln.dsub + (size_t)L.key * D + L.col, m8);
  }
#pragma unroll
  for (int k = 0; k < 3; ++k)
#pragma unroll
    for (int e = 0; e < 8; ++e) sums3[k][e] = LnLane<D>::both(sums3[k][e]);
  if (lane < D / 8) {
    floatx4* to = reinterpret_cast<floatx4*>(sums) + wave * 3 * (D / 4) + lane * 2;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      to[k * (D / 4)] = floatx4{sums3[k][0], sums3[k][1], sums3[k][2], sums3[k][3]};
      to[k * (D / 4) + 1] = floatx4{sums3[k][4], sums3[k][5], sums3[k][6], sums3[k][7]};
    }
  }
}
// The work-group's partial row of column sums, wavefronts in their order.
template <int D>
__device__ __forceinline__ void store_sums(const float* sums, float* partial) {
  const int i = threadIdx.x;
  static_assert(3 * D / 4 <= kThreads, "four columns to a thread");
  if (i >= 3 * D / 4) return;
  const floatx4* at = reinterpret_cast<const floatx4*>(sums) + i;
  floatx4 s = at[0];
#pragma unroll
  for (int w = 1; w < kWaves; ++w) s += at[w * (3 * D / 4)];
  reinterpret_cast<floatx4*>(partial + (size_t)blockIdx.x * 3 * D)[i] = s;
}

// CF: columns a lane loads of the products with F columns (8, or 2 where there are few).
template <int D, int CF>
__global__ void __launch_bounds__(kThreads) row_chain_bwd_kernel(const RowChainBwd a, int wide_pitch) {
  extern __shared__ __align__(16) half_t chain_lds[];
  touch(a);
  constexpr int kPitch = D + kPad, kTile = kRows * kPitch, KS = D == 256 && CF == 2 ? 2 : D / 64, KF = CF == 8 ? 1 : KS;  // (an even number of units in a tile)
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int row0 = blockIdx.x * kRows, rows = a.rows;
  const LdsTile dout{chain_lds, kPitch}, dy{chain_lds + kTile, kPitch}, dsub{chain_lds + 2 * kTile, kPitch}, wide{chain_lds + 3 * kTile, wide_pitch};
  float* sums = reinterpret_cast<float*>(chain_lds + 3 * kTile + kRows * wide_pitch);
  const BwdProduct head{a.head_w, a.head_k, D}, ffn2{a.w2, D, a.F}, ffn1{a.w1, a.F, D}, attn_out{a.wo, D, D};

  BwdUnit<2, KS> unit[2];
  BwdUnit<CF, KF> unit_f[2];
  LnBwdRow ln;
  const LnLane<D> L(row0, rows, wave, lane);
  // dout: the gradient that enters the chain, or what is added to its head's product; wide: that one's operand, then h
  TileRegs<D> first;
  TileRegs<3 * D> operand;
  TileRegs<4 * D> h;
  first.request(a.head_k ? a.dy_in : a.dx, D, row0, rows);
  if (a.head_k) {
    operand.request(a.head_a, a.head_k, row0, rows);
    load_first(unit, head, wave, lane);
  }
  ln_request<D>(ln, a.ln_a, L);
  if (a.F) {
    h.request(a.h, a.F, row0, rows);
  }
  first.store(dout, D);
  if (a.head_k) operand.store(wide, a.head_k);
  lds_barrier();
  if (a.head_k) {
    product_t<2, KS, kSideAdd>(unit, head, wide, dout, dout, wave, lane);
    if (!a.F) load_first(unit, attn_out, wave, lane);
    lds_barrier();
  } else if (!a.F) {
    load_first(unit, attn_out, wave, lane);
  }
  if (a.F) {
    load_first(unit_f, ffn2, wave, lane);
    h.store(wide, a.F);
    ln_backward<D>(ln, a.ln_a, L, dout, &dy, nullptr, dsub, sums, wave, lane);
    ln_request<D>(ln, a.ln_b, L);
    lds_barrier();
    store_sums<D>(sums, a.ln_a.partial);
    product_t<CF, KF, kSideMask>(unit_f, ffn2, dsub, wide, wide, wave, lane);
    load_first(unit, ffn1, wave, lane);
    lds_barrier();
    store_tile(wide, a.dh, a.F, row0, rows);
    product_t<2, KS, kSideAdd>(unit, ffn1, wide, dout, dy, wave, lane);
    load_first(unit, attn_out, wave, lane);
    lds_barrier();
  }
  ln_backward<D>(ln, a.F ? a.ln_b : a.ln_a, L, dout, nullptr, a.dy_out, dsub, sums, wave, lane);
  lds_barrier();
  store_sums<D>(sums, a.F ? a.ln_b.partial : a.ln_a.partial);
  product_t<2, KS, kNoSide>(unit, attn_out, dsub, wide, wide, wave, lane);
  lds_barrier();
  store_tile(wide, a.dO, D, row0, rows);
}

constexpr int64_t kLdsBytes = 160 * 1024;
int64_t fwd_lds(int d, int F, int wide, int n_proj) {
  const int unit = d == 256 ? 256 : d / 2;
  return (int64_t)sizeof(half_t) * (kRows * (3 * (d + kPad) + kWaves * (unit + kPad) + wide + kPad) + d + (F ? F + d : 0) + 3 * d * n_proj);
}
int64_t bwd_lds(int d, int wide) { return (int64_t)kRows * (3 * (d + kPad) + wide + kPad) * sizeof(half_t) + (int64_t)kWaves * 3 * d * sizeof(float); }

}  // namespace

bool row_chain_fits(int d, int F) {
  return (d == 64 || d == 128 || d == 256) && F % d == 0 && F <= 4 * d && fwd_lds(d, F, F > 3 * d ? F : 3 * d, kMaxRowChainProj) <= kLdsBytes &&
         bwd_lds(d, F > 3 * d ? F : 3 * d) <= kLdsBytes;
}
int row_chain_blocks(int rows) { return ceil_div(rows, kRows); }

int launch_row_chain_fwd(const RowChainFwd& a, int d, hipStream_t stream) {
  NMT_REQUIRE(a.rows > 0 && row_chain_fits(d, a.F ? a.F : d) && a.n_proj >= 0 && a.n_proj <= kMaxRowChainProj && a.ln1.drop.rowkey, "row chain: bad shape rows=%d d=%d F=%d", a.rows, d, a.F);
  int wide = a.F > d ? a.F : d;
  for (int i = 0; i < a.n_proj; ++i) {
    NMT_REQUIRE(a.proj[i].n > 0 && a.proj[i].n % d == 0 && a.proj[i].n <= 3 * d, "row chain: projection of %d columns", a.proj[i].n);
    wide = a.proj[i].n > wide ? a.proj[i].n : wide;
  }
  const size_t lds = (size_t)fwd_lds(d, a.F, wide, a.n_proj);
  auto run = [&](auto kernel) -> int {
    if (int rc = allow_lds(reinterpret_cast<const void*>(kernel), lds)) return rc;
    hipLaunchKernelGGL(kernel, dim3(row_chain_blocks(a.rows)), dim3(kThreads), lds, stream, a, wide + kPad);
    NMT_LAUNCH_CHECK();
    return NMT_OK;
  };
  return d == 64 ? run(row_chain_fwd_kernel<64>) : d == 128 ? run(row_chain_fwd_kernel<128>) : run(row_chain_fwd_kernel<256>);
}

int launch_row_chain_bwd(const RowChainBwd& a, int d, hipStream_t stream) {
  NMT_REQUIRE(a.rows > 0 && row_chain_fits(d, a.F ? a.F : d) && a.head_k % 64 == 0 && a.head_k <= 3 * d && a.ln_a.drop.rowkey, "row chain: bad shape rows=%d d=%d F=%d k=%d", a.rows, d,
              a.F, a.head_k);
  int wide = a.F > a.head_k ? a.F : a.head_k;
  wide = wide > d ? wide : d;
  const size_t lds = (size_t)bwd_lds(d, wide);
  auto run = [&](auto kernel) -> int {
    if (int rc = allow_lds(reinterpret_cast<const void*>(kernel), lds)) return rc;
    hipLaunchKernelGGL(kernel, dim3(row_chain_blocks(a.rows)), dim3(kThreads), lds, stream, a, wide + kPad);
    NMT_LAUNCH_CHECK();
    return NMT_OK;
  };
  const bool wide_loads = a.F >= kWaves * 128 && a.F % 128 == 0;  // (a tile of 128 columns for every wavefront)
  if (d == 64) return run(row_chain_bwd_kernel<64, 2>);
  if (d == 128) return run(row_chain_bwd_kernel<128, 2>);
  return wide_loads ? run(row_chain_bwd_kernel<256, 8>) : run(row_chain_bwd_kernel<256, 2>);
}
