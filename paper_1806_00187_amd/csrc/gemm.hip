// fp16-in / fp32-accumulate MFMA GEMM with LDS-staged tiles and a fused epilogue
// (bias, ReLU, dropout, residual/gradient add, ReLU-backward mask) for gfx950.
//
// C[M,N] = epilogue(sum_k A(m,k) * B(n,k)).  Either operand may be stored with the contraction
// index contiguous ("direct": [rows][K]) or with its other index contiguous ("transposed":
// [K][rows]).  This covers the three products of a linear layer: forward x W^T (both direct),
// input gradient dy W (B transposed) and weight gradient dy^T x (both transposed).
//
// Measured on this chip: ds_read_b128 streams ~200 B/clk per CU (the 8-byte transposing read half
// of that), global -> LDS loads ~50 B/clk per CU.  With fp16 data of full entropy the clock drops under matrix load
// (1.4-1.8 GHz), and how far depends on the instruction: 16x16x32 sustains 1820 TFLOP/s on register operands where
// 32x32x16 sustains 1580 (its result is read and written half as often per product), so that is the one used.  The loop is
// organised around the load path and around keeping the matrix pipe fed:
//  * global -> LDS directly (buffer_load ... lds, 16 bytes per lane, 1 KB contiguous per wave
//    instruction): no ds_write, no staging registers.  Every k-tile gets a buffer descriptor that
//    starts at the tile's first element and ends at its last, so out-of-range rows / k arrive as
//    zeros, ragged edges need no branches, and operands may be larger than 4 GB;
//  * both tile layouts are kept as they are in memory (direct [row][k], transposed [k][row]) and
//    made bank-conflict free by permuting, on the global-address side, which 16-byte chunk lands
//    in which slot (XOR swizzles chosen so that every LDS address is one per-lane base plus
//    compile-time offsets);
//  * LDS -> MFMA fragments: one ds_read_b128 per fragment for a direct tile; two
//    ds_read_b64_tr_b16 (the gfx950 transposing read: within 16 lanes, lane L receives element
//    L%4 of the 8-byte words addressed by lanes 4j + L/4, j = 0..3) for a transposed tile, so
//    no register shuffling is needed;
//  * the fragments of the next step are read while the MFMAs of the current one issue;
//  * a ring of 2 or 4 LDS stages of 64 k: the next 1 or 3 k-tiles stream in while one is multiplied; one
//    barrier per k-tile both publishes the next tile and frees the current one for refilling;
//  * the requests of a k-tile are spread between the MFMAs.  Issued in one go behind the barrier they hold up all
//    wavefronts of the compute unit at once (the path to memory takes 16 clocks for each) while the matrix pipes run dry:
//    8192^3, x W^T form, 867 -> 839 us, and 773 with the smaller matrix instruction.
#include <stdlib.h>

#include <mutex>
#include <type_traits>
#include <vector>

#include "common.h"

namespace {

constexpr int kThreads = 256;  // threads of the split-k reduction kernel
constexpr uint32_t kOob = 0x80000000u;  // byte offset no operand reaches: such loads return 0

typedef short short4_t __attribute__((ext_vector_type(4)));
typedef short short8_t __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(3))) short4_t* lds_short4_ptr;
typedef __attribute__((address_space(3))) void* lds_void_ptr;

// The order work-groups take the tiles of a launch in (see xcd_order), and those of one product (see place_tile).
struct XcdOrder {
  Divisor xcds;        // dies with their own L2: consecutive work-group ids go round-robin over them
  uint32_t base, rem;  // work-groups to a die: base, or one more on the first rem
};
XcdOrder xcd_runs(uint32_t total) {
  const uint32_t xcds = (uint32_t)device_info().xcds;
  return XcdOrder{divisor(xcds), total / xcds, total % xcds};
}
struct TileOrder {
  int tiles_m, group_m;
  Divisor tiles, per_group, rows, last_rows;  // tiles of the product; of group_m tile rows; group_m; rows of the last, shorter group
};
TileOrder tile_order(int tiles_m, int tiles_n) {
  // tile rows per sweep: the 32 tiles an XCD works on at a time form a patch of 4 rows x 8 columns (or
  // the result's whole width); between 2 and 8 the whole update is flat within 0.5 %, 4 measured best and
  // fetches least past L2, 12 and more cost 2 %
  int group_m = tuning().gemm_group;
  group_m = group_m < tiles_m ? group_m : tiles_m;  // (the same order; callers may ask for groups of any size, whose tiles have to be counted in 32 bits)
  return TileOrder{tiles_m, group_m, divisor((uint32_t)tiles_m * tiles_n), divisor(group_m * tiles_n), divisor(group_m),
                   divisor(tiles_m % group_m ? tiles_m % group_m : group_m)};
}
struct GemmArgs {
  const half_t* A;
  const half_t* B;
  half_t* C;
  int lda, ldb, ldc, M, N, K;
  GemmEpilogue ep;
  // split-K: work-group (tile, z) contracts k in [z * k_chunk, min(K, (z + 1) * k_chunk)) and writes its
  // fp32 tile to partial[z][M][N]; partial == nullptr: one work-group per tile, epilogue, fp16 result
  float* partial;
  int k_chunk;
  // column sums of A over k, for the products of a weight-gradient group: `colsum` where the product is not cut along
  // k, else `partial_colsum`, fp32 [z][M]
  half_t* colsum = nullptr;
  float* partial_colsum = nullptr;
  XcdOrder runs = {};
  TileOrder order = {};
  int keep = 0;  // the result is written through (else non-temporally): by the epilogues of TileStore; store_tile and the persistent form never do
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const half_t* p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<half_t*>(p), 0, (int)bytes, 0x00020000);
}
// One wave instruction: lane L's 16 bytes at byte offset `voff` of the buffer land at lds + 16 L.
// The whole offset travels in the per-lane operand, which is what the hardware range-checks.
__device__ __forceinline__ void dma16(__amdgpu_buffer_rsrc_t rsrc, unsigned char* lds_wave_base, uint32_t voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (lds_void_ptr)lds_wave_base, 16, (int)voff, 0, 0, 0);
}

// ---- direct operand: memory [rows][K] (k contiguous), LDS tile [R][BK k] -------------------------
// 128 bytes per row; slot p (16 bytes) of row r holds chunk p ^ (r >> 1 & 7): a wavefront's ds_read_b128 of 16 rows x 4 chunks
// touches every bank equally often, and so does any 16 lanes of it that take every row once.
// All offsets are relative to the first element of the block's current k-tile, so operands of any
// size work with 32-bit offsets.
constexpr int BK = 64;  // k of one stage
template <int R, int NW>
struct DirectOp {
  static constexpr int ROWB = BK * 2;             // bytes per tile row
  static constexpr int CPR = BK / 8;              // 16-byte chunks per row
  static constexpr int RPI = 64 / CPR;            // rows per wave instruction (1 KB)
  static constexpr int BYTES = R * ROWB;
  static constexpr int NV = BYTES / (1024 * NW);  // wave instructions per wave and k-tile
  static_assert(NV >= 1 && BYTES % (1024 * NW) == 0, "tile too small for the work-group's waves");
  uint32_t voff;   // of wave instruction 0; instruction `it` starts RPI * NW rows further on: its descriptor does, not the lane
  int c8, wave, ld;
  __device__ __forceinline__ static int swz(int row) { return (row >> 1) & 7; }
  // first element of the k-tile at k0 of the block whose first row is r0
  __device__ __forceinline__ static const half_t* origin(const half_t* p, int ld, int r0, int k0) { return p + (size_t)r0 * ld + k0; }
  // bytes from there to the end of the tile's last row (0 if the k-tile lies past K)
  __device__ __forceinline__ static uint32_t extent(int rows_in, int ld, int kleft) {
    const uint32_t e = ((uint32_t)(rows_in - 1) * ld + (uint32_t)min(kleft, BK)) * 2u;
    return e & (uint32_t)~((kleft - 1) >> 31);  // (masked, not selected: see TransOp)
  }
  __device__ __forceinline__ void init(int ld_in, int /*rows_in*/, int tid) {
    ld = ld_in;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = tid & 63, rowl = L / CPR, p = L % CPR;
    // RPI * (wave + NW it) adds nothing to the swizzle bits except bit 3 of the row (= wave & 1)
    c8 = (p ^ swz(RPI * wave + rowl)) << 3;
    voff = ((uint32_t)(RPI * wave + rowl) * (uint32_t)ld + (uint32_t)c8) * 2u;  // (rows past the last lie beyond the extent)
  }
  // One wave instruction after the other of a k-tile: `p` and `left`, its first element and its extent, move on with each.
  static constexpr int STEP = RPI * NW;  // rows (or, transposed, k rows) from one to the next
  __device__ __forceinline__ void load_next(const half_t*& p, int& left, int step, unsigned char* tile, int kleft, int it) const {
    dma16(make_rsrc(p, (uint32_t)max(left, 0)), tile + (wave + NW * it) * 1024, c8 < kleft ? voff : kOob);  // (only the last k-tile can fail this)
    p += step;
    left -= step * 2;
  }
  __device__ __forceinline__ void load(const half_t* p, uint32_t bytes, unsigned char* tile, int kleft) const {
    int left = (int)bytes;
#pragma unroll
    for (int it = 0; it < NV; ++it) load_next(p, left, STEP * ld, tile, kleft, it);
  }
  // per-lane fragment addresses, one per k-step (the swizzle is an XOR in the k-step bits)
  struct Frag {
    uint32_t a[BK / 32];
    __device__ __forceinline__ void fresh() {}
  };
  __device__ __forceinline__ static Frag frag_init(int row0, int lane) {
    Frag f;
    const int row = row0 + (lane & 15);  // row0 and the 16-row steps between MFMA tiles leave the swizzle bits alone
#pragma unroll
    for (int s = 0; s < BK / 32; ++s) f.a[s] = row * ROWB + ((((lane >> 4) | (4 * s)) ^ swz(lane & 15)) << 4);
    return f;
  }
  static constexpr int READS = 1;  // LDS instructions per fragment
  __device__ __forceinline__ static half8_t frag(const unsigned char* tile, const Frag& f, int i, int s) {
    return *reinterpret_cast<const half8_t*>(tile + f.a[s] + i * 16 * ROWB);
  }
};

// ---- transposed operand: memory [K][rows] (rows contiguous), LDS tile [BK k][R] -------------------
// Within k row k, slot q (16 bytes) holds chunk q ^ sw(k).  A transposing read serves 32 lanes at a
// time: two 16-lane groups (k 8 apart), each touching four k rows x two chunks.  With sw(k) = k & 3 in chunk bits 1 and 2, k & 8 in
// bit 3 (bit 0 counts the two chunks of a group) those sixteen chunks are all different, i.e. the 32 lanes cover every bank of a
// 256-byte row segment once.  (A 64-wide tile has only 8 chunks per k row, and two k rows side by side in a segment: there k & 2 and k & 8.)
template <int R, int NW>
struct TransOp {
  static constexpr int ROWB = R * 2;        // bytes per k row
  static constexpr int BYTES = BK * ROWB;
  static constexpr int NV = BYTES / (1024 * NW);
  static constexpr int CPR = R / 8;         // 16-byte chunks per k row
  static constexpr int KPI = 64 / CPR;      // k rows per wave instruction
  static_assert(NV >= 1 && BYTES % (1024 * NW) == 0, "tile too small for the work-group's waves");
  uint32_t voff;   // (as above: KPI * NW k rows further on)
  int wave, ld;
  __device__ __forceinline__ static int sw(int k) { return R == 64 ? ((k & 2) | ((k & 8) >> 1)) : (((k & 3) << 1) | (k & 8)); }
  __device__ __forceinline__ static const half_t* origin(const half_t* p, int ld, int r0, int k0) { return p + (size_t)k0 * ld + r0; }
  // k rows >= K lie beyond the extent and arrive as zeros.  (Masked, not selected: with a branch here the compiler's
  // count of the requests in flight came out low in the loops of every k-major product, and it put a wait for all but
  // six -- in the two-stage rings for all -- of them in front of the first fragment read after each k-tile's requests:
  // 128 x 64 tiles, 384 x 1024 x 1024: 13.1 -> 11.5 us.)
  __device__ __forceinline__ static uint32_t extent(int rows_in, int ld, int kleft) {
    const uint32_t e = ((uint32_t)(min(kleft, BK) - 1) * ld + (uint32_t)rows_in) * 2u;
    return e & (uint32_t)~((kleft - 1) >> 31);
  }
  __device__ __forceinline__ void init(int ld_in, int rows_in, int tid) {
    ld = ld_in;
    wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int L = tid & 63, kl = L / CPR, slot = L % CPR;
    // k row of instruction `it` is KPI * (wave + NW it) + kl: the same bits 0, 1 and 3 for every it
    static_assert(NV == 1 || KPI * NW % 16 == 0, "the swizzle of a lane's chunk must not change with `it`");
    const int cc = slot ^ sw(KPI * wave + kl);
    voff = cc * 8 < rows_in ? ((uint32_t)(KPI * wave + kl) * (uint32_t)ld + (uint32_t)(cc * 8)) * 2u : kOob;
  }
  static constexpr int STEP = KPI * NW;
  __device__ __forceinline__ void load_next(const half_t*& p, int& left, int step, unsigned char* tile, int /*kleft*/, int it) const {
    dma16(make_rsrc(p, (uint32_t)max(left, 0)), tile + (wave + NW * it) * 1024, voff);
    p += step;
    left -= step * 2;
  }
  __device__ __forceinline__ void load(const half_t* p, uint32_t bytes, unsigned char* tile, int kleft) const {
    int left = (int)bytes;
#pragma unroll
    for (int it = 0; it < NV; ++it) load_next(p, left, STEP * ld, tile, kleft, it);
  }
  static constexpr int READS = 2;
  // 16-lane group q = lane / 16 serves the tile's 16 rows and k 8 q .. 8 q + 7; lane i of the group
  // addresses k row i/4, row offset 4*(i%4) of its 4(k) x 16(row) block.  A step of one MFMA tile changes chunk bits 1 to 3, which
  // the swizzle flips: the address is flipped likewise, by an instruction of its own (eight addresses kept would not fit the large
  // tiles' registers; `fresh` keeps the compiler from keeping them all the same).
  struct Frag {
    uint32_t a;
    __device__ __forceinline__ void fresh() { asm volatile("" : "+v"(a)); }
  };
  __device__ __forceinline__ static Frag frag_init(int row0, int lane) {
    const int q = lane >> 4, i = lane & 15;
    const int kk = 8 * q + (i >> 2), r = row0 + 4 * (i & 3);  // (row0 is a multiple of the wave's rows: the bits of its tiles are free)
    return Frag{(uint32_t)(kk * ROWB + ((r >> 3) ^ sw(kk)) * 16 + (r & 7) * 2)};
  }
  __device__ __forceinline__ static half8_t frag(const unsigned char* tile, const Frag& f, int i, int s) {
    const unsigned char* p = tile + (f.a ^ (uint32_t)(i * 32)) + s * 32 * ROWB;
    const short4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(p));
    const short4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(p + 4 * ROWB));
    const short8_t r = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(half8_t, r);
  }
};

template <int BM, int BN, bool AT, bool BT, int NW>
struct Tile {
  using OpA = typename std::conditional<AT, TransOp<BM, NW>, DirectOp<BM, NW>>::type;
  using OpB = typename std::conditional<BT, TransOp<BN, NW>, DirectOp<BN, NW>>::type;
  static constexpr int STAGE = OpA::BYTES + OpB::BYTES;   // (BM + BN) * BK * 2 bytes
};

// s_waitcnt immediates (gfx9 encoding): at most n vector-memory operations outstanding, with or
// without also waiting for every LDS operation
constexpr int wait_vm(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0F70; }
constexpr int wait_vm_lds(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0070; }

// Work-group -> (k-split, tile).  Consecutive work-group ids go round-robin over the XCDs; undo
// that so each XCD (own L2) gets a contiguous run of tiles of as few k-splits as possible: the
// tiles of one split read the same k-range of A and B and share those panels in L2.
// Then grouped order: group_m tile rows are swept column by column, so the work-groups an XCD runs at a
// time form a patch of tiles and each A / B panel they stream is shared by several of them in L2.
__device__ __forceinline__ uint32_t xcd_order(uint32_t lin, const XcdOrder& o) {
  uint32_t xcd;
  const uint32_t idx = div_mod(lin, o.xcds, xcd);
  return xcd * o.base + min(xcd, o.rem) + idx;
}
__device__ __forceinline__ void place_tile(const TileOrder& o, uint32_t pid, int& tm, int& tn) {
  uint32_t in_group, row;
  const int first = (int)div_mod(pid, o.per_group, in_group) * o.group_m;
  tn = (int)div_mod(in_group, first + o.group_m <= o.tiles_m ? o.rows : o.last_rows, row);
  tm = first + (int)row;
}
__device__ __forceinline__ void place(const GemmArgs& g, uint32_t lin, int& split, int& tm, int& tn) {
  uint32_t pid;
  split = (int)div_mod(xcd_order(lin, g.runs), g.order.tiles, pid);
  place_tile(g.order, pid, tm, tn);
}

// What an epilogue does: nothing; bias; bias and ReLU; a sum with another matrix; the ReLU mask of the backward pass; whatever it is told,
// fp32 partial sums of a product cut along k among it; output scale or partial sums (weight gradients).  A kernel each for the
// first five: chosen per value they cost an instruction more each, and what is loaded for one form has to be waited for in all.
enum StoreForm { kStorePlain, kStoreBias, kStoreRelu, kStoreAdd, kStoreMask, kStoreAny, kStoreGroup };
typedef _Float16 half4v_t __attribute__((ext_vector_type(4)));
typedef float floatx8 __attribute__((ext_vector_type(8)));
typedef uint32_t uint4v_t __attribute__((ext_vector_type(4)));
constexpr int kStream = 2;         // non-temporal
constexpr int kWriteThrough = 16;  // device scope
// A result up to this size is written through to the last-level cache, where the next kernel finds it: a non-temporal one it reads from memory.  Larger ones
// push out what the kernels after it read: written through without a limit in every form, a batch of 26000 tokens in validation (results of 54 to 100 MB) took 4 % longer,
// 16 batches of Transformer-big 2.5 % longer forward.  Where the limit lies between is of no account, because larger results mostly come from 256 x 256 tiles, which never
// write through: 16, 32 and 64 MB time the same (Transformer-base on 2990 and 13000 tokens, -big on 2600 and 18000, validation), 8 MB costs
// Transformer-base on 2990 tokens 1161 / 1718 -> 1205 / 1771 us forward / backward.
constexpr int64_t kKeptBytes = 16ll << 20;
// 16 bytes at byte offset `off` (past the extent: zeros come back, nothing is stored)
__device__ __forceinline__ half8_t buffer_half8(__amdgpu_buffer_rsrc_t r, uint32_t off) {
  return __builtin_bit_cast(half8_t, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 0));
}
// streaming store: a result tile is not read again by its product, and letting it stay in L2 pushes out
// the operand panels the XCD's other tiles are reading (products with wide results: +5-7 %)
template <int POLICY = kStream>
__device__ __forceinline__ void buffer_store_half8(__amdgpu_buffer_rsrc_t r, uint32_t off, half8_t v) {
  __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(uint4v_t, v), r, (int)off, 0, POLICY);
}

// Epilogue of one tile whose form is known when it is compiled.  What it loads -- the bias of the lane's columns as the sums lie in registers, or what is added or
// masks in the pieces the results leave in -- is requested before the first operands, so that nothing is waited for behind the last product but LDS; the
// wavefront's whole share of the tile passes through LDS at once and leaves in whole rows, bounds by the descriptor of C, no branches.  (Loading the
// bias with each 32 rows, every load waited for the stores before it: with that and the order of tiles computed by division, 4.0 us of each product of a few
// hundred rows besides its k-tiles, whole forward pass of 3100 x 512 1360 us; now 1237.)
template <int BM, int BN, int NW, int STAGE, StoreForm FORM>
struct TileStore {
  static constexpr int WGN = NW / 2, WM = BM / 2, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  static constexpr bool kLoads = FORM == kStoreAdd || FORM == kStoreMask, kBias = FORM == kStoreBias || FORM == kStoreRelu;
  static constexpr int CH = WN / 8, RPI = 64 / CH, P = WM / RPI;  // 16-byte pieces of a row of results, rows to an instruction, pieces a lane
  static constexpr int HW = NW / 2, SHARE = WM * WN * (kLoads ? 4 : 2);
  static_assert(HW * SHARE <= STAGE, "half of the wavefronts' shares fit one stage");
  half4v_t bias[kBias ? TN : 1];
  half8_t pre[kLoads ? P : 1];
  uint32_t at, step;
  __device__ __forceinline__ void request(const GemmArgs& g, int m0, int n0, int rows, int cols, int wave, int lane) {
    const int wm = wave / WGN, wn = wave % WGN, col = wn * WN + lane % CH * 8;
    step = (uint32_t)RPI * (uint32_t)g.ldc * 2u;
    at = col < cols ? ((uint32_t)(wm * WM + lane / CH) * (uint32_t)g.ldc + (uint32_t)col) * 2u : kOob;
    if constexpr (kBias) {
      const __amdgpu_buffer_rsrc_t r = make_rsrc(g.ep.bias + n0, (uint32_t)cols * 2u);
#pragma unroll
      for (int j = 0; j < TN; ++j) bias[j] = __builtin_bit_cast(half4v_t, __builtin_amdgcn_raw_buffer_load_b64(r, (wn * WN + 16 * j + 4 * (lane >> 4)) * 2, 0, 0));
    }
    if constexpr (kLoads) {
      const __amdgpu_buffer_rsrc_t r = make_rsrc((FORM == kStoreAdd ? g.ep.add : g.ep.relu_src) + (size_t)m0 * g.ldc + n0,
                                                 ((uint32_t)(rows - 1) * (uint32_t)g.ldc + (uint32_t)cols) * 2u);
#pragma unroll
      for (int q = 0; q < P; ++q) pre[q] = buffer_half8(r, at + q * step);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void store(const GemmArgs& g, const floatx4 (&acc)[TM][TN], int m0, int n0, int rows, int cols, int wave, int lane,
                                        unsigned char* stage0, unsigned char* stage1) {
    unsigned char* const own = (wave < HW ? stage0 : stage1) + wave % HW * SHARE;
    const __amdgpu_buffer_rsrc_t to = make_rsrc(g.C + (size_t)m0 * g.ldc + n0, ((uint32_t)(rows - 1) * (uint32_t)g.ldc + (uint32_t)cols) * 2u);
    const int row = lane & 15, quad = lane >> 4, r0 = lane / CH, c8 = lane % CH;
    if constexpr (!kLoads) {
      // fp16; row r, 16-byte chunk c at r * 2 WN + (c ^ (r >> 1 & 7)) * 16, or, of 64 bytes, c ^ (r >> 2 & 3): 32 lanes' 8-byte pieces hit every bank once
      auto place = [&](int r, int c) { return own + r * (2 * WN) + ((CH == 8 ? c ^ (r >> 1 & 7) : c ^ (r >> 2 & 3)) << 4); };
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          floatx4 v = acc[i][j];
          if constexpr (kBias) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
              v[e] += (float)bias[j][e];
              if constexpr (FORM == kStoreRelu) v[e] = fmaxf(v[e], 0.f);
            }
          }
          *reinterpret_cast<half4v_t*>(place(16 * i + row, 2 * j + (quad >> 1)) + ((quad & 1) << 3)) = __builtin_convertvector(v, half4v_t);
        }
      wave_sync();
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const half8_t v = *reinterpret_cast<const half8_t*>(place(q * RPI + r0, c8));
        if (g.keep) buffer_store_half8<kWriteThrough>(to, at + q * step, v);
        else buffer_store_half8(to, at + q * step, v);
      }
    } else {
      // the sums as they are (one rounding, at the end); 16-byte chunks of four columns
      auto place = [&](int r, int c) { return own + r * (4 * WN) + ((WN == 64 ? c ^ (r & 15) : c ^ (r >> 1 & 7)) << 4); };
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<floatx4*>(place(16 * i + row, 4 * j + quad)) = acc[i][j];
      wave_sync();
#pragma unroll
      for (int q = 0; q < P; ++q) {
        const floatx4 lo = *reinterpret_cast<const floatx4*>(place(q * RPI + r0, 2 * c8)), hi = *reinterpret_cast<const floatx4*>(place(q * RPI + r0, 2 * c8 + 1));
        floatx8 v;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const float x = e < 4 ? lo[e] : hi[e - 4];
          v[e] = FORM == kStoreAdd ? x + (float)pre[q][e] : (float)pre[q][e] > 0.f ? x * g.ep.mask_scale : 0.f;
        }
        const half8_t o = __builtin_convertvector(v, half8_t);
        if (g.keep) buffer_store_half8<kWriteThrough>(to, at + q * step, o);
        else buffer_store_half8(to, at + q * step, o);
      }
    }
  }
};

// Epilogue of one tile of any form: accumulators -> per-wave LDS staging (fp32) -> row-wise 16-byte stores.
// PLAIN: the epilogue is the output scale alone (weight gradients).
template <int BM, int BN, int NW, int STAGE, bool PLAIN>
__device__ __forceinline__ void store_tile(const GemmArgs& g, const floatx4 (&acc)[BM / 32][BN / (16 * (NW / 2))], int m0, int n0, int split,
                                           unsigned char* stage0, unsigned char* stage1) {
  constexpr int WGN = NW / 2, WM = BM / 2, WN = BN / WGN, TM = WM / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  // The products were formed as (B tile) x (A tile)^T, so in the MFMA result layout lane l holds row
  // l%16 of a 16 x 16 tile of C and the four consecutive columns 4(l/16) .. +3: one 16-byte LDS write per tile.  A staged row is SW floats; its 16-byte chunks are
  // XOR-swizzled with the row so that 16 lanes (16 rows, same logical chunk) hit every bank once.
  // staging width per pass: the wave's whole width if NW waves x 32 rows of it fit one stage, else less
  // (half of the waves stage in stage0, the other half in stage1, so that a staged row can be 64 columns
  //  = whole 128-byte lines of fp16 output even when a stage is small)
  constexpr int HW = NW / 2;
  constexpr int SW = (HW * 32 * WN * 4 <= STAGE) ? WN : (HW * 32 * 64 * 4 <= STAGE && WN % 64 == 0) ? 64 : 32;
  static_assert(HW * 32 * SW * 4 <= STAGE, "epilogue staging does not fit");
  float* stg = reinterpret_cast<float*>(wave < HW ? stage0 : stage1) + (wave % HW) * (32 * SW);
  constexpr int CH = SW / 8;    // 8-column chunks per staged row
  constexpr int QC = SW / 4;    // 16-byte chunks per staged row (8, 16 or 32)
  auto swz = [](int row, int chunk) { return QC >= 16 ? (chunk ^ (row & 15)) : (chunk ^ ((row >> 1) & 7)); };
  const GemmEpilogue& ep = g.ep;
  // The addend (or the ReLU mask source) of the wave's whole share is requested up front, into registers
  // the fragments no longer need, so that its latency is paid once and behind the staging of the first rows
  // rather than once per 32 rows.  (Reading it all before any store is also what lets it alias C.)
  constexpr int kPre = TM * (WN / SW) * (CH / 2);
  constexpr bool PRELOAD = !PLAIN && kPre <= 16;
  const half_t* pre_src = ep.add ? ep.add : ep.relu_src;
  half8_t pre[PRELOAD ? kPre : 1];
  if constexpr (PRELOAD) {
    if (pre_src && !g.partial) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int jg = 0; jg < WN / SW; ++jg)
#pragma unroll
          for (int it = 0; it < CH / 2; ++it) {
            const int q = it * 64 + lane;
            const int gr = m0 + wm * WM + i * 32 + q / CH, gc = n0 + wn * WN + jg * SW + (q % CH) * 8;
            pre[(i * (WN / SW) + jg) * (CH / 2) + it] = (gr < g.M && gc < g.N) ? ld_half8(pre_src + (size_t)gr * g.ldc + gc) : zero_half8();
          }
    }
  }
#pragma unroll
  for (int i = 0; i < TM; ++i) {
#pragma unroll
    for (int jg = 0; jg < WN / SW; ++jg) {
      if (i || jg) wave_sync();  // the staging area is the wave's own: no work-group barrier needed
#pragma unroll
      for (int jj = 0; jj < SW / 16; ++jj)
#pragma unroll
        for (int ii = 0; ii < 2; ++ii) {
          const int row = ii * 16 + (lane & 15), chunk = jj * 4 + (lane >> 4);
          *reinterpret_cast<floatx4*>(stg + row * SW + swz(row, chunk) * 4) = acc[2 * i + ii][jg * (SW / 16) + jj];
        }
      wave_sync();
#pragma unroll
      for (int it = 0; it < CH / 2; ++it) {
        const int q = it * 64 + lane;
        const int rl = q / CH, c8 = q % CH;
        const int gr = m0 + wm * WM + i * 32 + rl, gc = n0 + wn * WN + jg * SW + c8 * 8;
        if (gr < g.M && gc < g.N) {
          float v[8];
          const floatx4 lo = *reinterpret_cast<const floatx4*>(stg + rl * SW + swz(rl, 2 * c8) * 4);
          const floatx4 hi = *reinterpret_cast<const floatx4*>(stg + rl * SW + swz(rl, 2 * c8 + 1) * 4);
          if (g.partial) {
            float* dst = g.partial + ((size_t)split * g.M + gr) * g.N + gc;
            *reinterpret_cast<floatx4*>(dst) = lo;
            *reinterpret_cast<floatx4*>(dst + 4) = hi;
            continue;
          }
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            v[e] = lo[e] * ep.out_scale;
            v[4 + e] = hi[e] * ep.out_scale;
          }
          const size_t off = (size_t)gr * g.ldc + gc;
          if constexpr (!PLAIN) {
            if (ep.bias) {
              const half8_t b = ld_half8(ep.bias + gc);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] += (float)b[e];
            }
            if (ep.relu) {
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] = fmaxf(v[e], 0.f);
            }
            if (ep.drop.thr) {
              const uint32_t bits = drop_keep8(ep.drop, (uint32_t)(gr + ep.row0), (uint32_t)gc >> 3);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] = ((bits >> e) & 1u) ? v[e] * ep.drop.scale : 0.f;
            }
            if (ep.add) {
              half8_t a;
              if constexpr (PRELOAD) a = pre[(i * (WN / SW) + jg) * (CH / 2) + it];
              else a = ld_half8(ep.add + off);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] += (float)a[e];
            }
            if (ep.relu_src) {
              half8_t h;
              if (PRELOAD && !ep.add) h = pre[(i * (WN / SW) + jg) * (CH / 2) + it];
              else h = ld_half8(ep.relu_src + off);
#pragma unroll
              for (int e = 0; e < 8; ++e) v[e] = ((float)h[e] > 0.f) ? v[e] * ep.mask_scale : 0.f;
            }
          }
          half8_t o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = (half_t)v[e];
          // streaming store: a result tile is not read again by this product, and letting it stay in L2 pushes out
          // the operand panels the XCD's other tiles are reading (products with wide results: +5-7 %)
          __builtin_nontemporal_store(o, reinterpret_cast<half8_t*>(g.C + off));
        }
      }
    }
  }
}

// Column sums of the A operand, the bias gradient of the weight-gradient products whose C tile this is.  The fragments are in
// registers anyway, so the bias gradients cost no pass over memory of their own; only the work-groups of the first tile column do it.
// A lane adds up the eight k of its row in each A fragment (lanes 16 q of a fragment hold its k 8 q .. 8 q + 7).  A row has two running
// sums, of the pieces of eight k of even and of odd number, each added up in increasing k: the order depends neither on the tile nor on
// the instruction the products are formed with (bias gradients are the updates' most sensitive sums: those of the keys are zero but for
// rounding).  Lanes 0..31 keep them for one strip, lanes 32..63 for the next: the swap puts q = 0 and 1 of both in one register, q = 2 and 3
// in the other.  Every wavefront of a row half has the same fragments, so each sums a pair of strips of its own: sixteen sub-batches
// of a 1024 wide model, whole update, 73.4 ms with all of them summing all strips, 72.1 so; an encoder layer's group over 3000 positions 512
// wide, alone, 40.5 and 34.0 us.
__device__ __forceinline__ float piece_sum(const half8_t& f) {
  typedef _Float16 half2v_t __attribute__((ext_vector_type(2)));
  struct Pairs { half2v_t p[4]; };
  const half2v_t ones = {(_Float16)1.f, (_Float16)1.f};
  const Pairs h = __builtin_bit_cast(Pairs, f);
  float s = 0.f;  // (the two-element product adds in fp32 and keeps denormal halves)
#pragma unroll
  for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_fdot2(h.p[e], ones, s, false);
  return s;
}
__device__ __forceinline__ void add_colsum(float& sum, float strip, float next_strip) {
  const auto halves = __builtin_amdgcn_permlane32_swap(__float_as_uint(strip), __float_as_uint(next_strip), false, false);
  sum += __uint_as_float(halves[0]);
  sum += __uint_as_float(halves[1]);
}
// (`pair`: the wavefront's place in its row half; it has summed strips 2 pair and 2 pair + 1, if there are so many)
template <int WGN, int TM>
__device__ __forceinline__ void store_colsum(const GemmArgs& g, float sum, int m0, int pair, int split) {
  static_assert(TM / 2 <= WGN, "a wavefront for each pair of strips");
  const int lane = threadIdx.x & 63;
  const float s = sum + __shfl_xor(sum, 16, kWave);
  const int row = m0 + pair * 32 + (lane >> 5) * 16 + (lane & 15);
  if (pair < TM / 2 && (lane & 16) == 0 && row < g.M) {
    if (g.partial) g.partial_colsum[(size_t)split * g.M + row] = s;
    else g.colsum[row] = (half_t)(s * g.ep.out_scale);
  }
}

// ------------------------------------------------------------------------------------------------
// Tiles multiplied strip by strip: 256 x 256 on eight wavefronts (2 x 4 of 128 x 64), one work-group per compute unit, and the tiles of
// which two or three work-groups share one (128 x 128, 128 x 64 on four wavefronts).  Two stages: while one k-tile is multiplied, the
// next is in LDS or on its way.  (The stages are separate arrays, so that the compiler can tell that fragment reads of one
// do not depend on the loads in flight into the other.)
// What bounds it: the power the chip may take (matrix pipes busy 0.7-0.8 of the cycles at 1.4-1.8 GHz) and, at k = 1024, the
// 3-5 us a tile takes besides its k-tiles.  TFLOP/s before (32x32x16, requests in one go, four stages of 32 for k-major operands) and
// now: 8192^3 x W^T 1268 / 1423, dy W 1244 / 1400, dy^T x 1251 / 1360; 52704 rows: 3072 x 1024 x W^T 1056 / 1150, 1024 x 4096 1116 / 1218,
// 4096 x 1024 dy W 1083 / 1140; a layer's weight gradients over 52700 positions 1024 wide 840 / 933
// (without and with each wavefront summing bias gradients of its own strips only, on another chip: 1017 / 1072).  Two stages of 64 k against
// four of 32 here: x W^T 760 / 808 us, dy W 773 / 793, dy^T x 794 / 805 (8192^3).
// ------------------------------------------------------------------------------------------------
// The product as an instruction of its own, so that the sums stay where they are: the compiler's form of this shape has a result
// apart from the addend, and its register allocation then moves accumulators about, runs out and spills inside the loop (a
// layer's weight gradients over 52700 positions 1024 wide: 1.65 -> 4.0 ms).  A result may be read (other than as the addend of
// the same sum) a few instructions later only; `settle` is between the loop and the epilogue.  Nothing here keeps the compiler from
// moving a source or a result about within that time, so tests/test_matrix_products_compiled.py looks for it in every kernel of
// the built library (there is none in that of AMD clang 22.0.0git, ROCm 7.2.0: 2 wait states ahead of a product, 19 behind it).
__device__ __forceinline__ void mfma_add(floatx4& acc, const half8_t& b, const half8_t& a) {
  asm volatile("v_mfma_f32_16x16x32_f16 %0, %1, %2, %0" : "+v"(acc) : "v"(b), "v"(a));
}
// Waits that the compiler puts around products it knows: the last results have arrived before they are read (at most 19 wait states;
// 16 for each strip of tiles here), and cleared sums are in place before the first product (2).
template <int TM, int TN>
__device__ __forceinline__ void settle_sums(floatx4 (&acc)[TM][TN]) {
  static_assert(TN == 2 || TN == 4, "two or four tiles in a strip");
#pragma unroll
  for (int i = TM - 1; i >= 0; --i) {
    if constexpr (TN == 4) asm volatile("s_nop 15" : "+v"(acc[i][0]), "+v"(acc[i][1]), "+v"(acc[i][2]), "+v"(acc[i][3]));
    else asm volatile("s_nop 15" : "+v"(acc[i][0]), "+v"(acc[i][1]));
  }
}
template <int BM, int BN, bool AT, bool BT, int NW, bool SUMS>
struct StripTile {
  static constexpr int WGN = NW / 2, WM = BM / 2, WN = BN / WGN, TM = WM / 16, TN = WN / 16;
  using T = Tile<BM, BN, AT, BT, NW>;
  using OpA = typename T::OpA;
  using OpB = typename T::OpB;
  const GemmArgs& g;
  int m0, n0, rows_a, rows_b, k_end;
  OpA opa;
  OpB opb;
  typename OpA::Frag fa;
  typename OpB::Frag fb;
  floatx4 acc[TM][TN];
  half8_t af[TM], bf[2][TN];
  float sum, strip_sum;  // column sums of strips 2 pair and 2 pair + 1, and the first one's current piece
  int pair;

  __device__ __forceinline__ explicit StripTile(const GemmArgs& args) : g(args) {}
  __device__ __forceinline__ void set_tile(int row, int col, int tid) {
    m0 = row;
    n0 = col;
    rows_a = min(g.M - m0, BM);
    rows_b = min(g.N - n0, BN);
    opa.init(g.lda, rows_a, tid);
    opb.init(g.ldb, rows_b, tid);
  }
  __device__ __forceinline__ void set_fragments(int wave, int lane) {
    fa = OpA::frag_init(wave / WGN * WM, lane);
    fb = OpB::frag_init(wave % WGN * WN, lane);
    pair = __builtin_amdgcn_readfirstlane(wave % WGN);
  }
  __device__ __forceinline__ void clear() {
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    settle();
    sum = 0.f;
  }
  __device__ __forceinline__ const half_t* origin_a(int k0) const { return OpA::origin(g.A, g.lda, m0, k0); }
  __device__ __forceinline__ const half_t* origin_b(int k0) const { return OpB::origin(g.B, g.ldb, n0, k0); }
  __device__ __forceinline__ uint32_t extent_a(int k0) const { return OpA::extent(rows_a, g.lda, k_end - k0); }
  __device__ __forceinline__ uint32_t extent_b(int k0) const { return OpB::extent(rows_b, g.ldb, k_end - k0); }
  // What is in flight when the loop starts: the first k-tile and the A half of the second (asynchronous).
  static constexpr int kAhead = OpA::NV;  // vector-memory instructions behind the first k-tile's
  __device__ __forceinline__ void request_first(unsigned char* s0, unsigned char* s1, int k0) const {
    opa.load(origin_a(k0), extent_a(k0), s0, k_end - k0);
    opb.load(origin_b(k0), extent_b(k0), s0 + OpA::BYTES, k_end - k0);
    opa.load(origin_a(k0 + BK), extent_a(k0 + BK), s1, k_end - k0 - BK);
    __builtin_amdgcn_sched_barrier(0);
  }
  __device__ __forceinline__ void first_fragments(const unsigned char* stage) {
#pragma unroll
    for (int i = 0; i < TM; ++i) af[i] = OpA::frag(stage, fa, i, 0);
#pragma unroll
    for (int j = 0; j < TN; ++j) bf[0][j] = OpB::frag(stage + OpA::BYTES, fb, j, 0);
  }
  __device__ __forceinline__ void add_strip(int i) {
    if (pair != i / 2) return;
    if (i & 1) add_colsum(sum, strip_sum, piece_sum(af[i]));
    else strip_sum = piece_sum(af[i]);
  }
  // One step of 32 k, S = 0 or 1 of a k-tile.  On entry its fragments are in registers, A in `af`, B in bf[S].  The step multiplies one
  // 16-row strip of A after the other; a strip's registers take its fragment of the next step (from stage `from`) once its
  // products are issued, B's go to the other set.  The second step of a k-tile changes stages, half its strips in: by then every
  // wave's last fragments of `to` have arrived and it has seen its own part of `from` land; the barrier publishes `from` and
  // frees `to`.  The A half of `to` is requested over the strips behind the barrier (k-tile at k0), the B half over the first strips
  // of the step after.
  // With REFILL false nothing is requested (a tile's last k-tiles).
  template <int S, bool REFILL = true>
  __device__ __forceinline__ void k_step(const unsigned char* from, unsigned char* to, int k0) {
    constexpr int kAt = S ? TM / 2 : 0, kBehind = TM - kAt;  // strips before the first read from `from`, and behind it
    constexpr int kReq = S ? OpA::NV : OpB::NV, kOver = S ? kBehind : TM / 2;  // requests, and the strips they are spread over
    const int kleft = k_end - k0;
    const half_t* at = S ? origin_a(k0) : origin_b(k0);
    int left = (int)(S ? extent_a(k0) : extent_b(k0)), step = S ? OpA::STEP * g.lda : OpB::STEP * g.ldb;
    asm volatile("" : "+s"(step));  // (multiples of it made ahead of the loop would fill the scalar registers)
    fa.fresh();
    fb.fresh();
#pragma unroll
    for (int i = 0; i < TM; ++i) {
      if (S && i == kAt) {
        __builtin_amdgcn_s_waitcnt(wait_vm_lds(0));
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
      }
#pragma unroll
      for (int jj = 0; jj < TN; ++jj) {  // B first: the result tile is transposed, lane = row of C, registers = columns
        const int j = i & 1 ? TN - 1 - jj : jj;  // (back and forth: from strip to strip B's operand stays, 0.2-1 % of the time, power again)
        mfma_add(acc[i][j], bf[S][j], af[i]);
      }
      if constexpr (SUMS) add_strip(i);
      __builtin_amdgcn_sched_barrier(0);  // (a read moved ahead of these products would take registers of its own)
      if (i >= kAt) {
        const int r = i - kAt;
#pragma unroll
        for (int j = r; j < TN; j += kBehind) bf[S ^ 1][j] = OpB::frag(from + OpA::BYTES, fb, j, S ^ 1);
        if (S && i == kAt) {
#pragma unroll
          for (int t = 0; t < kAt; ++t) af[t] = OpA::frag(from, fa, t, S ^ 1);
        }
        af[i] = OpA::frag(from, fa, i, S ^ 1);
#pragma unroll
        for (int q = r * kReq / kOver; REFILL && q < (r + 1) * kReq / kOver && q < kReq; ++q) {
          if (S) opa.load_next(at, left, step, to, kleft, q);
          else opb.load_next(at, left, step, to + OpA::BYTES, kleft, q);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  // The last step of all: its products alone.
  __device__ __forceinline__ void last_step() {
#pragma unroll
    for (int i = 0; i < TM; ++i) {
#pragma unroll
      for (int j = 0; j < TN; ++j) mfma_add(acc[i][j], bf[1][j], af[i]);
      if constexpr (SUMS) add_strip(i);
    }
  }
  // The k-tiles come in pairs; of an odd number the last one's partner reads zeros (it lies outside the extent of its buffer
  // descriptor) and multiplying it changes nothing.
  __device__ __forceinline__ void multiply(unsigned char* s0, unsigned char* s1, int k0) {
    const int nk = (k_end - k0 + BK - 1) / BK;
    // (the large tile's loop runs to the end, past which its requests read zeros: it has the registers for one loop only)
    constexpr int kPeeled = NW == 4 ? 2 : 0;
    int k = k0;
    for (int left = nk; left > kPeeled; left -= 2, k += 2 * BK) {
      k_step<0>(s0, s1, k + BK);
      k_step<1>(s1, s0, k + 2 * BK);
      k_step<0>(s1, s0, k + 2 * BK);
      k_step<1>(s0, s1, k + 3 * BK);
    }
    if constexpr (kPeeled > 0) {
      k_step<0>(s0, s1, k + BK);
      k_step<1, false>(s1, s0, 0);
      k_step<0, false>(s1, s0, 0);
      last_step();
    }
    settle();
  }
  __device__ __forceinline__ void settle() { settle_sums(acc); }
};
// One tile by one work-group.
template <int BM, int BN, bool AT, bool BT, int NW, bool SUMS, StoreForm FORM>
__device__ __forceinline__ void gemm_tile(const GemmArgs& g, int split, int tm, int tn, unsigned char* stage0, unsigned char* stage1) {
  using L = StripTile<BM, BN, AT, BT, NW, SUMS>;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const bool cut = FORM >= kStoreAny && g.partial;
  const int k_base = cut ? split * g.k_chunk : 0;
  L t(g);
  t.k_end = cut ? min(g.K, k_base + g.k_chunk) : g.K;
  t.set_tile(tm * BM, tn * BN, tid);
  TileStore<BM, BN, NW, L::T::STAGE, FORM < kStoreAny ? FORM : kStorePlain> out;
  if constexpr (FORM < kStoreAny) out.request(g, t.m0, t.n0, t.rows_a, t.rows_b, wave, lane);
  t.set_fragments(wave, lane);
  t.clear();
  t.request_first(stage0, stage1, k_base);
  __builtin_amdgcn_s_waitcnt(wait_vm(L::kAhead));
  __builtin_amdgcn_s_barrier();
  t.first_fragments(stage0);
  t.multiply(stage0, stage1, k_base);
  __builtin_amdgcn_s_waitcnt(wait_vm_lds(0));  // the last refills (all zeros) must land before the stages are reused
  __syncthreads();
  if constexpr (SUMS) {
    store_colsum<L::WGN, L::TM>(g, t.sum, t.m0 + wave / L::WGN * L::WM, t.pair, split);
  }
  if constexpr (FORM < kStoreAny) out.store(g, t.acc, t.m0, t.n0, t.rows_a, t.rows_b, wave, lane, stage0, stage1);
  else store_tile<BM, BN, NW, L::T::STAGE, FORM == kStoreGroup>(g, t.acc, t.m0, t.n0, split, stage0, stage1);
}
template <int BM, int BN, bool AT, bool BT, int NW, StoreForm FORM>
__global__ void __launch_bounds__(64 * NW) gemm_kernel(const GemmArgs g) {
  touch(g);
  using T = Tile<BM, BN, AT, BT, NW>;
  __shared__ __align__(1024) unsigned char stage0[T::STAGE];
  __shared__ __align__(1024) unsigned char stage1[T::STAGE];
  int split, tm, tn;
  place(g, blockIdx.x + blockIdx.y * g.order.tiles.d, split, tm, tn);
  gemm_tile<BM, BN, AT, BT, NW, false, FORM>(g, split, tm, tn, stage0, stage1);
}

// ------------------------------------------------------------------------------------------------
// Tiles of up to 128 x 128: products with too few rows for 256 x 256 tiles.  Such a product is one round of
// work-groups that each walk 8 to 64 k-tiles, so its time is a fixed part (launch, first operands, epilogue: 4-5 us)
// plus k-tiles x the time of one.  What bounds a k-tile here is its trip through the vector-memory unit (64 bytes per
// clock and compute unit; 43 reached), as long as two things do not come first: the latency of the requests, so the
// ring has four stages and three k-tiles are in flight; and the latency of the fragment reads (a k-step of a small
// tile has 1 to 4 matrix instructions, less than the ~120 clocks of an LDS read), so a whole k-tile of fragments is
// held in registers and the next k-tile's are read behind all matrix instructions of the current one.  Per 64-deep k-tile on
// one work-group per compute unit: 64 x 64 0.42 -> 0.165 us, 128 x 64 0.48 -> 0.24, 128 x 128 0.55 -> 0.33 (0.45 with every
// compute unit busy) against the same tiles with two stages and one k-step of fragments ahead; 3000 x 1024 x 4096: 42.4 -> 33.2 us,
// 384 x 1024 x 1024: 11.5 -> 6.5 us, 384 x 1024 x 4096: 34.4 -> 14.4 us.
// The two-stage ring remains for 128 x 128 tiles on four wavefronts, two work-groups per compute unit, where there are
// enough tiles for that: the second work-group's k-tiles then cover the first one's prologue and epilogue.
// ------------------------------------------------------------------------------------------------
template <int BM, int BN, bool AT, bool BT, int NW, bool SUMS, StoreForm FORM>
__device__ __forceinline__ void gemm_small_tile(const GemmArgs& g, int split, int tm, int tn, unsigned char* stage0, unsigned char* stage1,
                                                unsigned char* stage2, unsigned char* stage3) {
  constexpr int NS = 4;
  using T = Tile<BM, BN, AT, BT, NW>;
  using OpA = typename T::OpA;
  using OpB = typename T::OpB;
  constexpr int WGN = NW / 2, WM = BM / 2, WN = BN / WGN, TM = WM / 16, TN = WN / 16, KS = BK / 32;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WGN, wn = wave % WGN;
  const int m0 = tm * BM, n0 = tn * BN;
  float colsum = 0.f, strip_sum = 0.f;  // (as in StripTile)
  const int pair = __builtin_amdgcn_readfirstlane(wn);

  floatx4 acc[TM][TN];
#pragma unroll
  for (int i = 0; i < TM; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

  OpA opa;
  OpB opb;
  const int rows_a = min(g.M - m0, BM), rows_b = min(g.N - n0, BN);
  opa.init(g.lda, rows_a, tid);
  opb.init(g.ldb, rows_b, tid);
  const typename OpA::Frag fa = OpA::frag_init(wm * WM, lane);
  const typename OpB::Frag fb = OpB::frag_init(wn * WN, lane);
  const bool cut = FORM >= kStoreAny && g.partial;
  const int k_base = cut ? split * g.k_chunk : 0;
  const int k_end = cut ? min(g.K, k_base + g.k_chunk) : g.K;
  TileStore<BM, BN, NW, T::STAGE, FORM < kStoreAny ? FORM : kStorePlain> out;
  if constexpr (FORM < kStoreAny) out.request(g, m0, n0, rows_a, rows_b, wave, lane);
  auto request = [&](unsigned char* stage, int k0) {
    const int kleft = k_end - k0;
    opa.load(OpA::origin(g.A, g.lda, m0, k0), OpA::extent(rows_a, g.lda, kleft), stage, kleft);
    opb.load(OpB::origin(g.B, g.ldb, n0, k0), OpB::extent(rows_b, g.ldb, kleft), stage + OpA::BYTES, kleft);
  };
  constexpr int kPerTile = OpA::NV + OpB::NV;
  half8_t af[2][KS][TM], bf[2][KS][TN];  // the fragments of two consecutive k-tiles
  auto fetch = [&](const unsigned char* stage, int set) {
#pragma unroll
    for (int s = 0; s < KS; ++s) {
#pragma unroll
      for (int i = 0; i < TM; ++i) af[set][s][i] = OpA::frag(stage, fa, i, s);
#pragma unroll
      for (int j = 0; j < TN; ++j) bf[set][s][j] = OpB::frag(stage + OpA::BYTES, fb, j, s);
    }
  };
  // One k-tile, whose fragments are in register set `set`, product by product; between them go the reads of the next k-tile's fragments
  // from `nxt` (if there is one; over the first three quarters, so that every read has returned before they are needed) and the requests that
  // refill `cur` (if there is something to refill it with).
  constexpr int kProducts = KS * TM * TN, kReadUnits = KS * (TM + TN), kReadOver = kProducts - kProducts / 4;
  auto interleaved = [&](unsigned char* cur, const unsigned char* nxt, int k_refill, int set, auto reads, auto refill) {
    const int kleft = k_end - k_refill;
    const half_t *pa = OpA::origin(g.A, g.lda, m0, k_refill), *pb = OpB::origin(g.B, g.ldb, n0, k_refill);
    int left_a = (int)OpA::extent(rows_a, g.lda, kleft), left_b = (int)OpB::extent(rows_b, g.ldb, kleft);
#pragma unroll
    for (int q = 0; q < kProducts; ++q) {
      const int s = q / (TM * TN), i = q / TN % TM, j = q % TN;  // (k-steps in increasing order: the same sums as gemm_kernel's)
      acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_f16(bf[set][s][j], af[set][s][i], acc[i][j], 0, 0, 0);
      if constexpr (SUMS) {
        if (j == 0 && pair == i / 2) {
          if (i & 1) add_colsum(colsum, strip_sum, piece_sum(af[set][s][i]));
          else strip_sum = piece_sum(af[set][s][i]);
        }
      }
      if constexpr (reads()) {
#pragma unroll
        for (int r = q * kReadUnits / kReadOver; r < (q + 1) * kReadUnits / kReadOver && r < kReadUnits; ++r) {
          const int rs = r / (TM + TN), ri = r % (TM + TN);
          if (ri < TN) bf[set ^ 1][rs][ri] = OpB::frag(nxt + OpA::BYTES, fb, ri, rs);
          else af[set ^ 1][rs][ri - TN] = OpA::frag(nxt, fa, ri - TN, rs);
        }
      }
      if constexpr (refill()) {
#pragma unroll
        for (int v = q * kPerTile / kProducts; v < (q + 1) * kPerTile / kProducts; ++v) {
          if (v < OpA::NV) opa.load_next(pa, left_a, OpA::STEP * g.lda, cur, kleft, v);
          else opb.load_next(pb, left_b, OpB::STEP * g.ldb, cur + OpA::BYTES, kleft, v - OpA::NV);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // The barrier publishes `nxt` (every wave has seen its own part of it land; `later` k-tiles are on their way behind it)
  // and frees `cur` (every wave's fragments of it have arrived), which is refilled at once.
  auto change = [&](auto later) {
    __builtin_amdgcn_s_waitcnt(wait_vm_lds(later() * kPerTile));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
  };
  auto k_tile = [&](unsigned char* cur, const unsigned char* nxt, int k_refill, int set) {
    change(std::integral_constant<int, NS - 2>{});
    interleaved(cur, nxt, k_refill, set, std::true_type{}, std::true_type{});
  };
  auto last_four = [&](const unsigned char* second, const unsigned char* third, const unsigned char* fourth, int set) {
    change(std::integral_constant<int, 2>{});
    interleaved(nullptr, second, 0, set, std::true_type{}, std::false_type{});
    change(std::integral_constant<int, 1>{});
    interleaved(nullptr, third, 0, set ^ 1, std::true_type{}, std::false_type{});
    change(std::integral_constant<int, 0>{});
    interleaved(nullptr, fourth, 0, set, std::true_type{}, std::false_type{});
    interleaved(nullptr, nullptr, 0, set ^ 1, std::false_type{}, std::false_type{});
  };

  // Nothing is requested past the end of the contraction: a request whose lanes are all out of bounds takes its turn on the way to memory like
  // any other, and the end of a product waited for four k-tiles of them (as nodes of a graph: 136 x 64 x 64 5.04 -> 3.90 us, 380 x 1024 x 1024
  // 5.80 -> 5.54, 380 x 4096 x 1024 8.54 -> 7.95, 1670 x 256 x 1024 5.91 -> 5.59).
  // (Not on eight wavefronts: the code of the last k-tiles takes registers, and those are left to others there; k-tiles past the end are
  // requested as zeros and multiplied.)
  const int nk = (k_end - k_base + BK - 1) / BK;
  if constexpr (NW == 8) {
    request(stage0, k_base);
    request(stage1, k_base + BK);
    request(stage2, k_base + 2 * BK);
    request(stage3, k_base + 3 * BK);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm((NS - 1) * kPerTile));
    __builtin_amdgcn_s_barrier();
    fetch(stage0, 0);
    for (int kt = 0; kt < nk; kt += NS) {
      k_tile(stage0, stage1, k_base + (kt + 4) * BK, 0);
      k_tile(stage1, stage2, k_base + (kt + 5) * BK, 1);
      k_tile(stage2, stage3, k_base + (kt + 6) * BK, 0);
      k_tile(stage3, stage0, k_base + (kt + 7) * BK, 1);
    }
  } else if (nk >= NS) {
    request(stage0, k_base);
    request(stage1, k_base + BK);
    request(stage2, k_base + 2 * BK);
    request(stage3, k_base + 3 * BK);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm((NS - 1) * kPerTile));
    __builtin_amdgcn_s_barrier();
    fetch(stage0, 0);
    int k = k_base + NS * BK, left = nk - NS;  // `left` k-tiles are not requested yet
    for (; left >= NS; k += NS * BK, left -= NS) {
      k_tile(stage0, stage1, k, 0);
      k_tile(stage1, stage2, k + BK, 1);
      k_tile(stage2, stage3, k + 2 * BK, 0);
      k_tile(stage3, stage0, k + 3 * BK, 1);
    }
    if (left == 0) {
      last_four(stage1, stage2, stage3, 0);
    } else if (left == 1) {
      k_tile(stage0, stage1, k, 0);
      last_four(stage2, stage3, stage0, 1);
    } else if (left == 2) {
      k_tile(stage0, stage1, k, 0);
      k_tile(stage1, stage2, k + BK, 1);
      last_four(stage3, stage0, stage1, 0);
    } else {
      k_tile(stage0, stage1, k, 0);
      k_tile(stage1, stage2, k + BK, 1);
      k_tile(stage2, stage3, k + 2 * BK, 0);
      last_four(stage0, stage1, stage2, 1);
    }
  } else if (nk > 0) {
    request(stage0, k_base);
    if (nk > 1) request(stage1, k_base + BK);
    if (nk > 2) request(stage2, k_base + 2 * BK);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_waitcnt(wait_vm(0));
    __builtin_amdgcn_s_barrier();
    fetch(stage0, 0);
    interleaved(nullptr, nullptr, 0, 0, std::false_type{}, std::false_type{});
    if (nk > 1) {
      fetch(stage1, 0);
      interleaved(nullptr, nullptr, 0, 0, std::false_type{}, std::false_type{});
    }
    if (nk > 2) {
      fetch(stage2, 0);
      interleaved(nullptr, nullptr, 0, 0, std::false_type{}, std::false_type{});
    }
  }
  __builtin_amdgcn_s_waitcnt(wait_vm_lds(0));  // every wave has its last fragments, and every request has landed, before the stages are reused
  __syncthreads();
  if constexpr (SUMS) {
    store_colsum<WGN, TM>(g, colsum, m0 + wm * WM, pair, split);
  }
  if constexpr (FORM < kStoreAny) out.store(g, acc, m0, n0, rows_a, rows_b, wave, lane, stage0, stage1);
  else store_tile<BM, BN, NW, T::STAGE, FORM == kStoreGroup>(g, acc, m0, n0, split, stage0, stage1);
}
template <int BM, int BN, bool AT, bool BT, int NW, StoreForm FORM>
__device__ __forceinline__ void gemm_small_group(const GemmArgs& g) {
  touch(g);
  using T = Tile<BM, BN, AT, BT, NW>;
  __shared__ __align__(1024) unsigned char stage0[T::STAGE];  // separate arrays (see StripTile)
  __shared__ __align__(1024) unsigned char stage1[T::STAGE];
  __shared__ __align__(1024) unsigned char stage2[T::STAGE];
  __shared__ __align__(1024) unsigned char stage3[T::STAGE];
  int split, tm, tn;
  place(g, blockIdx.x + blockIdx.y * g.order.tiles.d, split, tm, tn);
  gemm_small_tile<BM, BN, AT, BT, NW, false, FORM>(g, split, tm, tn, stage0, stage1, stage2, stage3);
}
template <int BM, int BN, bool AT, bool BT, int NW, StoreForm FORM>
__global__ void __launch_bounds__(64 * NW) gemm_small_kernel(const GemmArgs g) {
  gemm_small_group<BM, BN, AT, BT, NW, FORM>(g);
}
// Eight wavefronts: one such work-group fills a compute unit's LDS.  Registers for a third wavefront per SIMD (160 of 512) are left, so that the other
// stream's row kernels can run beside it (LayerNorm backward of a 512 wide model over 3000 positions, a third of the calls beside a layer's weight
// gradients: 16.8 us on average with 220 registers here, 14.1 with 154).  The attribute counts half of the register file.
template <int BM, int BN, bool AT, bool BT, StoreForm FORM>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_num_vgpr(88))) gemm_small_kernel_8(const GemmArgs g) {
  gemm_small_group<BM, BN, AT, BT, 8, FORM>(g);
}

// ------------------------------------------------------------------------------------------------
// Persistent form of the 256 x 256, 8-wave kernel: one work-group per compute unit walks its tiles (the same tile -> XCD assignment
// as above) in one unbroken sequence of k-tiles.  The requests that the last k-tiles of a tile would make past its end are the
// first ones of the next tile, and the fragment reads of its last step are the next tile's first, so that between the
// last product of a tile and the first of the next there is the epilogue and nothing else: no drained ring, no first operands to
// wait for.  The epilogue leaves the stages and the fragments' registers alone: results pass through the 32 KB of LDS that the stage
// ring leaves free (wave-private, so no work-group barrier) and leave as whole 128-byte rows.  Bounds are checked by the
// buffer descriptors of C and of what the epilogue loads, so it has no branches per row.
// Before (next tile's first k-tiles requested in one go after the last product, one epilogue for all forms with a select per value,
// sum and mask in the form with one tile per work-group) and now, us, 52704 rows: 4096 x 1024 with bias and ReLU 383 / 360, 1024 x 1024 104 /
// 99, 32768 x 1024 3079 / 2810, + another matrix 1024 x 4096 421 / 375, ReLU mask 4096 x 1024 502 / 425; 26000 x 2048 x 512 with mask 89 / 73.
// What is left per tile besides its k-tiles is 3-4 us at k = 1024 (5 before); the k-tiles are bound by power (see StripTile).
// ------------------------------------------------------------------------------------------------
// LDS accesses of the staging rows, written as instructions: while requests into the stages are in
// flight the compiler would otherwise put a wait for ALL of them in front of any LDS access it
// cannot tell apart from their targets.
__device__ __forceinline__ uint32_t lds_addr(const void* p) { return (uint32_t)(uintptr_t)(lds_void_ptr)p; }
// eight 8-byte writes: one 32 x 64 slab of results (the lane's four consecutive columns in two rows of four column groups)
__device__ __forceinline__ void out_write_slab(const uint32_t (&a)[8], const half4v_t (&v)[8]) {
  asm volatile(
      "ds_write_b64 %0, %8\n\tds_write_b64 %1, %9\n\tds_write_b64 %2, %10\n\tds_write_b64 %3, %11\n\t"
      "ds_write_b64 %4, %12\n\tds_write_b64 %5, %13\n\tds_write_b64 %6, %14\n\tds_write_b64 %7, %15"
      :
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(a[4]), "v"(a[5]), "v"(a[6]), "v"(a[7]), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3]),
        "v"(v[4]), "v"(v[5]), "v"(v[6]), "v"(v[7])
      : "memory");
}
// four 16-byte writes: one 16 x 64 slab of sums
__device__ __forceinline__ void out_write_sums(const uint32_t (&a)[4], const floatx4 (&v)[4]) {
  asm volatile("ds_write_b128 %0, %4\n\tds_write_b128 %1, %5\n\tds_write_b128 %2, %6\n\tds_write_b128 %3, %7"
               :
               : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3]), "v"(v[0]), "v"(v[1]), "v"(v[2]), "v"(v[3])
               : "memory");
}
// the slab back as rows: four 16-byte reads, returned once all have arrived (LDS operations of a wave complete in
// order, so the writes above are done too); one instruction sequence, so that nothing touches the registers between
// the reads and the wait
template <typename V>
__device__ __forceinline__ void out_read_slab(const uint32_t (&a)[4], V (&d)[4]) {
  asm volatile(
      "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
      "s_waitcnt lgkmcnt(0)"
      : "=&v"(d[0]), "=&v"(d[1]), "=&v"(d[2]), "=&v"(d[3])
      : "v"(a[0]), "v"(a[1]), "v"(a[2]), "v"(a[3])
      : "memory");
}
template <bool BT, StoreForm FORM>
__global__ void __launch_bounds__(512) gemm_persistent_kernel(const GemmArgs g) {
  constexpr int BM = 256, BN = 256, NW = 8;
  using L = StripTile<BM, BN, false, BT, NW, false>;
  static_assert(2 * L::T::STAGE == 128 * 1024, "the ring takes 128 KB; the staging rows take the 32 KB that are left");
  __shared__ __align__(1024) unsigned char stage0[L::T::STAGE];  // separate arrays (see StripTile)
  __shared__ __align__(1024) unsigned char stage1[L::T::STAGE];
  constexpr int kOutBytes = 4096;  // staging of a wave: 32 rows of 64 fp16, or 16 rows of 64 fp32
  __shared__ __align__(16) unsigned char out_rows[NW * kOutBytes];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / L::WGN, wn = wave % L::WGN;
  const int nt = (int)g.order.tiles.d;

  L t(g);
  t.k_end = g.K;
  auto set_tile = [&](int lin) {
    int split, tm, tn;
    place(g, (uint32_t)lin, split, tm, tn);
    t.set_tile(tm * BM, tn * BN, tid);
  };
  const GemmEpilogue& ep = g.ep;
  const uint32_t out = lds_addr(out_rows) + wave * kOutBytes;
  const int last = ((g.K + BK - 1) / BK + 1) / 2 * 2;  // k-tiles of a tile, an even number (one past the end multiplies zeros)

  int lin = blockIdx.x;
  set_tile(lin);
  t.set_fragments(wave, lane);
  t.request_first(stage0, stage1, 0);
  __builtin_amdgcn_s_waitcnt(wait_vm(L::kAhead));
  __builtin_amdgcn_s_barrier();
  t.first_fragments(stage0);
  for (;;) {
    t.clear();
    for (int kt = 0; kt + 2 < last; kt += 2) {
      t.template k_step<0>(stage0, stage1, (kt + 1) * BK);
      t.template k_step<1>(stage1, stage0, (kt + 2) * BK);
      t.template k_step<0>(stage1, stage0, (kt + 2) * BK);
      t.template k_step<1>(stage0, stage1, (kt + 3) * BK);
    }
    // the last two k-tiles: from the stage change on, requests and fragment reads are the next tile's (there is none: past the end)
    t.template k_step<0>(stage0, stage1, (last - 1) * BK);
    const int m0 = t.m0, n0 = t.n0, rows = t.rows_a, cols = t.rows_b;
    lin += (int)gridDim.x;
    const bool more = lin < nt;
    if (more) set_tile(lin);
    const int k_next = more ? 0 : t.k_end;
    half4v_t bias[L::TN];
    if constexpr (FORM == kStoreBias || FORM == kStoreRelu) {
      // the bias of the lane's columns in the MFMA layout (16 j + 4 (lane / 16) .. + 3 of the wave's 64; no bias: extent 0), waited for
      // with the operands at the next stage change
      const __amdgpu_buffer_rsrc_t r = make_rsrc(ep.bias + n0, ep.bias ? (uint32_t)cols * 2u : 0u);
#pragma unroll
      for (int j = 0; j < L::TN; ++j)
        bias[j] = __builtin_bit_cast(half4v_t, __builtin_amdgcn_raw_buffer_load_b64(r, (wn * L::WN + 16 * j + 4 * (lane >> 4)) * 2, 0, 0));
    }
    t.template k_step<1>(stage1, stage0, k_next);
    t.template k_step<0>(stage1, stage0, k_next);
    t.template k_step<1>(stage0, stage1, k_next + BK);
    t.settle();

    // ---- epilogue of the tile at (m0, n0) ----
    // a lane's piece of a staged row: eight columns, in rows lane / 8, + 8, + 16, ... of the wave's 128
    const int c8 = lane & 7, r8 = lane >> 3, quad = lane >> 4, row = lane & 15;
    const uint32_t extent = ((uint32_t)(rows - 1) * (uint32_t)g.ldc + (uint32_t)cols) * 2u;
    const __amdgpu_buffer_rsrc_t to = make_rsrc(g.C + (size_t)m0 * g.ldc + n0, extent);
    const int col = wn * L::WN + c8 * 8;
    const uint32_t step = 16u * (uint32_t)g.ldc;  // bytes of eight rows
    uint32_t at = col < cols ? ((uint32_t)(wm * L::WM + r8) * (uint32_t)g.ldc + (uint32_t)col) * 2u : kOob;
    if constexpr (FORM <= kStoreRelu) {
      // accumulators -> fp16 -> 32 staged rows -> 16-byte pieces of whole rows.  Staged row r, 16-byte chunk c (eight columns) at
      // r * 128 + (c ^ (r >> 1 & 7)) * 16: the eight lanes that read a row back cover its 128 bytes, and the 8-byte pieces that 32 lanes
      // write every bank once.
#pragma unroll
      for (int i = 0; i < L::TM / 2; ++i) {
        uint32_t wa[8];
        half4v_t wv[8];
#pragma unroll
        for (int j = 0; j < L::TN; ++j)
#pragma unroll
          for (int ii = 0; ii < 2; ++ii) {
            floatx4 v = t.acc[2 * i + ii][j];
            if constexpr (FORM != kStorePlain) {
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                v[e] += (float)bias[j][e];
                if constexpr (FORM == kStoreRelu) v[e] = fmaxf(v[e], 0.f);
              }
            }
            wv[2 * j + ii] = __builtin_convertvector(v, half4v_t);
            wa[2 * j + ii] = out + (16 * ii + row) * 128 + (((2 * j + (quad >> 1)) ^ (row >> 1)) << 4) + ((quad & 1) << 3);
          }
        out_write_slab(wa, wv);   // (the reads of the previous slab have returned: out_read_slab waits for them)
        uint32_t ra[4];
        half8_t rv[4];
#pragma unroll
        for (int it = 0; it < 4; ++it) {
          const int rl = it * 8 + r8;
          ra[it] = out + rl * 128 + ((c8 ^ (rl >> 1 & 7)) << 4);
        }
        out_read_slab(ra, rv);
#pragma unroll
        for (int it = 0; it < 4; ++it, at += step) buffer_store_half8(to, at, rv[it]);
      }
    } else {
      // what is added, or masks, comes in the pieces the results leave in, eight at a time; the sums are staged as they are, 16 rows
      // at a time (one rounding, at the end).  Staged row r, 16-byte chunk c (four columns) at r * 256 + (c ^ r) * 16.
      const half_t* const src = FORM == kStoreAdd ? ep.add : ep.relu_src;
      const __amdgpu_buffer_rsrc_t from = make_rsrc(src + (size_t)m0 * g.ldc + n0, extent);
      uint32_t next = at;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        half8_t pre[8];
#pragma unroll
        for (int q = 0; q < 8; ++q, next += step) pre[q] = buffer_half8(from, next);
#pragma unroll
        for (int i = 4 * h; i < 4 * h + 4; ++i) {
          uint32_t wa[4], ra[4];
          floatx4 rv[4];
#pragma unroll
          for (int j = 0; j < L::TN; ++j) wa[j] = out + row * 256 + (((4 * j + quad) ^ row) << 4);
#pragma unroll
          for (int it = 0; it < 4; ++it) {
            const int rl = (it >> 1) * 8 + r8;
            ra[it] = out + rl * 256 + (((2 * c8 + (it & 1)) ^ rl) << 4);
          }
          out_write_sums(wa, t.acc[i]);
          out_read_slab(ra, rv);
#pragma unroll
          for (int it = 0; it < 2; ++it, at += step) {
            const half8_t p = pre[2 * (i - 4 * h) + it];
            floatx8 v;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float x = rv[2 * it + (e >> 2)][e & 3];
              v[e] = FORM == kStoreAdd ? x + (float)p[e] : (float)p[e] > 0.f ? x * ep.mask_scale : 0.f;
            }
            buffer_store_half8(to, at, __builtin_convertvector(v, half8_t));  // (rounded to fp32 first, as in the form with one tile per work-group)
          }
        }
      }
    }
    if (!more) break;
  }
  __builtin_amdgcn_s_waitcnt(wait_vm(0));  // (the last requests, zeros, land in this work-group's LDS)
}

// C[m, n] = fp16(sum_z partial[z][m][n]), 8 columns per thread, splits summed in increasing order
__global__ void __launch_bounds__(kThreads) splitk_reduce_kernel(const float* __restrict__ partial, int splits, int M, int N,
                                                                half_t* __restrict__ C, int ldc, float scale) {
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int chunks = N >> 3;
  if (gid >= (int64_t)M * chunks) return;
  const int row = (int)(gid / chunks), c8 = (int)(gid % chunks);
  const size_t off = (size_t)row * N + c8 * 8, plane = (size_t)M * N;
  floatx4 lo = *reinterpret_cast<const floatx4*>(partial + off), hi = *reinterpret_cast<const floatx4*>(partial + off + 4);
  for (int z = 1; z < splits; ++z) {
    lo += *reinterpret_cast<const floatx4*>(partial + z * plane + off);
    hi += *reinterpret_cast<const floatx4*>(partial + z * plane + off + 4);
  }
  half8_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    o[e] = (half_t)(lo[e] * scale);
    o[4 + e] = (half_t)(hi[e] * scale);
  }
  st_half8(C + (size_t)row * ldc + c8 * 8, o);
}

// ------------------------------------------------------------------------------------------------
// Weight gradients of one layer in one launch.  Each of them alone is too small to fill the chip (512 x 2048 results are
// 64 tiles of 128 x 128), so one by one they were cut along the positions, wrote fp32 partial sums and needed a
// second kernel each; together a layer's four to seven products are one launch of whole tiles, and the bias gradients
// ride along (no pass over memory for the column sums).  An encoder layer's over 3000 positions, alone on the chip: 34 us
// 512 wide, 78 us 1024 wide (0.97 PFLOP/s), where the products, reductions and column sums one by one took 145 and 276 us of kernel
// time beside the chain; over 52700 positions 1024 wide: 1.24 ms (1.07 PFLOP/s).
// ------------------------------------------------------------------------------------------------
struct GroupArgs {
  int n, total;
  XcdOrder runs;          // of the whole group
  float out_scale;
  struct Product {
    WgradProduct w;
    float *partial, *partial_colsum;
    int begin;            // first work item of the product
    int k_chunk;
    TileOrder order;
  } p[kMaxWgrad];
};
// Work item -> product, split and tile; consecutive items of one XCD's run share operand panels (as in place()).
__device__ __forceinline__ GemmArgs group_item(const GroupArgs& a, int lin, int& split, int& tm, int& tn, bool& sums) {
  const int at = (int)xcd_order((uint32_t)lin, a.runs);
  int i = 0;
  while (i + 1 < a.n && at >= a.p[i + 1].begin) ++i;
  const GroupArgs::Product& p = a.p[i];
  GemmArgs g{p.w.A, p.w.B, p.w.C, p.w.lda, p.w.ldb, p.w.ldc, p.w.M, p.w.N, p.w.K, GemmEpilogue{}, p.partial, p.k_chunk, p.w.colsum, p.partial_colsum};
  g.ep.out_scale = a.out_scale;
  uint32_t pid;
  split = (int)div_mod((uint32_t)(at - p.begin), p.order.tiles, pid);
  place_tile(p.order, pid, tm, tn);
  sums = tn == 0 && g.colsum;
  return g;
}
template <int BM, int BN, int NS, int NW>
__device__ __forceinline__ void wgrad_group(const GroupArgs& a) {
  using T = Tile<BM, BN, true, true, NW>;
  __shared__ __align__(1024) unsigned char stage0[T::STAGE];
  __shared__ __align__(1024) unsigned char stage1[T::STAGE];
  int split, tm, tn;
  bool sums;
  const GemmArgs g = group_item(a, (int)blockIdx.x, split, tm, tn, sums);
  if constexpr (NS == 2) {
    if (sums) gemm_tile<BM, BN, true, true, NW, true, kStoreGroup>(g, split, tm, tn, stage0, stage1);
    else gemm_tile<BM, BN, true, true, NW, false, kStoreGroup>(g, split, tm, tn, stage0, stage1);
  } else {
    __shared__ __align__(1024) unsigned char stage2[T::STAGE];
    __shared__ __align__(1024) unsigned char stage3[T::STAGE];
    if (sums) gemm_small_tile<BM, BN, true, true, NW, true, kStoreGroup>(g, split, tm, tn, stage0, stage1, stage2, stage3);
    else gemm_small_tile<BM, BN, true, true, NW, false, kStoreGroup>(g, split, tm, tn, stage0, stage1, stage2, stage3);
  }
}
template <int BM, int BN, int NS, int NW>
__global__ void __launch_bounds__(64 * NW) wgrad_group_kernel(const GroupArgs a) {
  wgrad_group<BM, BN, NS, NW>(a);
}
// The smallest tiles, with the sums of partial rows (if any) that the layer's LayerNorm gradients are: work-groups of 8 columns behind the products'.
// Passes with such groups are bound by the number of their launches, 4 us each: whole updates of 136 positions, two layers 64 wide, 526 -> 508 us
// (medians of ten processes of each form in turn; 521 to 538 and 505 to 518 but for one and two that ran faster, 481 and 469 / 489).  The larger tiles' groups keep the sums' own launch: their passes are not bound by launches.
__global__ void __launch_bounds__(256) wgrad_group_sums_kernel(const GroupArgs a, const FinalizeArgs f) {
  if ((int)blockIdx.x >= a.total) {
    __shared__ float red[32 * 9];
    finalize_columns<256>(f, (int)blockIdx.x - a.total, red);
    return;
  }
  wgrad_group<64, 64, 4, 4>(a);
}
// (as gemm_small_kernel_8)
template <int BM, int BN>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_num_vgpr(88))) wgrad_group_kernel_8(const GroupArgs a) {
  wgrad_group<BM, BN, 4, 8>(a);
}
// C and the column sums of every product of the group from the splits' fp32 sums, 8 columns per thread, splits in
// increasing order
struct GroupReduceArgs {
  int n, splits;
  float scale;
  struct Product {
    const float *partial, *partial_colsum;
    half_t *C, *colsum;
    int M, N, ldc;
    int64_t begin;  // first work item: M * N / 8 of C, then ceil(M / 8) of the column sums
  } p[kMaxWgrad];
  int64_t total;
};
__global__ void __launch_bounds__(kThreads) wgrad_group_reduce_kernel(const GroupReduceArgs a) {
  const int64_t gid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  if (gid >= a.total) return;
  int i = 0;
  while (i + 1 < a.n && gid >= a.p[i + 1].begin) ++i;
  const GroupReduceArgs::Product& p = a.p[i];
  const int64_t at = gid - p.begin, chunks = p.N >> 3, of_c = (int64_t)p.M * chunks;
  if (at >= of_c) {
    const int m0 = (int)(at - of_c) * 8;
    for (int m = m0; m < min(m0 + 8, p.M); ++m) {
      float s = 0.f;
      for (int z = 0; z < a.splits; ++z) s += p.partial_colsum[(size_t)z * p.M + m];
      p.colsum[m] = (half_t)(s * a.scale);
    }
    return;
  }
  const int row = (int)(at / chunks), c8 = (int)(at % chunks);
  const size_t off = (size_t)row * p.N + c8 * 8, plane = (size_t)p.M * p.N;
  floatx4 lo = *reinterpret_cast<const floatx4*>(p.partial + off), hi = *reinterpret_cast<const floatx4*>(p.partial + off + 4);
  for (int z = 1; z < a.splits; ++z) {
    lo += *reinterpret_cast<const floatx4*>(p.partial + z * plane + off);
    hi += *reinterpret_cast<const floatx4*>(p.partial + z * plane + off + 4);
  }
  half8_t o;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    o[e] = (half_t)(lo[e] * a.scale);
    o[4 + e] = (half_t)(hi[e] * a.scale);
  }
  st_half8(p.C + (size_t)row * p.ldc + c8 * 8, o);
}

// The form of an epilogue that the kernels have compiled in: with x W^T nothing, bias, or bias and ReLU, with dy W nothing, a sum or the mask; kStoreAny otherwise.
StoreForm store_form(const GemmEpilogue& ep, bool b_t, bool cut) {
  if (cut || ep.drop.thr || ep.out_scale != 1.f) return kStoreAny;
  if (!ep.bias && !ep.relu && !ep.add && !ep.relu_src) return kStorePlain;
  if (!b_t && ep.bias && !ep.add && !ep.relu_src) return ep.relu ? kStoreRelu : kStoreBias;
  if (b_t && !ep.bias && !ep.relu && !(ep.add && ep.relu_src)) return ep.add ? kStoreAdd : kStoreMask;
  return kStoreAny;
}
// NS = 2: two stages, strip by strip; 4: a ring of four, a whole k-tile of fragments ahead
template <int BM, int BN, bool AT, bool BT, int NS, int NW, StoreForm FORM>
void launch_variant(const GemmArgs& g, int splits, hipStream_t stream) {
  const dim3 grid(g.order.tiles.d, splits), block(64 * NW);
  if constexpr (NS == 2) hipLaunchKernelGGL((gemm_kernel<BM, BN, AT, BT, NW, FORM>), grid, block, 0, stream, g);
  else if constexpr (NW == 8) hipLaunchKernelGGL((gemm_small_kernel_8<BM, BN, AT, BT, FORM>), grid, block, 0, stream, g);
  else hipLaunchKernelGGL((gemm_small_kernel<BM, BN, AT, BT, NW, FORM>), grid, block, 0, stream, g);
}

template <int BM, int BN, int NS, int NW = 4>
int launch_tile(const GemmArgs& a, bool a_t, bool b_t, int splits, hipStream_t stream) {
  GemmArgs g = a;
  if (splits > 1) {
    g.k_chunk = (int)round_up(ceil_div(g.K, splits), 64);  // (whatever the tile, so that its shape changes no bit)
    splits = ceil_div(g.K, g.k_chunk);  // no empty split
  }
  if (splits <= 1) {
    g.partial = nullptr;
    splits = 1;
  }
  g.order = tile_order(ceil_div(g.M, BM), ceil_div(g.N, BN));
  g.runs = xcd_runs(g.order.tiles.d * splits);
  g.keep = (int64_t)g.M * g.N * 2 <= kKeptBytes;
  constexpr bool kForms = BM < 256;  // (256 x 256 tiles have theirs in the persistent form)
  const StoreForm form = kForms && !a_t ? store_form(g.ep, b_t, g.partial != nullptr) : kStoreAny;
  auto run = [&](auto at, auto bt, auto f) { launch_variant<BM, BN, decltype(at)::value, decltype(bt)::value, NS, NW, decltype(f)::value>(g, splits, stream); };
  const std::false_type no;
  const std::true_type yes;
#define NMT_FORM(f) std::integral_constant<StoreForm, f>{}
  if (a_t && b_t) run(yes, yes, NMT_FORM(kStoreAny));
  else if (a_t) run(yes, no, NMT_FORM(kStoreAny));
  else if (form == kStoreAny && b_t) run(no, yes, NMT_FORM(kStoreAny));
  else if (form == kStoreAny) run(no, no, NMT_FORM(kStoreAny));
  if constexpr (kForms) {
    if (form == kStorePlain && b_t) run(no, yes, NMT_FORM(kStorePlain));
    else if (form == kStorePlain) run(no, no, NMT_FORM(kStorePlain));
    else if (form == kStoreBias) run(no, no, NMT_FORM(kStoreBias));
    else if (form == kStoreRelu) run(no, no, NMT_FORM(kStoreRelu));
    else if (form == kStoreAdd) run(no, yes, NMT_FORM(kStoreAdd));
    else if (form == kStoreMask) run(no, yes, NMT_FORM(kStoreMask));
  }
#undef NMT_FORM
  NMT_LAUNCH_CHECK();
  if (splits == 1) return NMT_OK;
  const int64_t n = (int64_t)g.M * (g.N / 8);
  hipLaunchKernelGGL(splitk_reduce_kernel, dim3(ceil_div(n, kThreads)), dim3(kThreads), 0, stream, g.partial, splits, g.M, g.N, g.C, g.ldc, g.ep.out_scale);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

// The tile shapes below 256 x 256 and what a product takes with each, in us, fitted to timings of 160 shapes (130 to 26000 rows,
// 64 to 4096 columns, k 64 to 4096; x W^T and dy W, operands rotating through 300 MB): `fixed` (launch, first operands,
// epilogue) + k-tiles of 64 x the time of one, which depends on how many tiles share a compute unit (at most `per_cu`, by
// LDS), + `again` for every further round of work-groups.  The model was within 3 to 5 % of
// the measured times on average; the shape it picks, with the large tile among them, costs 0.6 % more than the fastest on average and 15 % at worst
// (constants fitted to the kernels before these: 1.3 % and 26 %, 6000 x 1024 x 3072 in large tiles, 55 us, for 44 in 128 x 128).
// Since then an epilogue of its own for each form and arguments fetched together have taken 1.3 to 1.7 us off every shape alike: with operands in the
// last-level cache the model is 10 to 23 % high, but over 286 products of 130 to 13000 rows its pick costs 0.8 % more than the fastest on average, 10 % at worst;
// constants fitted to those timings pick no better (0.7 %, 13 %).
enum SmallTile { kTile64, kTile128x64, kTile64x128, kTile128, kTile128x64Many, kTile128Many, kSmallTiles };
struct TileCost {
  int bm, bn, per_cu;
  double fixed, again;
  double k_tile[3];  // one k-tile while 1, 2, 3 tiles share the compute unit
};
constexpr TileCost kTileCost[kSmallTiles] = {
    {64, 64, 2, 4.3, 1.5, {0.16, 0.35, 0.}},          // four stages
    {128, 64, 1, 4.0, 2.6, {0.295, 0., 0.}},          // four stages
    {64, 128, 1, 4.0, 2.6, {0.295, 0., 0.}},          // four stages
    {128, 128, 1, 4.0, 4.2, {0.41, 0., 0.}},          // four stages, eight wavefronts
    {128, 64, 3, 4.5, 1.9, {0.49, 0.61, 0.875}},      // two stages
    {128, 128, 2, 4.9, 3.6, {0.63, 0.87, 0.}},        // two stages
};
double tile_us(const TileCost& c, int64_t tiles, int K, int cus) {
  const int nk = ceil_div(K, 64);
  const int64_t slots = (int64_t)cus * c.per_cu, rounds = tiles / slots, rest = tiles - rounds * slots;
  double us = c.fixed + rounds * nk * c.k_tile[c.per_cu - 1];
  if (rest) us += nk * c.k_tile[ceil_div(rest, cus) - 1];
  return us + c.again * (double)(rounds + (rest ? 1 : 0) - 1);
}
SmallTile choose_small_tile(int M, int N, int K, int cus, double& best_us) {
  int best = kTile64;
  best_us = 0.;
  for (int t = 0; t < kSmallTiles; ++t) {
    const double us = tile_us(kTileCost[t], (int64_t)ceil_div(M, kTileCost[t].bm) * ceil_div(N, kTileCost[t].bn), K, cus);
    if (t == 0 || us < best_us) { best = t; best_us = us; }
  }
  return (SmallTile)best;
}
// The same for at most one 256 x 256 tile per compute unit (row-major A; within 3 % of the measured times on average): a k-tile costs more the more compute units are at work, because the clocks drop.
double large_us(int64_t tiles, int K, int cus) {
  constexpr double kFixed = 5.5, kFew = 1.09, kFull = 1.65;
  const double fill = (double)tiles / cus;
  return kFixed + ceil_div(K, 64) * (kFew + (kFull - kFew) * fill * fill * fill);
}
int launch_small_tile(SmallTile t, const GemmArgs& g, bool a_t, bool b_t, int splits, hipStream_t stream) {
  switch (t) {
    case kTile64: return launch_tile<64, 64, 4>(g, a_t, b_t, splits, stream);
    case kTile128x64: return launch_tile<128, 64, 4>(g, a_t, b_t, splits, stream);
    case kTile64x128: return launch_tile<64, 128, 4>(g, a_t, b_t, splits, stream);
    case kTile128: return launch_tile<128, 128, 4, 8>(g, a_t, b_t, splits, stream);
    case kTile128x64Many: return launch_tile<128, 64, 2>(g, a_t, b_t, splits, stream);
    default: return launch_tile<128, 128, 2>(g, a_t, b_t, splits, stream);
  }
}

}  // namespace

namespace {
int launch_gemm_impl(const half_t* A, bool a_t, int lda, const half_t* B, bool b_t, int ldb, half_t* C, int ldc, int M,
                     int N, int K, const GemmEpilogue& ep, hipStream_t stream, float* partial, int64_t partial_floats, int splits) {
  NMT_REQUIRE(M > 0 && N > 0 && K > 0, "gemm: empty problem M=%d N=%d K=%d", M, N, K);
  NMT_REQUIRE(A && B && C, "gemm: null operand");
  NMT_REQUIRE(aligned16(A) && aligned16(B) && aligned16(C), "gemm: operands must be 16-byte aligned");
  NMT_REQUIRE(lda % 8 == 0 && ldb % 8 == 0 && ldc % 8 == 0 && N % 8 == 0, "gemm: lda/ldb/ldc/N must be multiples of 8");
  NMT_REQUIRE((a_t ? M : K) % 8 == 0 && (b_t ? N : K) % 8 == 0, "gemm: contiguous operand dimension must be a multiple of 8");
  NMT_REQUIRE(lda >= (a_t ? M : K) && ldb >= (b_t ? N : K) && ldc >= N, "gemm: leading dimension too small");
  NMT_REQUIRE(lda <= (1 << 20) && ldb <= (1 << 20) && ldc <= (1 << 20), "gemm: leading dimensions above 2^20 are not supported");
  NMT_REQUIRE(!ep.bias || aligned16(ep.bias), "gemm: bias must be 16-byte aligned");
  NMT_REQUIRE((!ep.add || aligned16(ep.add)) && (!ep.relu_src || aligned16(ep.relu_src)), "gemm: epilogue operand misaligned");
  NMT_REQUIRE(splits >= 0 && splits <= 64, "gemm: number of k splits %d outside [0, 64]", splits);
  const bool plain = !ep.bias && !ep.relu && !ep.drop.thr && !ep.add && !ep.relu_src;  // (out_scale is applied by the reduction)
  NMT_REQUIRE(splits <= 1 || (partial && plain), "gemm: splitting k needs a partial-sum buffer and no epilogue");
  NMT_REQUIRE(!partial || (reinterpret_cast<uintptr_t>(partial) & 15u) == 0, "gemm: partial-sum buffer must be 16-byte aligned");
  GemmArgs g{A, B, C, lda, ldb, ldc, M, N, K, ep, partial, 0};
  const int cus = device_info().cus;
  const int64_t plane = (int64_t)M * N;
  // Work-groups of 256 x 256 tiles run one per compute unit; they pay off once there are enough of them.
  const int64_t t256 = (int64_t)ceil_div(M, 256) * ceil_div(N, 256);
  const int64_t full = 3 * (int64_t)cus / 4;  // large tiles from three quarters of a round on
  if (splits == 0) {  // choose: a problem with a small result and a long contraction is cut along k
    splits = 1;
    if (partial && plain && t256 < full) {
      int64_t want = (cus + t256 / 2) / t256;                   // large tiles: one work-group per compute unit
      want = want < K / 2048 ? want : K / 2048;                 // at least 2048 k per split
      want = want < partial_floats / plane ? want : partial_floats / plane;
      want = want < 64 ? want : 64;
      if (want >= 2) {
        splits = (int)want;
      } else {
        // a contraction too short for that (the weight gradient of a single sub-batch): 128 x 128 tiles, two
        // work-groups per compute unit, at least 512 k per split
        const int64_t t128 = (int64_t)ceil_div(M, 128) * ceil_div(N, 128);
        want = 2 * cus / t128;
        want = want < K / 512 ? want : K / 512;
        want = want < partial_floats / plane ? want : partial_floats / plane;
        want = want < 64 ? want : 64;
        if (want >= 2) splits = (int)want;
      }
    }
  }
  NMT_REQUIRE(splits == 1 || plane * splits <= partial_floats, "gemm: partial-sum buffer of %lld floats too small for %d splits",
              (long long)partial_floats, splits);
  if (const int forced = tuning().gemm_tile; forced && splits <= 1) {
    switch (forced) {
      case 1: return launch_tile<256, 256, 2, 8>(g, a_t, b_t, 1, stream);
      case 2: return launch_small_tile(kTile128, g, a_t, b_t, 1, stream);
      case 3: return launch_small_tile(kTile128x64, g, a_t, b_t, 1, stream);
      case 4: return launch_small_tile(kTile64x128, g, a_t, b_t, 1, stream);
      default: return launch_small_tile(kTile64, g, a_t, b_t, 1, stream);
    }
  }
  // (a caller that keeps several passes in flight says so: each product then counts on its share of the chip)
  const int share = tuning().gemm_share;
  double small_us;
  const SmallTile small = choose_small_tile(M, N, K, cus, small_us);
  // Up to one round of large tiles they are taken where they cost less than the best small ones (9000 x 1024 x 4096, 144 large tiles:
  // 79 us against 90; 17700 x 512 x 2048, 140: 42 against 50; 6000 x 1024 x 4096, 96: 75 against 54); a fixed line at three quarters of a round gave all of these small
  // ones.  That line remains where the costs were not measured: products cut along k, with a k-major A, or beside others.
  const bool large = (splits > 1 || a_t || share > 1 || t256 > cus) ? t256 * splits * share >= full : large_us(t256, K, cus) <= small_us;
  if (large) {
    // A last, partly filled round of 256 x 256 tiles leaves compute units idle for a whole tile's
    // time.  If that round is small, the rows it would cover are given to a second launch with small
    // tiles (two work-groups per compute unit), which costs about 0.4 of a round for every round of its own.  (Up to half a round:
    // 17700 x 2048 x 512, 2.2 rounds: 52 -> 45 us; not above: 26000 x 1024 x 4096, 1.6 rounds, 192 us in one launch, was 217 in two.)
    const int tiles_n = ceil_div(N, 256), rounds = (int)(t256 / cus);
    if (splits == 1 && rounds >= 1 && t256 % cus != 0) {
      const int main_tm = cus * rounds / tiles_n, m_main = main_tm * 256, m_tail = M - m_main;
      const int64_t tail128 = (int64_t)ceil_div(m_tail, 128) * ceil_div(N, 128);
      const double cost_split = ceil_div((int64_t)main_tm * tiles_n, cus) + 0.4 * ceil_div(tail128, 2 * cus);
      if (main_tm >= 1 && cost_split + 0.25 <= rounds + 1) {
        int rc = launch_gemm_impl(A, a_t, lda, B, b_t, ldb, C, ldc, m_main, N, K, ep, stream, nullptr, 0, 1);
        if (rc != NMT_OK) return rc;
        GemmEpilogue tail = ep;
        tail.row0 = ep.row0 + m_main;
        if (tail.add) tail.add += (size_t)m_main * ldc;
        if (tail.relu_src) tail.relu_src += (size_t)m_main * ldc;
        return launch_gemm_impl(a_t ? A + m_main : A + (size_t)m_main * lda, a_t, lda, B, b_t, ldb, C + (size_t)m_main * ldc, ldc, m_tail, N,
                                K, tail, stream, nullptr, 0, 1);
      }
    }
    // No split along k, row-major A, one of the epilogues that have it: the persistent form, also where every work-group has one tile
    // only (its epilogue is the faster one).  Not for a k-major A: the one such product without a split, the
    // vocabulary weight gradient, has so long a contraction that the tile change hardly counts, and measured
    // 6 % slower in this form.  That one is also the only product with an output scale besides the groups: no epilogue here has it.
    if (splits == 1 && !a_t && ep.out_scale == 1.f && tuning().gemm_persist && !ep.drop.thr && !((ep.add || ep.relu_src) && (ep.bias || ep.relu)) &&
        !(ep.add && ep.relu_src)) {
      const int groups = (int)(t256 < cus ? t256 : cus);
      GemmArgs pg = g;
      pg.order = tile_order(ceil_div(M, 256), ceil_div(N, 256));
      pg.runs = xcd_runs(pg.order.tiles.d);
      pg.partial = nullptr;
      auto run = [&](auto bt) {
        constexpr bool BT = decltype(bt)::value;
        if (ep.add) hipLaunchKernelGGL((gemm_persistent_kernel<BT, kStoreAdd>), dim3(groups), dim3(512), 0, stream, pg);
        else if (ep.relu_src) hipLaunchKernelGGL((gemm_persistent_kernel<BT, kStoreMask>), dim3(groups), dim3(512), 0, stream, pg);
        else if (ep.relu) hipLaunchKernelGGL((gemm_persistent_kernel<BT, kStoreRelu>), dim3(groups), dim3(512), 0, stream, pg);
        else if (ep.bias) hipLaunchKernelGGL((gemm_persistent_kernel<BT, kStoreBias>), dim3(groups), dim3(512), 0, stream, pg);
        else hipLaunchKernelGGL((gemm_persistent_kernel<BT, kStorePlain>), dim3(groups), dim3(512), 0, stream, pg);
      };
      if (b_t) run(std::true_type{});
      else run(std::false_type{});
      NMT_LAUNCH_CHECK();
      return NMT_OK;
    }
    return launch_tile<256, 256, 2, 8>(g, a_t, b_t, splits, stream);
  }
  if (splits > 1) return launch_small_tile(kTile128Many, g, a_t, b_t, splits, stream);
  return launch_small_tile(small, g, a_t, b_t, 1, stream);
}

// ---- weight-gradient groups ----
enum GroupTile { kGroup256 = 1, kGroup128Many, kGroup128, kGroup64, kGroupTiles = kGroup64 };
constexpr int kGroupEdge[kGroupTiles + 1] = {0, 256, 128, 128, 64};
// What one work-group takes for a 64-deep piece of the contraction, in us, from timings of the layer groups of four widths
// (64 to 1024) over 130 to 53000 positions: with few compute units at work, and with all of them; per_cu work-groups share one.
// (The figures are older than the kernels: an encoder layer's group over 52200 positions 1024 wide, 1584 us by them, takes 1221.)
struct GroupCost {
  int per_cu;
  double fixed, k_tile_few, k_tile[2];
};
constexpr GroupCost kGroupCost[kGroupTiles + 1] = {
    {}, {1, 8.0, 1.50, {2.05, 0.}}, {2, 6.0, 0.62, {0.72, 1.13}}, {1, 6.0, 0.54, {0.68, 0.}}, {2, 4.0, 0.25, {0.31, 0.53}}};
// Time of the whole group alone on `cus` compute units, and the compute-unit time it takes (us x compute units).
double group_us(int tile, const WgradProduct* p, int n, int splits, int cus, double& cu_us) {
  const GroupCost& c = kGroupCost[tile];
  const int edge = kGroupEdge[tile];
  int64_t tiles = 0, floats = 0;
  int longest = 0;
  for (int i = 0; i < n; ++i) {
    tiles += (int64_t)ceil_div(p[i].M, edge) * ceil_div(p[i].N, edge) * splits;
    floats += (int64_t)p[i].M * p[i].N;
    longest = p[i].K > longest ? p[i].K : longest;
  }
  const int nk = ceil_div(ceil_div(longest, splits), 64);
  const int64_t slots = (int64_t)cus * c.per_cu, rounds = tiles / slots, rest = tiles - rounds * slots;
  double us = rounds * (c.fixed + nk * c.k_tile[c.per_cu - 1]);
  cu_us = us * cus;
  if (rest) {
    const int on_one = ceil_div(rest, cus);
    const double fill = rest < cus ? (double)rest / cus : 1.0;
    const double last = c.fixed + nk * (on_one > 1 ? c.k_tile[1] : c.k_tile_few + fill * (c.k_tile[0] - c.k_tile_few));
    us += last;
    cu_us += last * (rest < cus ? (double)rest : (double)cus);
  }
  if (splits > 1) {  // fp32 sums written and read back, one more launch
    const double reduce = 4.0 + (double)floats * splits * 8.0 / 8e6;
    us += reduce;
    cu_us += reduce * cus;
  }
  return us;
}
// The tile and the number of k splits of a group.  A group runs beside the next layer's chain of input gradients, so
// what counts is the compute-unit time it takes from that chain; its own latency counts too (the last group of a pass has
// only the embedding kernels beside it, and with one stream there is nothing).  Weights of 0 to 4 for it measured the
// same updates within 1 to 2 %, this one at the lower end throughout.  (What the model leaves out: a group of 256 x 256 tiles takes every
// compute unit whole, one work-group of 128 KB of LDS each, so the next layer's first kernels wait for it or crawl beside it: over
// 52000 positions 1024 wide LayerNorm backward takes 171 us on average beside the groups, 106 alone, while attention backward, later in
// the layer, finds nothing beside it any more.)
constexpr double kGroupLatencyWeight = 0.5;
// The numbers of k splits looked at, and the fewest positions a split may have.
constexpr int kGroupMaxSplits = 32, kGroupMinRows = 256;
int next_splits(int z) { return z < 4 ? z + 1 : z * 2; }
void choose_group(const WgradProduct* p, int n, int64_t most, int cus, int& tile, int& splits) {
  int shortest = p[0].K, best_tile = tile ? tile : kGroup256, best_splits = splits ? splits : 1;
  for (int i = 1; i < n; ++i) shortest = p[i].K < shortest ? p[i].K : shortest;
  double best = 0.;
  for (int t = tile ? tile : 1; t <= (tile ? tile : kGroupTiles); ++t) {
    for (int z = splits ? splits : 1; z <= (splits ? splits : kGroupMaxSplits); z = next_splits(z)) {
      if (!splits && z > 1 && (z > most || shortest / z < kGroupMinRows)) break;
      double cu_us;
      const double us = group_us(t, p, n, z, cus, cu_us), score = kGroupLatencyWeight * us + cu_us / cus;
      if (best == 0. || score < best) {
        best = score;
        best_tile = t;
        best_splits = z;
      }
    }
  }
  tile = best_tile;
  splits = best_splits;
}
int check_wgrad(const WgradProduct& w) {
  NMT_REQUIRE(w.M > 0 && w.N > 0 && w.K > 0, "weight gradient: empty problem M=%d N=%d K=%d", w.M, w.N, w.K);
  NMT_REQUIRE(w.A && w.B && w.C && aligned16(w.A) && aligned16(w.B) && aligned16(w.C), "weight gradient: null or misaligned operand");
  NMT_REQUIRE(w.lda % 8 == 0 && w.ldb % 8 == 0 && w.ldc % 8 == 0 && w.N % 8 == 0 && w.M % 8 == 0, "weight gradient: lda/ldb/ldc/M/N must be multiples of 8");
  NMT_REQUIRE(w.lda >= w.M && w.ldb >= w.N && w.ldc >= w.N, "weight gradient: leading dimension too small");
  NMT_REQUIRE(w.lda <= (1 << 20) && w.ldb <= (1 << 20) && w.ldc <= (1 << 20), "weight gradient: leading dimensions above 2^20 are not supported");
  return NMT_OK;
}
int launch_wgrad_group_impl(const WgradProduct* products, int n, float out_scale, float* partial, int64_t partial_floats, hipStream_t stream,
                            int tile, int splits, const FinalizeArgs& sums, int n_sums, bool& sums_done) {
  NMT_REQUIRE(products && n >= 1 && n <= kMaxWgrad, "weight gradients: %d products outside [1, %d]", n, kMaxWgrad);
  NMT_REQUIRE(tile >= 0 && tile <= kGroupTiles && splits >= 0 && splits <= 64, "weight gradients: tile %d or number of k splits %d out of range", tile, splits);
  NMT_REQUIRE(!partial || aligned16(partial), "weight gradients: partial-sum buffer must be 16-byte aligned");
  int64_t per_split = 0;  // floats one split leaves behind
  for (int i = 0; i < n; ++i) {
    if (int rc = check_wgrad(products[i])) return rc;
    per_split += (int64_t)products[i].M * products[i].N + products[i].M;
  }
  const int64_t most = partial ? partial_floats / per_split : 1;
  // (callers that keep several passes in flight: the tile is chosen for the group's share of the chip, the splits are not,
  //  so that sums do not depend on how many passes are in flight)
  int whole_chip_tile = tile;
  choose_group(products, n, most, device_info().cus, whole_chip_tile, splits);
  choose_group(products, n, most, device_info().cus / tuning().gemm_share > 1 ? device_info().cus / tuning().gemm_share : 1, tile, splits);
  NMT_REQUIRE(splits == 1 || splits <= most, "weight gradients: partial-sum buffer of %lld floats too small for %d splits", (long long)partial_floats, splits);
  const int edge = kGroupEdge[tile];
  GroupArgs a = {};
  GroupReduceArgs ra = {};
  a.n = ra.n = n;
  ra.splits = splits;
  a.out_scale = ra.scale = out_scale;
  float* at = partial;
  for (int i = 0; i < n; ++i) {
    const WgradProduct& w = products[i];
    GroupArgs::Product& p = a.p[i];
    p.w = w;
    p.begin = a.total;
    const int tiles_m = ceil_div(w.M, edge), tiles_n = ceil_div(w.N, edge);
    p.order = tile_order(tiles_m, tiles_n);
    p.k_chunk = (int)round_up(ceil_div(w.K, splits), 64);  // (a split past the end of a short contraction writes zeros)
    a.total += tiles_m * tiles_n * splits;
    if (splits > 1) {
      p.partial = at;
      p.partial_colsum = at + (int64_t)splits * w.M * w.N;
      at += (int64_t)splits * ((int64_t)w.M * w.N + w.M);
      ra.p[i] = {p.partial, p.partial_colsum, w.C, w.colsum, w.M, w.N, w.ldc, ra.total};
      ra.total += (int64_t)w.M * (w.N / 8) + (w.colsum ? w.M / 8 : 0);
    }
  }
  a.runs = xcd_runs(a.total);
  const dim3 grid(a.total);
  switch (tile) {
    case kGroup256: hipLaunchKernelGGL((wgrad_group_kernel<256, 256, 2, 8>), grid, dim3(512), 0, stream, a); break;
    case kGroup128Many: hipLaunchKernelGGL((wgrad_group_kernel<128, 128, 2, 4>), grid, dim3(256), 0, stream, a); break;
    case kGroup128: hipLaunchKernelGGL((wgrad_group_kernel_8<128, 128>), grid, dim3(512), 0, stream, a); break;
    default:
      hipLaunchKernelGGL(wgrad_group_sums_kernel, dim3(a.total + n_sums * sums.nq * ceil_div(sums.cols, 256 / 32)), dim3(256), 0, stream, a, sums);
      sums_done = true;
  }
  NMT_LAUNCH_CHECK();
  if (splits == 1) return NMT_OK;
  hipLaunchKernelGGL(wgrad_group_reduce_kernel, dim3(ceil_div(ra.total, kThreads)), dim3(kThreads), 0, stream, ra);
  NMT_LAUNCH_CHECK();
  return NMT_OK;
}

// Optional timing of every product with HIP events on the stream it is launched on (the benchmark's roofline leg):
// pairs of events from a pool that grows as needed and is read and reset by gemm_timing_read.
struct TimedProduct {
  hipEvent_t start, stop;
  double flops;
};
std::vector<TimedProduct> g_timed;
size_t g_timed_used = 0;
std::mutex g_timed_mutex;
}  // namespace

template <typename Launch>
static int timed_launch(double flops, hipStream_t stream, Launch launch) {
  if (!tuning().gemm_timing) return launch();
  TimedProduct t;
  {
    std::lock_guard<std::mutex> lock(g_timed_mutex);
    if (g_timed_used == g_timed.size()) {
      TimedProduct fresh = {};
      NMT_HIP_CHECK(hipEventCreate(&fresh.start));
      NMT_HIP_CHECK(hipEventCreate(&fresh.stop));
      g_timed.push_back(fresh);
    }
    g_timed[g_timed_used].flops = flops;
    t = g_timed[g_timed_used++];
  }
  NMT_HIP_CHECK(hipEventRecord(t.start, stream));
  const int rc = launch();
  NMT_HIP_CHECK(hipEventRecord(t.stop, stream));
  return rc;
}

int launch_gemm(const half_t* A, bool a_t, int lda, const half_t* B, bool b_t, int ldb, half_t* C, int ldc, int M,
                int N, int K, const GemmEpilogue& ep, hipStream_t stream, float* partial, int64_t partial_floats, int splits) {
  return timed_launch(2.0 * M * N * K, stream, [&] {
    return launch_gemm_impl(A, a_t, lda, B, b_t, ldb, C, ldc, M, N, K, ep, stream, partial, partial_floats, splits);
  });
}

int64_t wgrad_group_floats(int64_t per_split, int64_t rows, int64_t most) {
  int64_t used = 0;
  for (int z = 2; z <= kGroupMaxSplits && rows / z >= kGroupMinRows && z * per_split <= most; z = next_splits(z)) used = z * per_split;
  return used;
}

int launch_wgrad_group(const WgradProduct* products, int n, float out_scale, float* partial, int64_t partial_floats, hipStream_t stream,
                       int tile, int splits, const ColumnSums* sums, int n_sums, int d) {
  NMT_REQUIRE(n_sums >= 0 && n_sums <= kMaxColumnSums && (!n_sums || (sums && d > 0)), "weight gradients: %d column sums outside [0, %d]", n_sums, kMaxColumnSums);
  double flops = 0.0;
  for (int i = 0; products && i < n && i < kMaxWgrad; ++i) flops += 2.0 * products[i].M * products[i].N * products[i].K;
  FinalizeArgs f = {3, d, d, out_scale, {}};
  for (int i = 0; i < n_sums; ++i) f.in[i] = sums[i];
  bool done = false;
  const int rc = timed_launch(flops, stream, [&] {
    return launch_wgrad_group_impl(products, n, out_scale, partial, partial_floats, stream, tile, splits, f, n_sums, done);
  });
  if (rc != NMT_OK || !n_sums || done) return rc;
  return launch_layernorm_param_grads(sums, n_sums, d, out_scale, stream);
}

int gemm_timing_read(double* ms, int64_t* products, double* flops) {
  std::lock_guard<std::mutex> lock(g_timed_mutex);
  double total = 0.0, fl = 0.0;
  for (size_t i = 0; i < g_timed_used; ++i) {
    float one = 0.f;
    NMT_HIP_CHECK(hipEventSynchronize(g_timed[i].stop));
    NMT_HIP_CHECK(hipEventElapsedTime(&one, g_timed[i].start, g_timed[i].stop));
    total += one;
    fl += g_timed[i].flops;
  }
  if (ms) *ms = total;
  if (products) *products = (int64_t)g_timed_used;
  if (flops) *flops = fl;
  g_timed_used = 0;
  return NMT_OK;
}
