// k_sdpa_mfma.hip -- bf16 causal SDPA on the gathered sub-sequence with gfx950 MFMA
// (Sec. 3.5, Eq. attn-sub with Eq. sdpa): forward, and the deterministic backward
// (dK/dV and dQ workgroups in one launch), per (b, hq) over [S, D] rows.
//
// Numerics: v_mfma_f32_32x32x16_bf16 with fp32 accumulation; the softmax runs in the exp2
// domain with the scale folded into one FMA; P and dS are rounded to bf16 for their products.
// The forward rescales its accumulator only when the running row maximum grows by more than
// 2^8 (the final O / l uses the same maximum throughout, so the result is unchanged).
//
// Layout facts used throughout (lane l of a wave, h = l / 32):
//   MFMA 32x32x16: A[m = l % 32][k = 8h + 0..7], B[k = 8h + 0..7][n = l % 32],
//                  C[m = 8(i/4) + 4h + i%4][n = l % 32], i = 0..15.
//   Forward and dQ compute S^T = K Q^T, so each lane owns one query row; dK/dV computes
//   S = Q K^T, so each lane owns one key. The k-order inside every 16-row MFMA step follows
//   the C layout (slots 0-3 = rows 4h + 0..3, slots 4-7 = rows 8 + 4h + 0..3), so an
//   accumulator converted to bf16 is directly the next product's operand; the matching
//   transposed operand is read from the row-major LDS tile with ds_read_b64_tr_b16.
//
// LDS tiles: rows of D bf16 (2D bytes, no padding) with an XOR swizzle of 16-byte chunks
// (chunk c of row r sits at position c ^ swz(r)), filled straight from global memory with
// global_load_lds_dwordx4 (no staging registers), double-buffered so the next tile streams in
// while the current one is used. All three kernels use a swizzle under which both read
// patterns are bank-conflict free (measured with SQ_LDS_BANK_CONFLICT): 16 consecutive rows
// reading one logical chunk (b128 operand reads) land on 16 different chunk positions, and the
// 4 consecutive rows of a transposed read, each reading an aligned group of 4 chunks, land in 4
// different groups. Every lane's LDS offsets are computed once; tile bases are compile-time
// constants (the tile loop is unrolled over the ring of slots).
//
// Occupancy: with F = 1 (below) the forward runs 12 waves per workgroup, 3 per SIMD (at most 168
// registers), so that two waves can be in their softmax while a third feeds the MFMA unit. The
// backward holds 128 (dK/dV) or 160 (dQ) accumulator and operand registers per lane and runs 2
// waves per SIMD.
//
// Pipeline: each kernel keeps a two-slot ring of tiles in LDS. Before using tile t, a wave waits
// until its own LDS-DMA loads have landed, then the block barrier publishes tile t from every
// wave; right after the barrier the loads of tile t + 1 go into the slot tile t - 1 used. Loads
// past the end read clamped rows into the free slot.
#include <math.h>

#include <type_traits>

#include "lh_common.h"

namespace lh {

typedef s16x4 __attribute__((address_space(3))) lds_s16x4;

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;
constexpr float kRescale = 8.0f;  // lazy rescaling threshold (log2 units)

template <int N>
using IC = std::integral_constant<int, N>;

// Swizzle of the 16-byte chunks of a row. D = 128 (16 chunks per row): swap the two 2-bit halves
// of r % 16. D = 64 (8 chunks per row, two rows per 256-byte bank line): a bijection of (r / 2) % 8
// whose top bit follows bit 1 of r. The 16 lanes that read one logical chunk of 16 consecutive
// rows hit 16 different chunk positions: row and transposed reads are conflict free.
template <int D>
__device__ __forceinline__ int swz(int r) {
  if constexpr (D == 128) return ((r & 3) << 2) | ((r >> 2) & 3);
  else return (((r >> 1) & 1) << 2) | ((r >> 2) & 3);
}

// Byte offsets of one lane inside any swizzled tile (row blocks start at multiples of 16).
template <int D>
struct LaneOff {
  int row[D / 16];  // row operand (A or B) of k-step kk: row l % 32, columns 16 kk + 8h .. +7
  int trl[D / 32];  // transposed operand, column block d, rows 4h + (l % 16) / 4 (slots 0-3)
  int trh[D / 32];  // the same 8 rows further (slots 4-7)
};

// rows0: first tile row of this wave's share (a multiple of 32)
template <int D>
__device__ __forceinline__ LaneOff<D> lane_offsets(int lane, int rows0) {
  constexpr int RB = 2 * D;
  LaneOff<D> o;
  const int h = lane >> 5, r = lane & 31, base = rows0 * RB;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) o.row[kk] = base + r * RB + (((2 * kk + h) ^ swz<D>(r)) << 4);
  const int r0 = 4 * h + ((lane & 15) >> 2);
#pragma unroll
  for (int d = 0; d < D / 32; ++d) {
    const int chunk = 4 * d + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1);
    o.trl[d] = base + r0 * RB + ((chunk ^ swz<D>(r0)) << 4) + 8 * (lane & 1);
    o.trh[d] = base + (r0 + 8) * RB + ((chunk ^ swz<D>(r0 + 8)) << 4) + 8 * (lane & 1);
  }
  return o;
}

// Row operand at byte offset `off` (lane offset plus a constant) of an LDS tile.
__device__ __forceinline__ bf16x8 row8(const bf16_t* tile, int off) {
  return *reinterpret_cast<const bf16x8*>(reinterpret_cast<const char*>(tile) + off);
}

// Transposed operand: within each 16-lane group, lane i receives Mat[r0 + j][c0 + i] (j = 0..3)
// from the lanes' addresses (lane s points at Mat[r0 + s / 4][c0 + 4 (s % 4)]); two reads give
// slots 0-3 (rows +0..3) and 4-7 (rows +8..11).
__device__ __forceinline__ bf16x8 tr8(const bf16_t* tile, int off_lo, int off_hi) {
  typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
  const char* p = reinterpret_cast<const char*>(tile);
  const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + off_lo));
  const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(p + off_hi));
  s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ bf16x8 cvt8(const float* f) {
  typedef __attribute__((__vector_size__(8 * sizeof(float)))) float f32x8;
  f32x8 v = {f[0], f[1], f[2], f[3], f[4], f[5], f[6], f[7]};
  return __builtin_convertvector(v, bf16x8);
}

__device__ __forceinline__ bf16x8 gld8(const bf16_t* p) { return *reinterpret_cast<const bf16x8*>(p); }

// Direct global -> LDS copy of TR rows starting at row r0 of a [S, D] bf16 matrix into a
// swizzled tile by the NW waves of the block. A wave instruction writes 1 KB of LDS
// contiguously (lane i -> byte 16 i), so every lane fetches the logical chunk that belongs at
// its physical position. Rows past S are clamped to row S - 1 (callers mask them out). Every
// wave issues loads_per_wave<D, TR, NW>() instructions; when the 1 KB blocks do not divide
// evenly, the extra instructions repeat a block another wave also writes (same bytes).
template <int D, int TR, int NW>
__device__ __forceinline__ constexpr int loads_per_wave() { return (TR * D / 512 + NW - 1) / NW; }

template <int D, int TR, int NW, bool CLAMP>
__device__ __forceinline__ void load_tile_rows(bf16_t* tile, const bf16_t* src, int r0, int S, int w, int lane) {
  constexpr int CPR = D / 8;
  constexpr int BLOCKS = TR * CPR / 64;  // 1 KB blocks of the tile
  static_assert(BLOCKS * 64 == TR * CPR, "a tile is a whole number of 1 KB blocks");
  const char* base = reinterpret_cast<const char*>(src + (int64_t)r0 * D);
#pragma unroll
  for (int j = 0; j < loads_per_wave<D, TR, NW>(); ++j) {
    int blk = j * NW + w;
    if (BLOCKS % NW != 0 && blk >= BLOCKS) blk -= BLOCKS;
    const int pos = blk * 64 + lane;
    const int r = pos / CPR;
    const int c = (pos % CPR) ^ swz<D>(r);
    // rows past S read row S - 1; the clamp stays a 32-bit lane offset from the tile's uniform
    // base, so no lane holds a 64-bit address (fewer live registers in every kernel)
    const int rr = CLAMP ? (r < S - 1 - r0 ? r : S - 1 - r0) : r;
    const char* g = base + (int32_t)((rr * D + c * 8) * 2);
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)(tile + blk * 512), 16, 0, 0);
  }
}

// r0 and w are uniform: a tile that lies inside the matrix is one scalar base address plus a
// fixed 32-bit offset per lane; only a tile that crosses row S clamps row by row.
template <int D, int TR, int NW>
__device__ __forceinline__ void load_tile(bf16_t* tile, const bf16_t* src, int r0, int S, int w, int lane) {
  if (r0 + TR <= S) load_tile_rows<D, TR, NW, false>(tile, src, r0, S, w, lane);
  else load_tile_rows<D, TR, NW, true>(tile, src, r0, S, w, lane);
}

// Index-driven rows (the gather fused into the loads). Row m of a gathered head is pyramid id
// idx[m]: ids below N are rows of the input [B, N, H, D], the rest rows of the pyramid
// [B, R, H, D]. Ids outside [0, N + R) are clamped into it (never an out-of-range read).
struct SdpaIdx {
  const bf16_t *q, *k, *v, *qp, *kp, *vp;
  const int32_t* idx;  // [B, Hq, S]
  int64_t N, R;
  int32_t Hq, Hkv, G;
};

// Query heads and selection heads: query head hq reads the gathered K~, V~ (and idx) of
// selection head hq / Gq; there are Hs selection heads per batch (Hs = Hq, Gq = 1 when every
// query head selects on its own).
struct HeadMap {
  int32_t Hq, Hs, Gq;
};

// Block order. Blocks are dispatched in linear-id order and go round-robin to the 8 XCDs. Linear
// id = rank * heads + head, where rank 0 is the longest block of a head (most causal tiles): the
// longest blocks of every head start first, so no long block is left to run alone at the end, and
// (heads being a multiple of 8) every block of a head lands on the same XCD, whose L2 then holds
// that head's streamed tiles.
struct BlockPos {
  int rank;      // 0 = the head's longest block
  int64_t head;
};
__device__ __forceinline__ BlockPos block_pos(uint32_t lin, uint32_t heads) {
  const uint32_t r = lin / heads;
  return BlockPos{(int)r, (int64_t)(lin - r * heads)};
}

struct RowSrc {
  const char* l0;  // row 0 of the head in the input
  const char* py;  // row 0 of the head in the pyramid, less N rows: pyramid id i is at py + i rb
  uint32_t rb;     // bytes between consecutive rows: H * D * 2
  int32_t N, last;  // last = N + R - 1
};

__device__ __forceinline__ RowSrc row_src(const bf16_t* x, const bf16_t* pyr, int64_t b, int h, int H,
                                          const SdpaIdx& ix, int D) {
  RowSrc r;
  r.rb = (uint32_t)(H * D * 2);
  r.l0 = reinterpret_cast<const char*>(x + (b * ix.N * H + h) * D);
  r.py = reinterpret_cast<const char*>(pyr + (b * ix.R * H + h) * D) - (int64_t)ix.N * r.rb;
  r.N = (int32_t)ix.N;
  r.last = (int32_t)(ix.N + ix.R - 1);
  return r;
}

// One clamp (a median of three), one compare with two selects for the base, one 32 x 32 -> 64-bit
// multiply-add.
__device__ __forceinline__ const bf16_t* rs_row(const RowSrc& s, int32_t id) {
  id = id < 0 ? 0 : id > s.last ? s.last : id;
  const char* base = id < s.N ? s.l0 : s.py;
  return reinterpret_cast<const bf16_t*>(base + (uint64_t)(uint32_t)id * s.rb);
}

// Pyramid ids of the rows this lane copies in load_tile (rows past S take row S - 1's id).
template <int D, int TR, int NW>
__device__ __forceinline__ void tile_ids(const int32_t* idxh, int r0, int S, int w, int lane, int32_t* ids) {
  constexpr int CPR = D / 8;
  constexpr int BLOCKS = TR * CPR / 64;
#pragma unroll
  for (int j = 0; j < loads_per_wave<D, TR, NW>(); ++j) {
    int blk = j * NW + w;
    if (BLOCKS % NW != 0 && blk >= BLOCKS) blk -= BLOCKS;
    const int gr = r0 + (blk * 64 + lane) / CPR;
    ids[j] = idxh[gr < S ? gr : S - 1];
  }
}

// load_tile with every row read from its pyramid id.
template <int D, int TR, int NW>
__device__ __forceinline__ void load_tile_idx(bf16_t* tile, const RowSrc& src, const int32_t* ids, int w, int lane) {
  constexpr int CPR = D / 8;
  constexpr int BLOCKS = TR * CPR / 64;
#pragma unroll
  for (int j = 0; j < loads_per_wave<D, TR, NW>(); ++j) {
    int blk = j * NW + w;
    if (BLOCKS % NW != 0 && blk >= BLOCKS) blk -= BLOCKS;
    const int pos = blk * 64 + lane;
    const int c = (pos % CPR) ^ swz<D>(pos / CPR);
    const bf16_t* g = rs_row(src, ids[j]) + c * 8;
    __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)g,
                                     (__attribute__((address_space(3))) void*)(tile + blk * 512), 16, 0, 0);
  }
}

// Waits until at most N of this wave's vector-memory loads are outstanding and every LDS
// access of the wave has completed (s_waitcnt vmcnt(N) lgkmcnt(0)), then joins the block
// barrier. The empty asm statements keep the compiler from moving memory accesses across.
template <int N>
__device__ __forceinline__ void sync_tiles() {
  static_assert(N >= 0 && N < 64, "vmcnt holds 6 bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// Calls f(IC<t % 2>{}, t) for t = begin .. end - 1: a loop over a two-slot ring that may start
// on either slot.
template <typename F>
__device__ __forceinline__ void ring2_loop(int begin, int end, F& f) {
  int t = begin;
  if (t < end && (t & 1)) {
    f(IC<1>{}, t);
    ++t;
  }
  for (; t + 1 < end; t += 2) {
    f(IC<0>{}, t);
    f(IC<1>{}, t + 1);
  }
  if (t < end) f(IC<0>{}, t);
}

// Stores a lane's O^T-layout accumulator row (query row q, columns 32 d + 8 g + 4h + 0..3).
template <int D>
__device__ __forceinline__ void store_qrow(bf16_t* row, const f32x16* acc, float mul, int h) {
#pragma unroll
  for (int d = 0; d < D / 32; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int col = 32 * d + 8 * g + 4 * h;
      const uint32_t w0 = (uint32_t)f2bf(acc[d][4 * g + 0] * mul) | ((uint32_t)f2bf(acc[d][4 * g + 1] * mul) << 16);
      const uint32_t w1 = (uint32_t)f2bf(acc[d][4 * g + 2] * mul) | ((uint32_t)f2bf(acc[d][4 * g + 3] * mul) << 16);
      *reinterpret_cast<uint2*>(row + col) = make_uint2(w0, w1);
    }
}

// Ring slots are separate __shared__ arrays (not one indexed array), so the compiler can tell
// that a load streaming into one slot does not alias reads of another and does not wait for it.
struct Ring {  // two slots of two operands
  bf16_t *a0, *a1, *b0, *b1;
  template <int SL>
  __device__ __forceinline__ bf16_t* a() const { return SL ? a1 : a0; }
  template <int SL>
  __device__ __forceinline__ bf16_t* b() const { return SL ? b1 : b0; }
};

// Split of a workgroup's rows and tiles. The R = NW / F row blocks (32 rows each) of a workgroup
// are each shared by F waves: wave w works on row block w % R and, of every streamed tile of
// F 32 NB rows, on the NB 32-row blocks from f NB, f = w / R. With F > 1 the F partial
// accumulators of a row block are summed through LDS at the end, in the order of f.
//
// F = 1 has the fewest loads per product (a tile serves every wave) and is what a full chip
// wants. A problem with few row blocks leaves CUs idle, and its time is that of its longest
// block, a chain of tiles; F = 2 and 4 make the blocks 2 to 6 times as many and their chains 2
// to 4 times as short, for as many more tile loads. The rules beside the launches choose.
template <int F>
struct FwdCfg {
  static constexpr int NW = F == 1 ? 12 : 8;  // waves
  static constexpr int EU = F == 1 ? 3 : 2;   // waves per SIMD the register budget targets
  static constexpr int NB = F == 1 ? 2 : 1;   // 32-key blocks of a tile per wave
  static constexpr int R = NW / F, ROWS = 32 * R, TILE = 32 * NB * F;
};
template <int F>
struct BwdCfg {
  static constexpr int NW = 8, EU = 2;
  static constexpr int NB = F == 1 ? 2 : 1;
  static constexpr int R = NW / F, ROWS = 32 * R, TILE = 32 * NB * F;
};

// Where the backward forms a wave's row block and share at run time. With F = 1 they are w and 0;
// formed all the same, they steer the compiler to 0.4% less time (71.4 to 71.2 ms at S = 54,272,
// 32 heads), but in the index-driven kernels, at D = 128, to 60 spilled registers instead of 7.
template <bool IDX, int F>
constexpr bool kSplitAt = F > 1 || !IDX;

// Sums the accumulators of the F waves of each row block and hands the sums out: the tile ring
// (no longer in use) holds the partial accumulators of D / 32 * F / 4 column blocks of every wave
// at a time. A unit is 4 accumulator elements: out(d, g, x) receives elements 4 g .. 4 g + 3 of
// column block d, each unit in one of the F waves. wt[x]: weight of wave x's partial.
template <int D, int F, int R, typename Out>
__device__ __forceinline__ void combine(const Ring& ring, const f32x16* acc, const float* wt, int w, int lane,
                                        Out&& out) {
  constexpr int ND = D / 32 * F / 4;  // column blocks per round: a wave's share is half a slot
  constexpr int NU = 4 * ND / F;      // units per wave and round
  static_assert(ND >= 1 && NU >= 1 && F * R == 8, "two waves per slot array");
  constexpr int HALF = 32 * F * D / 2;  // elements of half a slot of 32 F rows
  const int r = w % R, f = w / R;
  auto part = [&](int x) __attribute__((always_inline)) {
    // (values, not lvalues: a choice among the members' addresses would put the struct in memory)
    bf16_t* const a = (x & 1) ? +ring.a1 : +ring.a0;
    bf16_t* const b = (x & 1) ? +ring.b1 : +ring.b0;
    bf16_t* const p = (x & 2) ? +b : +a;
    return reinterpret_cast<float*>(p + (x >> 2) * HALF);
  };
#pragma unroll
  for (int d0 = 0; d0 < D / 32; d0 += ND) {
    __syncthreads();  // the ring, or the last round's partials, are no longer read
    float* mine = part(w);
#pragma unroll
    for (int d = 0; d < ND; ++d)
#pragma unroll
      for (int g = 0; g < 4; ++g)
        *reinterpret_cast<float4*>(mine + ((4 * d + g) * 64 + lane) * 4) =
            make_float4(acc[d0 + d][4 * g], acc[d0 + d][4 * g + 1], acc[d0 + d][4 * g + 2], acc[d0 + d][4 * g + 3]);
    __syncthreads();
#pragma unroll
    for (int y = 0; y < NU; ++y) {
      const int u = f * NU + y;
      float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int x = 0; x < F; ++x) {
        const float4 t = *reinterpret_cast<const float4*>(part(x * R + r) + (u * 64 + lane) * 4);
        v[0] += wt[x] * t.x, v[1] += wt[x] * t.y, v[2] += wt[x] * t.z, v[3] += wt[x] * t.w;
      }
      out(d0 + u / 4, u % 4, v);
    }
  }
}

__device__ __forceinline__ void store_quad(bf16_t* p, const float* v, float mul) {
  const uint32_t w0 = (uint32_t)f2bf(v[0] * mul) | ((uint32_t)f2bf(v[1] * mul) << 16);
  const uint32_t w1 = (uint32_t)f2bf(v[2] * mul) | ((uint32_t)f2bf(v[3] * mul) << 16);
  *reinterpret_cast<uint2*>(p) = make_uint2(w0, w1);
}

// ------------------------------------------------------------------ forward
// IDX: Q, K, V are unused; rows come from the input / pyramid through ix.idx.
template <int D, bool IDX, int F>
__global__ void __launch_bounds__(64 * FwdCfg<F>::NW)
    __attribute__((amdgpu_waves_per_eu(FwdCfg<F>::EU, FwdCfg<F>::EU)))
sdpa_fwd_bf16(const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K, const bf16_t* __restrict__ V,
              bf16_t* __restrict__ O, float* __restrict__ LSE, int S, uint32_t heads, float sl2,
              SdpaIdx ix, HeadMap hm) {
  using C = FwdCfg<F>;
  constexpr int RB = 2 * D, FW = C::NW, FK = C::TILE, FQ = C::ROWS;
  constexpr int NB = C::NB;  // 32-key blocks of a tile per wave
  __shared__ __align__(16) bf16_t Ks0[FK * D], Ks1[FK * D], Vs0[FK * D], Vs1[FK * D];
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, r32 = lane & 31;
  const BlockPos bp = block_pos(blockIdx.x, heads);
  const int64_t bh = bp.head;
  const int nqt = (S + FQ - 1) / FQ;
  const int q0 = (nqt - 1 - bp.rank) * FQ;  // longest rows first
  const int f = F > 1 ? w / C::R : 0;        // this wave's share of a tile: keys 32 NB f ..
  const int qw = q0 + 32 * (F > 1 ? w % C::R : w);
  const int myq = qw + r32;
  const int64_t kvh = (bh / hm.Hq) * hm.Hs + (bh % hm.Hq) / hm.Gq;  // selection head
  const bf16_t* Qh = Q + bh * S * D;
  const bf16_t* Kh = K + kvh * S * D;
  const bf16_t* Vh = V + kvh * S * D;
  const LaneOff<D> lo = lane_offsets<D>(lane, 32 * NB * f);
  constexpr int LPW = loads_per_wave<D, FK, FW>();
  RowSrc qsrc{}, ksrc{}, vsrc{};
  const int32_t* idxh = nullptr;
  int32_t kv_ids[LPW];  // ids of the next tile to be loaded
  if constexpr (IDX) {
    const int64_t b = bh / ix.Hq;
    const int hq = (int)(bh - b * ix.Hq), g = hq / ix.G;
    qsrc = row_src(ix.q, ix.qp, b, hq, ix.Hq, ix, D);
    ksrc = row_src(ix.k, ix.kp, b, g, ix.Hkv, ix, D);
    vsrc = row_src(ix.v, ix.vp, b, g, ix.Hkv, ix, D);
    idxh = ix.idx + kvh * S;
  }
  auto load_kv = [&](int slot_, int r0) __attribute__((always_inline)) {
    bf16_t* kt_ = slot_ ? Ks1 : Ks0;
    bf16_t* vt_ = slot_ ? Vs1 : Vs0;
    if constexpr (IDX) {
      load_tile_idx<D, FK, FW>(kt_, ksrc, kv_ids, w, lane);
      load_tile_idx<D, FK, FW>(vt_, vsrc, kv_ids, w, lane);
      tile_ids<D, FK, FW>(idxh, r0 + FK, S, w, lane, kv_ids);  // the tile after this one
    } else {
      load_tile<D, FK, FW>(kt_, Kh, r0, S, w, lane);
      load_tile<D, FK, FW>(vt_, Vh, r0, S, w, lane);
    }
  };
  if constexpr (IDX) tile_ids<D, FK, FW>(idxh, 0, S, w, lane, kv_ids);

  const int kend = q0 + FQ < S ? q0 + FQ : S;
  const int nkt = (kend + FK - 1) / FK;
  bf16x8 qreg[D / 16];
  const int qrow = myq < S ? myq : S - 1;
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    const bf16_t* qr = IDX ? rs_row(qsrc, idxh[qrow]) : Qh + (int64_t)qrow * D;
    qreg[kk] = gld8(qr + 16 * kk + 8 * h);
  }
  if constexpr (F == 1) load_kv(0, 0);
  f32x16 oacc[D / 32];
#pragma unroll
  for (int d = 0; d < D / 32; ++d) oacc[d] = f32x16{};
  float m_run = -INFINITY, l_run = 0.0f;

  // S^T = K Q^T of this wave's keys of a tile, masked on the diagonal
  auto logits = [&](const bf16_t* Kt, int k0, f32x16* sacc) __attribute__((always_inline)) {
#pragma unroll
    for (int kb = 0; kb < NB; ++kb) sacc[kb] = f32x16{};
#pragma unroll
    for (int kk = 0; kk < D / 16; ++kk)
#pragma unroll
      for (int kb = 0; kb < NB; ++kb) sacc[kb] = mfma32(row8(Kt, kb * 32 * RB + lo.row[kk]), qreg[kk], sacc[kb]);
    if (k0 + 32 * NB - 1 > qw) {  // diagonal tile: mask keys after the row
#pragma unroll
      for (int kb = 0; kb < NB; ++kb)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (k0 + kb * 32 + 8 * (i >> 2) + 4 * h + (i & 3) > myq) sacc[kb][i] = -INFINITY;
    }
  };
  auto row_max = [&](const f32x16* sacc) __attribute__((always_inline)) {  // in log2 units
    float mloc = sacc[0][0];
#pragma unroll
    for (int kb = 0; kb < NB; ++kb)
#pragma unroll
      for (int i = 0; i < 16; ++i) mloc = fmaxf(mloc, sacc[kb][i]);
    return fmaxf(mloc, __shfl_xor(mloc, 32, 64)) * sl2;
  };
  if constexpr (F > 1) {
    // The running maximum of a row follows the maxima of its 64-key tiles, whichever waves hold
    // them, so P is rounded to bf16 at the scale that F = 1 gives it (with a maximum of its own per
    // wave, outputs moved by 1e-3 of their 2-norm where maxima grow by more than 2^8). A wave
    // leaves its keys' row maxima of tile t in LDS before the barrier that opens step t + 1 and
    // weighs the tile after it, so the exchange takes no barrier of its own: step t forms the
    // logits of tile t and weighs tile t - 1, and V streams one tile behind K. Against a maximum of
    // its own per wave and no such overlap: D = 128 0.92 to 1.00 of the time (3000 rows, 8 heads,
    // F = 4: 38.5 -> 35.9 us), D = 64 1.00 to 1.04 (12,000, 8, F = 2: 230 -> 239).
    static_assert(NB == 1, "one 32-key block of a tile per wave");
    constexpr int FR = C::R;
    __shared__ float mt[2][FW][32];  // row maxima of every wave's keys of a tile
    __shared__ float ms[FW][32], ls[FW][32];
    const int r = w % FR;
    float m_row = -INFINITY;  // the row's running maximum after the last weighed tile
    int32_t v_ids[LPW];  // ids of the tile that K was last loaded of; kv_ids: of the next
    auto load_k = [&](int slot_, int r0) __attribute__((always_inline)) {
      if constexpr (IDX) {
        load_tile_idx<D, FK, FW>(slot_ ? Ks1 : Ks0, ksrc, kv_ids, w, lane);
#pragma unroll
        for (int j = 0; j < LPW; ++j) v_ids[j] = kv_ids[j];  // V of this tile is loaded next
        tile_ids<D, FK, FW>(idxh, r0 + FK, S, w, lane, kv_ids);
      } else {
        load_tile<D, FK, FW>(slot_ ? Ks1 : Ks0, Kh, r0, S, w, lane);
      }
    };
    // The row's maximum after each 64 keys of the tile in slot SL; returns the one for this wave's keys.
    float mv[F];
    auto get_max = [&](auto slotc) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < F; ++x) mv[x] = mt[decltype(slotc)::value][x * FR + r][r32];
    };
    auto tile_max = [&]() __attribute__((always_inline)) {
      float mine = m_row;
#pragma unroll
      for (int x = 0; x < F; x += 2) {
        const float m = fmaxf(mv[x], mv[x + 1]);
        if (m > m_row + kRescale) m_row = m;
        if (f >= x) mine = m_row;
      }
      return mine;
    };
    auto rescale = [&](float m) __attribute__((always_inline)) {
      const float alpha = __builtin_amdgcn_exp2f(m_run - m);
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < D / 32; ++d)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[d][i] *= alpha;
      m_run = m;
    };
    // P of 16 of the 32 keys
    auto soft = [&](const f32x16& s, int u) __attribute__((always_inline)) {
      float p[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) p[t] = __builtin_amdgcn_exp2f(__builtin_fmaf(s[8 * u + t], sl2, -m_run));
      l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
      return cvt8(p);
    };
    auto pv = [&](const bf16_t* Vt, const bf16x8& p0, const bf16x8& p1) __attribute__((always_inline)) {
#pragma unroll
      for (int d = 0; d < D / 32; ++d) oacc[d] = mfma32(tr8(Vt, lo.trl[d], lo.trh[d]), p0, oacc[d]);
#pragma unroll
      for (int d = 0; d < D / 32; ++d)
        oacc[d] = mfma32(tr8(Vt, 16 * RB + lo.trl[d], 16 * RB + lo.trh[d]), p1, oacc[d]);
    };
    f32x16 sp[1] = {f32x16{}};  // logits of the tile before
    auto put_max = [&](auto slotc, float m) __attribute__((always_inline)) {
      if (h == 0) mt[decltype(slotc)::value][w][r32] = m;
    };
    // waits for K of tile kt and V of tile kt - 1, whose other slots are free, and loads the next
    auto turn = [&](auto slotc, int kt) __attribute__((always_inline)) {
      constexpr int SL = decltype(slotc)::value;
      sync_tiles<0>();
      get_max(IC<SL ^ 1>{});
      if constexpr (IDX) load_tile_idx<D, FK, FW>(SL ? Vs1 : Vs0, vsrc, v_ids, w, lane);
      else load_tile<D, FK, FW>(SL ? Vs1 : Vs0, Vh, kt * FK, S, w, lane);
      load_k(SL ^ 1, (kt + 1) * FK);
    };
    const int kw = 32 * f;  // this wave's first key of a tile
    load_k(0, 0);
    turn(IC<0>{}, 0);
    if (qw + 31 >= kw) logits(Ks0, kw, sp);
    put_max(IC<0>{}, qw + 31 >= kw ? row_max(sp) : -INFINITY);
    auto step = [&](auto slotc, int kt) __attribute__((always_inline)) {
      constexpr int SL = decltype(slotc)::value;
      turn(slotc, kt);
      const int k0 = kt * FK + kw;
      const bf16_t* const Kt = SL ? Ks1 : Ks0;
      float mloc = -INFINITY;
      f32x16 s = f32x16{};  // half of the logits while the maxima arrive
#pragma unroll
      for (int kk = 0; kk < D / 32; ++kk) s = mfma32(row8(Kt, lo.row[kk]), qreg[kk], s);
      const float mine = tile_max();
      if (qw + 31 >= k0 - FK) {  // else every key of its share was in the future of its rows
        if (mine > m_run) rescale(mine);
        __builtin_amdgcn_sched_barrier(0);
        // the rest of them under the softmax of the last tile (in the compiler's order: with
        // scheduling groups the kernel took 4 to 10% longer)
#pragma unroll
        for (int kk = D / 32; kk < D / 16; ++kk) s = mfma32(row8(Kt, lo.row[kk]), qreg[kk], s);
        const bf16x8 p0 = soft(sp[0], 0), p1 = soft(sp[0], 1);
        pv(SL ? Vs0 : Vs1, p0, p1);
        if (k0 + 31 > qw) {
#pragma unroll
          for (int i = 0; i < 16; ++i)
            if (k0 + 8 * (i >> 2) + 4 * h + (i & 3) > myq) s[i] = -INFINITY;
        }
        sp[0] = s;
        mloc = row_max(sp);
      }
      put_max(slotc, mloc);
    };
    // the last tile: V of tile nkt - 1, in slot SL
    auto last = [&](auto slotc) __attribute__((always_inline)) {
      constexpr int SL = decltype(slotc)::value;
      sync_tiles<0>();
      get_max(slotc);
      const float mine = tile_max();
      if (qw + 31 >= (nkt - 1) * FK + kw) {
        if (mine > m_run) rescale(mine);
        const bf16x8 p0 = soft(sp[0], 0), p1 = soft(sp[0], 1);
        pv(SL ? Vs1 : Vs0, p0, p1);
      }
    };
    ring2_loop(1, nkt, step);
    if (nkt & 1) last(IC<0>{});
    else last(IC<1>{});
    const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
    if (h == 0) ms[w][r32] = m_run, ls[w][r32] = l_tot;
    __syncthreads();
    float l = 0.0f, wt[F];
#pragma unroll
    for (int x = 0; x < F; ++x) {
      wt[x] = __builtin_amdgcn_exp2f(ms[x * FR + r][r32] - m_row);  // 0 for a wave without a key of the row
      l += wt[x] * ls[x * FR + r][r32];
    }
    const float inv = 1.0f / l;
    bf16_t* orow = O + (bh * S + myq) * D;
    combine<D, F, FR>(Ring{Ks0, Ks1, Vs0, Vs1}, oacc, wt, w, lane, [&](int d, int g, const float* v) {
      if (myq < S) store_quad(orow + 32 * d + 8 * g + 4 * h, v, inv);
    });
    if (myq < S && f == 0 && h == 0) LSE[bh * S + myq] = (m_row + __log2f(l)) * kLn2;
    return;
  }

  auto step = [&](auto slotc, int kt) {
    constexpr int SL = decltype(slotc)::value;
    sync_tiles<0>();  // tile kt landed in every wave; tile kt - 1 is done
    load_kv(SL ^ 1, (kt + 1) * FK);
    const int k0 = kt * FK + 32 * NB * f;  // this wave's first key of the tile
    if (qw + 31 < k0) return;  // every key of its share is in the future of this wave's rows
    const bf16_t* Kt = SL ? Ks1 : Ks0;
    const bf16_t* Vt = SL ? Vs1 : Vs0;
    f32x16 sacc[NB];
    logits(Kt, k0, sacc);
    const float mloc = row_max(sacc);
    if (mloc > m_run + kRescale) {  // new running maximum: rescale what was accumulated
      const float alpha = __builtin_amdgcn_exp2f(m_run - mloc);
      l_run *= alpha;
#pragma unroll
      for (int d = 0; d < D / 32; ++d)
#pragma unroll
        for (int i = 0; i < 16; ++i) oacc[d][i] *= alpha;
      m_run = mloc;
    }
    // P of 16 keys at a time. Step st + 1's softmax (independent of step st's MFMAs) is
    // scheduled between step st's four P V MFMAs, each MFMA's V operand read one MFMA ahead.
    float la = 0.0f, lb = 0.0f;
    auto soft = [&](int st) __attribute__((always_inline)) {
      float f[8];
#pragma unroll
      for (int t = 0; t < 8; ++t) f[t] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[st >> 1][8 * (st & 1) + t], sl2, -m_run));
      la += (f[0] + f[1]) + (f[2] + f[3]);
      lb += (f[4] + f[5]) + (f[6] + f[7]);
      return cvt8(f);
    };
    bf16x8 pcur = soft(0);
    asm volatile("" ::"v"(la), "v"(lb));  // the first step's sums stay ahead of the interleaving
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int st = 0; st < 2 * NB; ++st) {
      bf16x8 pnext = pcur;
      if (st + 1 < 2 * NB) pnext = soft(st + 1);
#pragma unroll
      for (int d = 0; d < D / 32; ++d)
        oacc[d] = mfma32(tr8(Vt, 16 * st * RB + lo.trl[d], 16 * st * RB + lo.trh[d]), pcur, oacc[d]);
      if (st + 1 < 2 * NB) {
        // groups: DS reads (mask 0x100), MFMA (0x008), VALU (0x002), transcendental (0x400)
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int d = 0; d < D / 32; ++d) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          if (d + 1 < D / 32) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);
          __builtin_amdgcn_sched_group_barrier(0x400, 2, 0);
        }
      }
      __builtin_amdgcn_sched_barrier(0);
      pcur = pnext;
    }
    l_run += la + lb;
  };
  for (int t0 = 0; t0 < nkt; t0 += 2) {
    step(IC<0>{}, t0);
    if (t0 + 1 < nkt) step(IC<1>{}, t0 + 1);
  }
  const float l_tot = l_run + __shfl_xor(l_run, 32, 64);
  if (myq < S) {
    store_qrow<D>(O + (bh * S + myq) * D, oacc, 1.0f / l_tot, h);
    if (h == 0) LSE[bh * S + myq] = (m_run + __log2f(l_tot)) * kLn2;
  }
}

// ------------------------------------------------------------------ backward: dQ
// Each wave owns 32 query rows (their Q and dO rows stay in registers) and streams the K/V
// tiles: S^T = K Q^T and dP^T = V dO^T give, per lane, one query row's
// P = exp2(S scale log2e - lse log2e) and dS = P (dP - Delta); dQ^T += K^T dS^T.
template <int D, bool IDX, int F>
__device__ __forceinline__ void
dq_block(const BlockPos bp, const Ring ring, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
         const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO, const float* __restrict__ LSE,
         const float* __restrict__ DELTA, bf16_t* __restrict__ dQ, int S, float sl2, float scale, const SdpaIdx& ix,
         const HeadMap& hm) {
  using C = BwdCfg<F>;
  constexpr int RB = 2 * D, QW = C::NW, BQ = C::ROWS, BK = C::TILE;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, r32 = lane & 31;
  const int64_t bh = bp.head;
  const int nqt = (S + BQ - 1) / BQ;
  const int q0 = (nqt - 1 - bp.rank) * BQ;
  const int f = kSplitAt<IDX, F> ? w / C::R : 0;
  const int qw = q0 + 32 * (kSplitAt<IDX, F> ? w % C::R : w);
  const int myq = qw + r32;
  const int64_t kvh = (bh / hm.Hq) * hm.Hs + (bh % hm.Hq) / hm.Gq;  // selection head
  const bf16_t* Qh = Q + bh * S * D;
  const bf16_t* Kh = K + kvh * S * D;
  const bf16_t* Vh = V + kvh * S * D;
  const bf16_t* dOh = dO + bh * S * D;
  const LaneOff<D> lo = lane_offsets<D>(lane, 32 * C::NB * f);
  constexpr int LPW = loads_per_wave<D, BK, QW>();
  RowSrc qsrc{}, ksrc{}, vsrc{};
  const int32_t* idxh = nullptr;
  int32_t kv_ids[LPW];  // ids of the next tile to be loaded
  if constexpr (IDX) {
    const int64_t b = bh / ix.Hq;
    const int hq = (int)(bh - b * ix.Hq), g = hq / ix.G;
    qsrc = row_src(ix.q, ix.qp, b, hq, ix.Hq, ix, D);
    ksrc = row_src(ix.k, ix.kp, b, g, ix.Hkv, ix, D);
    vsrc = row_src(ix.v, ix.vp, b, g, ix.Hkv, ix, D);
    idxh = ix.idx + kvh * S;
    tile_ids<D, BK, QW>(idxh, 0, S, w, lane, kv_ids);
  }
  auto load_kv = [&](int slot_, int r0) __attribute__((always_inline)) {
    bf16_t* kt_ = slot_ ? ring.a1 : ring.a0;
    bf16_t* vt_ = slot_ ? ring.b1 : ring.b0;
    if constexpr (IDX) {
      load_tile_idx<D, BK, QW>(kt_, ksrc, kv_ids, w, lane);
      load_tile_idx<D, BK, QW>(vt_, vsrc, kv_ids, w, lane);
      tile_ids<D, BK, QW>(idxh, r0 + BK, S, w, lane, kv_ids);
    } else {
      load_tile<D, BK, QW>(kt_, Kh, r0, S, w, lane);
      load_tile<D, BK, QW>(vt_, Vh, r0, S, w, lane);
    }
  };

  const int kend = q0 + BQ < S ? q0 + BQ : S;
  const int nkt = (kend + BK - 1) / BK;
  const int qrow = myq < S ? myq : S - 1;
  bf16x8 qreg[D / 16], doreg[D / 16];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) {
    const bf16_t* qr = IDX ? rs_row(qsrc, idxh[qrow]) : Qh + (int64_t)qrow * D;
    qreg[kk] = gld8(qr + 16 * kk + 8 * h);
    doreg[kk] = gld8(dOh + (int64_t)qrow * D + 16 * kk + 8 * h);
  }
  const float lse2 = myq < S ? LSE[bh * S + myq] * kLog2e : INFINITY;
  const float dlt = myq < S ? DELTA[bh * S + myq] : 0.0f;
  // every element of a lane's dP^T accumulator belongs to the lane's query row: the chain starts
  // from -Delta (a separate source operand of its first MFMA), so it ends as dP - Delta and no
  // subtraction is needed
  f32x16 ndlt;
#pragma unroll
  for (int i = 0; i < 16; ++i) ndlt[i] = -dlt;
  load_kv(0, 0);
  f32x16 dqacc[D / 32];
#pragma unroll
  for (int d = 0; d < D / 32; ++d) dqacc[d] = f32x16{};

  // Key tiles that end before q0 hold no key after any row of the block: no mask. Only the last
  // tiles (the diagonal band) run the masked body.
  auto step = [&](auto slotc, auto maskc, int kt) __attribute__((always_inline)) {
    constexpr int SL = decltype(slotc)::value;
    constexpr bool MASK = decltype(maskc)::value != 0;
    sync_tiles<0>();
    load_kv(SL ^ 1, (kt + 1) * BK);
    const int k0 = kt * BK + 32 * C::NB * f;  // this wave's first key of the tile
    if (qw + 31 < k0) return;
    const bf16_t* Kt = ring.a<SL>();
    const bf16_t* Vt = ring.b<SL>();
#pragma unroll
    for (int kb = 0; kb < C::NB; ++kb) {
      f32x16 sacc = f32x16{};
      f32x16 pacc = mfma32(row8(Vt, kb * 32 * RB + lo.row[0]), doreg[0], ndlt);
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        sacc = mfma32(row8(Kt, kb * 32 * RB + lo.row[kk]), qreg[kk], sacc);
        if (kk > 0) pacc = mfma32(row8(Vt, kb * 32 * RB + lo.row[kk]), doreg[kk], pacc);
      }
      // causal mask: element i holds key k0 + 32 kb + 4h + c_i, c_i = 8 (i / 4) + i % 4, which is
      // in the future of the lane's query exactly when c_i > tm
      const int tm = myq - k0 - kb * 32 - 4 * h;
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float f[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const int i = 8 * u + t;
          float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], sl2, -lse2));
          if (MASK && 8 * (i >> 2) + (i & 3) > tm) pv = 0.0f;
          f[t] = pv * pacc[i];
        }
        const bf16x8 db = cvt8(f);
#pragma unroll
        for (int d = 0; d < D / 32; ++d)
          dqacc[d] = mfma32(tr8(Kt, (kb * 32 + 16 * u) * RB + lo.trl[d], (kb * 32 + 16 * u) * RB + lo.trh[d]), db,
                            dqacc[d]);
      }
    }
  };
  const int nfree = q0 / BK < nkt ? q0 / BK : nkt;  // tiles [0, nfree) need no mask
  auto plain = [&](auto slotc, int kt) __attribute__((always_inline)) { step(slotc, IC<0>{}, kt); };
  auto masked = [&](auto slotc, int kt) __attribute__((always_inline)) { step(slotc, IC<1>{}, kt); };
  ring2_loop(0, nfree, plain);
  ring2_loop(nfree, nkt, masked);
  if constexpr (F > 1) {
    float one[F];
#pragma unroll
    for (int x = 0; x < F; ++x) one[x] = 1.0f;
    sync_tiles<0>();  // the last (unused) tile has landed
    bf16_t* row = dQ + (bh * S + myq) * D;
    combine<D, F, C::R>(ring, dqacc, one, w, lane, [&](int d, int g, const float* v) {
      if (myq < S) store_quad(row + 32 * d + 8 * g + 4 * h, v, scale);
    });
  } else {
    if (myq < S) store_qrow<D>(dQ + (bh * S + myq) * D, dqacc, scale, h);
  }
}

// ------------------------------------------------------------------ backward: dK, dV
// Each wave owns 32 keys: their V rows stay in registers and the workgroup's K rows stay in
// LDS for the whole kernel. Query tiles, with their lse and Delta, stream through two LDS slots:
// S = Q K^T and dP = dO V^T (per lane: one key, 16 queries), then dV += P^T dO and
// dK += dS^T Q with the transposed dO / Q operands read from the same tiles. Each query tile
// is processed in two 32-row halves to bound the live registers. The lse / Delta of a tile
// pass through registers, so each step waits for all of the wave's loads before the barrier.
// GRP: the workgroup's keys belong to a selection shared by hm.Gq query heads; their dK, dV sum
// over those heads (one pass of the query-tile loop per head, the accumulators kept).
template <int D, bool IDX, bool GRP, int F>
__device__ __forceinline__ void
dkdv_block(const BlockPos bp, const Ring ring, float* const ls0, float* const ls1, float* const ds0,
           float* const ds1, bf16_t* const Kw, const bf16_t* __restrict__ Q, const bf16_t* __restrict__ K,
           const bf16_t* __restrict__ V, const bf16_t* __restrict__ dO, const float* __restrict__ LSE,
           const float* __restrict__ DELTA, bf16_t* __restrict__ dK, bf16_t* __restrict__ dV, int S, float sl2,
           float scale, const SdpaIdx& ix, const HeadMap& hm) {
  using C = BwdCfg<F>;
  constexpr int RB = 2 * D, KWV = C::NW, CK = C::ROWS, CQ = C::TILE;
  bf16_t *const Qs0 = ring.a0, *const Qs1 = ring.a1, *const dOs0 = ring.b0, *const dOs1 = ring.b1;
  const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int h = lane >> 5, r32 = lane & 31;
  const int64_t bs = bp.head;  // b * Hs + hs: the selection head whose keys this block owns
  const int64_t bsb = bs / hm.Hs;
  const int hs0 = (int)(bs - bsb * hm.Hs);
  int64_t bh = bsb * hm.Hq + (int64_t)hs0 * hm.Gq;  // the query head being streamed
  const int k0 = bp.rank * CK;  // early keys see the most queries: launched first
  const int r = kSplitAt<IDX, F> ? w % C::R : w, f = kSplitAt<IDX, F> ? w / C::R : 0;
  const int kw = k0 + 32 * r;
  const int mykey = kw + r32;
  const bf16_t* Qh = Q + bh * S * D;
  const bf16_t* Kh = K + bs * S * D;
  const bf16_t* Vh = V + bs * S * D;
  const bf16_t* dOh = dO + bh * S * D;
  const float* Lh = LSE + bh * S;
  const float* Dh = DELTA + bh * S;
  const LaneOff<D> lo = lane_offsets<D>(lane, 32 * C::NB * f);
  // the K operand's row block is r, not the tile share f
  const int kwo = (r - C::NB * f) * 32 * RB;
  RowSrc qsrc{}, ksrc{}, vsrc{};
  const int32_t* idxh = nullptr;
  int32_t q_ids[loads_per_wave<D, CQ, KWV>()];  // ids of the next query tile to be staged
  if constexpr (IDX) {
    const int hq = hs0 * hm.Gq, g = hq / ix.G;
    qsrc = row_src(ix.q, ix.qp, bsb, hq, ix.Hq, ix, D);
    ksrc = row_src(ix.k, ix.kp, bsb, g, ix.Hkv, ix, D);
    vsrc = row_src(ix.v, ix.vp, bsb, g, ix.Hkv, ix, D);
    idxh = ix.idx + bs * S;
  }

  const int qstart = (k0 / CQ) * CQ;
  const int nqt = (S - qstart + CQ - 1) / CQ;
  // lse and Delta of a query tile enter LDS through the first CQ threads. The tile staged
  // before the loop is written at once; a tile staged inside the loop has its two values loaded
  // into nl, nd when its Q / dO copies are issued and written to LDS just before the barrier that
  // publishes the tile, so no wave waits for those loads in the middle of a tile.
  float nl = 0.0f, nd = 0.0f;
  auto put_ld = [&](auto bufc, int qt0, float lv, float dv) __attribute__((always_inline)) {
    constexpr int BUF = decltype(bufc)::value;
    const bool in = qt0 + tid < S;
    (BUF ? ls1 : ls0)[tid] = in ? lv * kLog2e : INFINITY;  // rows past S: P = 0
    (BUF ? ds1 : ds0)[tid] = in ? -dv : 0.0f;  // negated: it seeds the dP accumulator
  };
  auto stage = [&](auto bufc, auto deferc, int qt0) __attribute__((always_inline)) {
    constexpr int BUF = decltype(bufc)::value;
    if constexpr (IDX) load_tile_idx<D, CQ, KWV>(BUF ? Qs1 : Qs0, qsrc, q_ids, w, lane);
    else load_tile<D, CQ, KWV>(BUF ? Qs1 : Qs0, Qh, qt0, S, w, lane);
    load_tile<D, CQ, KWV>(BUF ? dOs1 : dOs0, dOh, qt0, S, w, lane);
    if (tid < CQ) {
      const int q = qt0 + tid < S ? qt0 + tid : S - 1;  // clamped; rows past S are masked in put_ld
      if constexpr (decltype(deferc)::value) {
        nl = Lh[q];
        nd = Dh[q];
      } else {
        put_ld(bufc, qt0, Lh[q], Dh[q]);
      }
    }
    // tiles are staged from the last one down: the next one starts CQ rows earlier
    if constexpr (IDX) tile_ids<D, CQ, KWV>(idxh, qt0 - CQ > 0 ? qt0 - CQ : 0, S, w, lane, q_ids);
  };
  // Query tiles are visited from the last one down to the diagonal: every key block of a head
  // then starts on the same tile and streams the same tiles in step with the others, so the
  // blocks running together on an XCD share each Q / dO tile through its L2.
  const int qlast = qstart + (nqt - 1) * CQ;
  if constexpr (IDX) {
    int32_t k_ids[loads_per_wave<D, CK, KWV>()];
    tile_ids<D, CK, KWV>(idxh, k0, S, w, lane, k_ids);
    load_tile_idx<D, CK, KWV>(Kw, ksrc, k_ids, w, lane);
    tile_ids<D, CQ, KWV>(idxh, qlast, S, w, lane, q_ids);
  } else {
    load_tile<D, CK, KWV>(Kw, Kh, k0, S, w, lane);
  }
  stage(IC<0>{}, IC<0>{}, qlast);

  const int krow = mykey < S ? mykey : S - 1;
  const bf16_t* vrow = IDX ? rs_row(vsrc, idxh[krow]) : Vh + (int64_t)krow * D;
  bf16x8 vreg[D / 16];
#pragma unroll
  for (int kk = 0; kk < D / 16; ++kk) vreg[kk] = gld8(vrow + 16 * kk + 8 * h);
  f32x16 dkacc[D / 32], dvacc[D / 32];
#pragma unroll
  for (int d = 0; d < D / 32; ++d) dkacc[d] = dvacc[d] = f32x16{};

  auto tile = [&](auto bufc, auto maskc, int it) __attribute__((always_inline)) {
    constexpr int BUF = decltype(bufc)::value;
    constexpr bool MASK = decltype(maskc)::value != 0;
    const bf16_t* Qt = BUF ? Qs1 : Qs0;
    const bf16_t* dOt = BUF ? dOs1 : dOs0;
    const int qt0 = qlast - it * CQ;
    if (it > 0 && tid < CQ) put_ld(bufc, qt0, nl, nd);  // staged with the previous tile
    sync_tiles<0>();  // this tile (and its lse / Delta) landed; the other slot is free
    if (it + 1 < nqt) stage(IC<BUF ^ 1>{}, IC<1>{}, qt0 - CQ);
    const int qs0 = qt0 + 32 * C::NB * f;  // this wave's first query of the tile
    if (qs0 + 32 * C::NB - 1 < kw || kw >= S) return;  // every query of its share precedes its keys
    const float* lt = (BUF ? ls1 : ls0) + 32 * C::NB * f;
    const float* dt = (BUF ? ds1 : ds0) + 32 * C::NB * f;
#pragma unroll
    for (int qb = 0; qb < C::NB; ++qb) {
      // causal mask: element i holds query row qs0 + 32 qb + 4h + c_i, c_i = 8 (i / 4) + i % 4, so
      // P = 0 exactly where c_i < t (t < 0 on every tile after this wave's diagonal one)
      const int tmask = mykey - qs0 - 32 * qb - 4 * h;
      // the dP accumulator starts at -Delta (stored negated), so it ends as dP - Delta
      f32x16 sacc = f32x16{}, pacc;
#pragma unroll
      for (int g = 0; g < 4; ++g) {  // rows qb * 32 + 8 g + 4 h + 0..3 of the C layout
        const float4 d4 = *reinterpret_cast<const float4*>(dt + qb * 32 + 8 * g + 4 * h);
        pacc[4 * g + 0] = d4.x, pacc[4 * g + 1] = d4.y, pacc[4 * g + 2] = d4.z, pacc[4 * g + 3] = d4.w;
      }
#pragma unroll
      for (int kk = 0; kk < D / 16; ++kk) {
        sacc = mfma32(row8(Qt, qb * 32 * RB + lo.row[kk]), row8(Kw, kwo + lo.row[kk]), sacc);
        pacc = mfma32(row8(dOt, qb * 32 * RB + lo.row[kk]), vreg[kk], pacc);
        if (kk & 1) __builtin_amdgcn_sched_barrier(0);  // bound the operand loads in flight
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        float pf[8], df[8];
#pragma unroll
        for (int g = 0; g < 2; ++g) {
          const int qg = qb * 32 + 16 * u + 8 * g + 4 * h;  // tile rows qg .. qg + 3
          const float4 l4 = *reinterpret_cast<const float4*>(lt + qg);
          const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int i = 8 * u + 4 * g + j;
            float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[i], sl2, -lv[j]));
            if (MASK && 8 * (i >> 2) + (i & 3) < tmask) pv = 0.0f;
            pf[4 * g + j] = pv;
            df[4 * g + j] = pv * pacc[i];
          }
        }
        const bf16x8 pb = cvt8(pf), db = cvt8(df);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < D / 32; ++d) {
          dvacc[d] = mfma32(pb, tr8(dOt, (qb * 32 + 16 * u) * RB + lo.trl[d], (qb * 32 + 16 * u) * RB + lo.trh[d]),
                            dvacc[d]);
          dkacc[d] = mfma32(db, tr8(Qt, (qb * 32 + 16 * u) * RB + lo.trl[d], (qb * 32 + 16 * u) * RB + lo.trh[d]),
                            dkacc[d]);
          if (d & 1) __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  };
  // Query tiles at or after k0 + CK hold no query before any key of the block: no mask. Only the
  // last tiles visited (the diagonal band) run the masked body.
  constexpr int NMASK = CK > CQ ? CK / CQ : 1;
  const int nfree = nqt > NMASK ? nqt - NMASK : 0;
  auto plain = [&](auto bufc, int it) __attribute__((always_inline)) { tile(bufc, IC<0>{}, it); };
  auto masked = [&](auto bufc, int it) __attribute__((always_inline)) { tile(bufc, IC<1>{}, it); };
  for (int mq = 0;;) {
    ring2_loop(0, nfree, plain);
    ring2_loop(nfree, nqt, masked);
    if (!GRP || ++mq >= hm.Gq) break;
    // next query head of the selection: restart the tile stream once every wave is done with
    // the buffers of the last tile
    __syncthreads();
    ++bh;
    Qh += (int64_t)S * D;
    dOh += (int64_t)S * D;
    Lh += S;
    Dh += S;
    if constexpr (IDX) {
      qsrc = row_src(ix.q, ix.qp, bsb, hs0 * hm.Gq + mq, ix.Hq, ix, D);
      tile_ids<D, CQ, KWV>(idxh, qlast, S, w, lane, q_ids);
    }
    stage(IC<0>{}, IC<0>{}, qlast);
  }
  // C layout: row = key kw + 8(i/4) + 4h + i%4, column 32 d + lane % 32
  if constexpr (F > 1) {
    float one[F];
#pragma unroll
    for (int x = 0; x < F; ++x) one[x] = 1.0f;
    auto put = [&](bf16_t* dst, float mul) __attribute__((always_inline)) {
      return [=](int d, int g, const float* v) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const int key = kw + 8 * g + 4 * h + j;
          if (key < S) dst[(bs * S + key) * D + 32 * d + r32] = f2bf(v[j] * mul);
        }
      };
    };
    combine<D, F, C::R>(ring, dkacc, one, w, lane, put(dK, scale));
    combine<D, F, C::R>(ring, dvacc, one, w, lane, put(dV, 1.0f));
  } else {
#pragma unroll
    for (int d = 0; d < D / 32; ++d)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int key = kw + 8 * (i >> 2) + 4 * h + (i & 3);
        if (key < S) {
          dK[(bs * S + key) * D + 32 * d + r32] = f2bf(dkacc[d][i] * scale);
          dV[(bs * S + key) * D + 32 * d + r32] = f2bf(dvacc[d][i]);
        }
      }
  }
}

// ------------------------------------------------------------------ backward: the launch
// dK/dV and dQ workgroups in one launch: they are independent and of one shape (8 waves, one
// workgroup per CU at D = 128), so the long dQ blocks fill the CUs that the last dK/dV blocks
// leave idle. Against two launches, F = 1: S = 2000, 8 heads 169 -> 103 us; 18,432, 8 heads 2161
// -> 2060; 10,752, 32 heads on 8 selections 3475 -> 2950 to 3010 (the call alone); no difference on a full chip (54,272, 32
// heads). Alternating the ranks of dK/dV and dQ blocks instead of all dK/dV first was slower
// (18,432, 8 heads 2269): the blocks running together then stream more different tiles through
// each L2. LDS is shared by name: dQ's K / V ring is dK/dV's Q / dO ring.
struct BwdArgs {
  const bf16_t *q, *k, *v, *go;
  const float *lse, *delta;
  bf16_t *dq, *dk, *dv;
  int S;
  uint32_t kheads, qheads;  // heads of dK/dV and of dQ blocks
  uint32_t kblocks;         // dK/dV blocks, the first of the launch
  float sl2, scale;
};

template <int D, bool IDX, bool GRP, int F>
__global__ void __launch_bounds__(64 * BwdCfg<F>::NW)
    __attribute__((amdgpu_waves_per_eu(BwdCfg<F>::EU, BwdCfg<F>::EU)))
sdpa_bwd_bf16(BwdArgs a, SdpaIdx ix, HeadMap hm) {
  using C = BwdCfg<F>;
  constexpr int CQ = C::TILE, CK = C::ROWS;
  // LDS is laid out by decreasing alignment: the lse / Delta rows first, then the streamed tiles,
  // so that with F < 4 both sit inside the first 64 KB, where a base address folds into the
  // 16-bit immediate offset of the LDS reads (the deepest tile read ends below 63 KB); K comes last.
  __shared__ __align__(128) float ls0[CQ], ls1[CQ], ds0[CQ], ds1[CQ];
  __shared__ __align__(64) bf16_t A0[CQ * D], A1[CQ * D], B0[CQ * D], B1[CQ * D];
  __shared__ __align__(16) bf16_t Kw[CK * D];
  const uint32_t lin = blockIdx.x;
  const Ring ring{A0, A1, B0, B1};
  if (lin < a.kblocks)
    dkdv_block<D, IDX, GRP, F>(block_pos(lin, a.kheads), ring, ls0, ls1, ds0, ds1, Kw, a.q, a.k, a.v, a.go, a.lse,
                               a.delta, a.dk, a.dv, a.S, a.sl2, a.scale, ix, hm);
  else
    dq_block<D, IDX, F>(block_pos(lin - a.kblocks, a.qheads), ring, a.q, a.k, a.v, a.go, a.lse, a.delta, a.dq, a.S, a.sl2,
                        a.scale, ix, hm);
}

// The split F of a launch (FwdCfg, BwdCfg): the one whose workgroups, taken in launch order by 256 CUs, one
// at a time, end first. A workgroup takes `fixed` us and `tile` us per tile; a launch of more than 256
// takes the longer of its longest chain and an even share of the sum, and with more than two a CU somewhat
// more where both are alike (the 4-norm of the two). The constants are fits to 3800 shapes of each direction
// (S = 33 .. 130,000, 1 .. 256 heads, groups of 1 .. 8), each timed with every F. Over those the split chosen
// so takes 0.1% (forward) and 0.2% (backward) longer than the best one, at worst 18%; on shapes that the fit
// did not see 0.1 and 0.2% too. Lines drawn at numbers of row blocks took 1% longer, and on rows of up to 1500 7%: those
// of many heads fill the chip with any F. Forward, us for F = 1, 2, 4, D = 128: S = 160, 192 heads (one
// round of 192 workgroups; two; three) 12.7, 16.7, 21.3; 192, 128 12.7, 10.1, 14.8; 512, 64 22.3, 15.8, 18.6;
// 1438, 64 60.2, 63.7, 82.8; 5000, 7 172, 84.5, 82.2; 24,000, 5 915, 839, 1049; 12,000, 12 472, 499, 608.
// Backward: S = 160, 96 heads 18.6, 23.2, 31.9; 1024, 48 68.0, 79.4, 108; 2000, 8 95.2, 62.9, 54.7; 8000, 6
// 392, 344, 420; 10,752, 8 on 2 selections 1975, 1130, 950.
struct SplitCost {
  double fixed, tile;
};
constexpr SplitCost kFwdCost[2][3] = {{{3.72, 1.479}, {4.84, 0.604}, {4.55, 0.664}},   // D = 64: F = 1, 2, 4
                                      {{4.60, 2.20}, {6.52, 0.949}, {6.74, 1.21}}};  // D = 128
constexpr SplitCost kBwdCost[2][3] = {{{1.63, 1.772}, {3.96, 0.96}, {3.61, 1.092}},
                                      {{2.42, 2.954}, {6.49, 1.671}, {6.27, 2.107}}};
constexpr int64_t kCUs = 256;

// `jobs` workgroups of `sum` tiles together; tiles(i): of job i in launch order; longest: of the longest job;
// shortest(i): the fewest tiles among the jobs before job i (forward: and i).
template <typename Tiles, typename Shortest>
static double split_time(SplitCost c, int64_t jobs, double sum, int64_t longest, Tiles tiles, Shortest shortest) {
  double chain = c.fixed + c.tile * longest;
  if (jobs <= kCUs) return chain;
  for (int64_t k = 1; k <= 3 && k * kCUs < jobs; ++k) {  // job 256 k comes after k jobs or more of its CU
    const double x = (k + 1) * c.fixed + c.tile * (k * shortest(k * kCUs) + tiles(k * kCUs));
    chain = x > chain ? x : chain;
  }
  const double share = (c.fixed * jobs + c.tile * sum) / kCUs;
  if (jobs <= 2 * kCUs) return share > chain ? share : chain;
  return sqrt(sqrt(chain * chain * chain * chain + share * share * share * share));
}

// The tiles of a head's n row blocks of R rows, tiles of T columns: block j ends at tile ends(j); sum over j.
struct RowTiles {
  int64_t S, n;
  int R, T;
  RowTiles(int64_t S_, int R_, int T_) : S(S_), n((S_ + R_ - 1) / R_), R(R_), T(T_) {}
  int64_t ends(int64_t j) const { return ((j + 1 < n ? (j + 1) * R : S) + T - 1) / T; }
  int64_t starts(int64_t j) const { return j * R / T; }
  double sum_ends() const { return ends(n - 1) + (R >= T ? (double)(R / T) * n * (n - 1) / 2 : (double)n * n / 4); }
  double sum_starts() const { return R >= T ? (double)(R / T) * n * (n - 1) / 2 : (double)(n - 1) * (n - 1) / 4; }
};

template <int F>
static double fwd_time(const LhShape& s) {
  const RowTiles t(s.S, FwdCfg<F>::ROWS, FwdCfg<F>::TILE);
  const int64_t heads = s.B * s.Hq;
  auto tiles = [&](int64_t i) { return t.ends(t.n - 1 - i / heads); };  // longest first
  return split_time(kFwdCost[s.D == 128][F / 2], t.n * heads, heads * t.sum_ends(), tiles(0), tiles, tiles);
}

template <int F>
static double bwd_time(const LhShape& s) {
  const RowTiles t(s.S, BwdCfg<F>::ROWS, BwdCfg<F>::TILE);
  const int64_t kheads = s.B * s.Hs, qheads = s.B * s.Hq, nk = t.n * kheads, all = t.ends(t.n - 1);
  auto tiles = [&](int64_t i) {  // dK/dV blocks, then dQ blocks, the longest of each first
    return i < nk ? s.Gq * (all - t.starts(i / kheads)) : t.ends(t.n - 1 - (i - nk) / qheads);
  };
  auto shortest = [&](int64_t i) {
    const int64_t x = tiles(i - 1), y = i <= nk ? x : tiles(nk - 1);
    return x < y ? x : y;
  };
  const double sum = kheads * s.Gq * (t.n * (double)all - t.sum_starts()) + qheads * t.sum_ends();
  return split_time(kBwdCost[s.D == 128][F / 2], nk + t.n * qheads, sum, s.Gq * all, tiles, shortest);
}

static int least(double t1, double t2, double t4) { return t4 <= t2 && t4 <= t1 ? 4 : t2 <= t1 ? 2 : 1; }
static int fwd_split(const LhShape& s) { return least(fwd_time<1>(s), fwd_time<2>(s), fwd_time<4>(s)); }
static int bwd_split(const LhShape& s) { return least(bwd_time<1>(s), bwd_time<2>(s), bwd_time<4>(s)); }

template <int D, bool IDX, int F>
static void launch_fwd_F(const LhShape& s, const void* qs, const void* ks, const void* vs, void* os, float* lse,
                         const SdpaIdx& ix, hipStream_t st) {
  using C = FwdCfg<F>;
  const int S = (int)s.S;
  const HeadMap hm{s.Hq, s.Hs, s.Gq};
  const uint32_t heads = (uint32_t)(s.B * s.Hq);
  const dim3 grid((uint32_t)((s.S + C::ROWS - 1) / C::ROWS) * heads);
  hipLaunchKernelGGL((sdpa_fwd_bf16<D, IDX, F>), grid, dim3(64 * C::NW), 0, st, (const bf16_t*)qs, (const bf16_t*)ks,
                     (const bf16_t*)vs, (bf16_t*)os, lse, S, heads, s.scale * kLog2e, ix, hm);
}

template <int D, bool IDX>
static void launch_fwd_D(const LhShape& s, const void* qs, const void* ks, const void* vs, void* os, float* lse,
                         const SdpaIdx& ix, hipStream_t st) {
  switch (fwd_split(s)) {
    case 1: launch_fwd_F<D, IDX, 1>(s, qs, ks, vs, os, lse, ix, st); break;
    case 2: launch_fwd_F<D, IDX, 2>(s, qs, ks, vs, os, lse, ix, st); break;
    default: launch_fwd_F<D, IDX, 4>(s, qs, ks, vs, os, lse, ix, st); break;
  }
}

template <bool IDX>
static void launch_fwd(const LhShape& s, const void* qs, const void* ks, const void* vs, void* os, float* lse,
                       const SdpaIdx& ix, hipStream_t st) {
  if (s.D == 128) launch_fwd_D<128, IDX>(s, qs, ks, vs, os, lse, ix, st);
  else launch_fwd_D<64, IDX>(s, qs, ks, vs, os, lse, ix, st);
}

template <int D, bool IDX, bool GRP, int F>
static void launch_bwd_F(const LhShape& s, BwdArgs a, const SdpaIdx& ix, hipStream_t st) {
  using C = BwdCfg<F>;
  const HeadMap hm{s.Hq, s.Hs, s.Gq};
  const uint32_t n = (uint32_t)((s.S + C::ROWS - 1) / C::ROWS);
  a.kblocks = n * a.kheads;
  const dim3 grid(a.kblocks + n * a.qheads);
  hipLaunchKernelGGL((sdpa_bwd_bf16<D, IDX, GRP, F>), grid, dim3(64 * C::NW), 0, st, a, ix, hm);
}

template <int D, bool IDX, bool GRP>
static void launch_bwd_D(const LhShape& s, const BwdArgs& a, const SdpaIdx& ix, hipStream_t st) {
  switch (bwd_split(s)) {
    case 1: launch_bwd_F<D, IDX, GRP, 1>(s, a, ix, st); break;
    case 2: launch_bwd_F<D, IDX, GRP, 2>(s, a, ix, st); break;
    default: launch_bwd_F<D, IDX, GRP, 4>(s, a, ix, st); break;
  }
}

template <bool IDX>
static void launch_bwd(const LhShape& s, const void* qs, const void* ks, const void* vs, const void* dos,
                       const float* lse, const float* delta, void* dqs, void* dks, void* dvs, const SdpaIdx& ix,
                       hipStream_t st) {
  const BwdArgs a{(const bf16_t*)qs, (const bf16_t*)ks, (const bf16_t*)vs, (const bf16_t*)dos, lse, delta,
                  (bf16_t*)dqs, (bf16_t*)dks, (bf16_t*)dvs, (int)s.S, (uint32_t)(s.B * s.Hs),
                  (uint32_t)(s.B * s.Hq), 0, s.scale * kLog2e, s.scale};
  const bool grp = s.Gq > 1;
  if (s.D == 128) {
    if (grp) launch_bwd_D<128, IDX, true>(s, a, ix, st);
    else launch_bwd_D<128, IDX, false>(s, a, ix, st);
  } else {
    if (grp) launch_bwd_D<64, IDX, true>(s, a, ix, st);
    else launch_bwd_D<64, IDX, false>(s, a, ix, st);
  }
}

static SdpaIdx make_idx(const LhShape& s, const void* q, const void* k, const void* v, const void* qp,
                        const void* kp, const void* vp, const int32_t* idx) {
  SdpaIdx ix{};
  ix.q = (const bf16_t*)q, ix.k = (const bf16_t*)k, ix.v = (const bf16_t*)v;
  // with L = 1 there is no pyramid: every id is below N, the pointers are never followed
  ix.qp = qp ? (const bf16_t*)qp : ix.q;
  ix.kp = kp ? (const bf16_t*)kp : ix.k;
  ix.vp = vp ? (const bf16_t*)vp : ix.v;
  ix.idx = idx;
  ix.N = s.N, ix.R = s.R > 0 ? s.R : 0;
  ix.Hq = s.Hq, ix.Hkv = s.Hkv, ix.G = s.G;
  return ix;
}

}  // namespace lh

using namespace lh;

hipError_t lh_launch_sdpa_fwd_bf16(const LhShape& s, const void* qs, const void* ks, const void* vs, void* os,
                                   float* lse, hipStream_t st) {
  launch_fwd<false>(s, qs, ks, vs, os, lse, SdpaIdx{}, st);
  return hipGetLastError();
}

hipError_t lh_launch_sdpa_bwd_bf16(const LhShape& s, const void* qs, const void* ks, const void* vs,
                                   const void* dos, const float* lse, const float* delta, void* dqs,
                                   void* dks, void* dvs, hipStream_t st) {
  launch_bwd<false>(s, qs, ks, vs, dos, lse, delta, dqs, dks, dvs, SdpaIdx{}, st);
  return hipGetLastError();
}

hipError_t lh_launch_sdpa_fwd_idx(const LhShape& s, const void* q, const void* k, const void* v, const void* qp,
                                  const void* kp, const void* vp, const int32_t* idx, void* os, float* lse,
                                  hipStream_t st) {
  launch_fwd<true>(s, nullptr, nullptr, nullptr, os, lse, make_idx(s, q, k, v, qp, kp, vp, idx), st);
  return hipGetLastError();
}

hipError_t lh_launch_sdpa_bwd_idx(const LhShape& s, const void* q, const void* k, const void* v, const void* qp,
                                  const void* kp, const void* vp, const int32_t* idx, const void* dos,
                                  const float* lse, const float* delta, void* dqs, void* dks, void* dvs,
                                  hipStream_t st) {
  launch_bwd<true>(s, nullptr, nullptr, nullptr, dos, lse, delta, dqs, dks, dvs,
                   make_idx(s, q, k, v, qp, kp, vp, idx), st);
  return hipGetLastError();
}
