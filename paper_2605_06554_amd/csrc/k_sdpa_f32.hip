// k_sdpa_f32.hip -- fp32 causal SDPA on the gathered sub-sequence with bf16 MFMA on split operands
// (Sec. 3.5, Eq. attn-sub with Eq. sdpa): forward, and the deterministic backward (dK/dV and dQ
// workgroups in one launch), per (b, hq) over [S, D] rows.
//
// Arithmetic. An fp32 value is split into three bf16 values (8 + 8 + 8 bits), whose sum it is
// exactly where its low part is in bf16's normal range (2^-103 and up). A product is formed
// from six of the nine products of parts, exact each, summed in the MFMA's fp32 accumulator (G. Henry, P.
// Tang, A. Heinecke, "Leveraging the bfloat16 artificial intelligence datatype for higher-precision
// computations", 2019). What is left out is below 2^-22 of a product and of either sign; that is
// less than the fp32 accumulation rounds off.
// Measured against 64 bits (2-norm, S = 2257, 8 heads, D = 128): o 2.9e-7, dQ 4.7e-7, dK 6.3e-7, dV
// 5.9e-7; with fp32 MFMA (v_mfma_f32_32x32x2) 3.6e-7, 5.5e-7, 7.5e-7, 7.0e-7; with fp32 FMAs, a thread
// per row, dK 1.2e-6. 16 columns of a 32 x 32 tile take 6 MFMAs of 32 clocks; the fp32 MFMA takes 8 of 64.
//
// Bound and split. A wave splits the streamed operand as it reads it (44 VALU instructions of 4
// clocks per 6 MFMAs), so the vector and the matrix units are about equally busy, and on few or short
// heads the time is that of a workgroup's chain of tiles. fp32 problems are small (a few thousand
// rows, a few heads), so the split of the work is for many waves: a workgroup owns 32 rows, and its
// NF waves share out the 32-row tiles that those rows meet (wave f takes tiles f, f + NF, ...). Each
// wave streams its tiles into LDS buffers of its own, without a barrier in the loop: the two operand
// tiles are used in different phases, so each is reloaded as soon as its last phase is done and lands
// under the next phase. The waves' partial results are summed in LDS at the end, in wave order
// (deterministic).
// Of the two split row operands of the backward, one is held in registers and one, which is the same for
// all waves, in LDS: with both in registers (96 each at D = 128, 48 at D = 64) the tile loops spilled
// 38 and 72 registers, and a reload waits for the tile prefetch issued before it. Backward with
// and without: S = 1000, 2 heads, D = 128 66.3 / 60.8 us; 2257 rows, 8 heads on 2 515 / 447; S = 832,
// 2 heads, D = 64 33.9 / 27.9; 4000, 8, 64 435 / 382.
// Forward / backward, us: S = 2257, 8 heads, D = 128: a thread per row 8950 / 62,900; fp32 MFMA in
// this split 130 / 372; this 99 / 283. S = 832, 2 heads, D = 64: 945 / 1780; 20.8 / 37.7; 15.6 /
// 27.9. S = 6000, 8 heads, D = 128: fp32 MFMA 774 / 2320, this 555 / 1730.
//
// Layout facts (lane l of a wave, h = l / 32):
//   MFMA 32x32x16: A[m = l % 32][k = 8 h + 0..7], B[k = 8 h + 0..7][n = l % 32],
//                  C[m = 8 (i / 4) + 4 h + i % 4][n = l % 32], i = 0..15.
//   A product over D takes columns 16 s + 4 h + 0..3 and 16 s + 8 + 4 h + 0..3 as a lane's 8 (two
//   16-byte reads). A product over the 32 rows of a tile takes rows 8 (i / 4) + 4 h + i % 4 for i =
//   8 u .. 8 u + 7, so the accumulator elements of those i, split, are that step's operand.
//
// A non-finite element of row j reaches no row before j of o and dQ, and one of Q or dO no key after j in dK
// and dV (contain). What it does reach is not finite, but may be NaN where fp32
// arithmetic has an infinity: the parts of an infinity are infinity and NaN.
//
// LDS tiles: 32 rows of D floats, chunk c (16 bytes) of row r at position c ^ (r mod chunks), so
// that the lanes reading one chunk of consecutive rows hit different banks.
#include <float.h>

#include <type_traits>

#include "lh_common.h"

namespace lh {

constexpr float kLog2eF = 1.4426950408889634f;

__device__ __forceinline__ f32x16 mfma_b16(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// 8 fp32 values as three bf16 vectors whose sum they are (see above for the smallest): h is the value cut to its top 16
// bits (8 significant ones; cut, not rounded, so that no finite value becomes infinite), m the rest
// rounded to 8 bits, l what is left, which has 8 bits or fewer.
struct Split8 {
  bf16x8 h, m, l;
};
typedef __attribute__((__vector_size__(8 * sizeof(float)))) float f32x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4s;
typedef __attribute__((__vector_size__(8 * sizeof(uint16_t)))) uint16_t u16x8;
__device__ __forceinline__ Split8 split8(const float* x) {
  Split8 r;
  u32x4s hp;
  f32x8 d, e;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t a = __float_as_uint(x[2 * i]), b = __float_as_uint(x[2 * i + 1]);
    hp[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);  // the upper halves of a and b
    d[2 * i] = x[2 * i] - __uint_as_float(a & 0xffff0000u);
    d[2 * i + 1] = x[2 * i + 1] - __uint_as_float(b & 0xffff0000u);
  }
  r.h = __builtin_bit_cast(bf16x8, hp);
  r.m = __builtin_convertvector(d, bf16x8);
  const u32x4s mp = __builtin_bit_cast(u32x4s, r.m);
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    e[2 * i] = d[2 * i] - __uint_as_float(mp[i] << 16);
    e[2 * i + 1] = d[2 * i + 1] - __uint_as_float(mp[i] & 0xffff0000u);
  }
  r.l = __builtin_convertvector(e, bf16x8);
  return r;
}

// acc += a b: the six products of the parts down to 2^-16 of the whole, smallest first. Left out are
// m l and l m, each below 2^-23 of a product (m is up to 2^-7 of its value, l up to 2^-16), and l l.
__device__ __forceinline__ f32x16 mfma_split(const Split8& a, const Split8& b, f32x16 acc) {
  acc = mfma_b16(a.m, b.m, acc);
  acc = mfma_b16(a.l, b.h, acc);
  acc = mfma_b16(a.h, b.l, acc);
  acc = mfma_b16(a.m, b.h, acc);
  acc = mfma_b16(a.h, b.m, acc);
  return mfma_b16(a.h, b.h, acc);
}

// Waits until at most N of this wave's vector-memory loads are outstanding and its LDS reads
// have completed. The empty asm statements keep the compiler from moving accesses across.
template <int N>
__device__ __forceinline__ void wait_loads() {
  static_assert(N >= 0 && N < 64, "vmcnt holds 6 bits");
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
  asm volatile("" ::: "memory");
}
__device__ __forceinline__ void wait_lds_reads() {  // vmcnt 63: loads in flight may stay
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(15 | (3 << 14) | (7 << 4));
  asm volatile("" ::: "memory");
}

// One wave's view of 32-row tiles of D floats.
template <int D>
struct Tile32 {
  static constexpr int CPR = D / 4;            // 16-byte chunks per row
  static constexpr int RB = 4 * D;             // bytes per row
  static constexpr int NL = 32 * CPR / 64;     // 1 KB load instructions per tile
  int row0;    // row operand: byte offset of chunk h of row l % 32
  int col[4];  // column operand: offsets for rows 4 h + b (b = 0..3), column l % 32
  __device__ __forceinline__ explicit Tile32(int lane) {
    const int h = lane >> 5, r = lane & 31;
    row0 = r * RB + ((h ^ (r & (CPR - 1))) << 4);
#pragma unroll
    for (int b = 0; b < 4; ++b) col[b] = (4 * h + b) * RB + (((r >> 2) ^ (4 * h + b)) << 4) + 4 * (r & 3);
  }
  // floats 8 kk + 4 h .. + 3 of row l % 32
  __device__ __forceinline__ float4 row(const float* t, int kk) const {
    return *reinterpret_cast<const float4*>(reinterpret_cast<const char*>(t) + (row0 ^ (kk << 5)));
  }
  // element [8 (i / 4) + 4 h + i % 4][32 db + l % 32]
  __device__ __forceinline__ float at(const float* t, int i, int db) const {
    const int a = i >> 2, b = i & 3;
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(t) + col[b] + 8 * a * RB +
                                           128 * (db ^ (a & (CPR / 8 - 1))));
  }
  // rows r0 .. r0 + 31 of src [S, D] (rows past S read row S - 1) into the tile, straight to LDS
  static __device__ __forceinline__ void load(float* t, const float* src, int r0, int S, int lane) {
    const char* base = reinterpret_cast<const char*>(src + (int64_t)r0 * D);
    const int lim = S - 1 - r0;
#pragma unroll
    for (int j = 0; j < NL; ++j) {
      const int pos = j * 64 + lane, r = pos / CPR, c = (pos % CPR) ^ (r & (CPR - 1));
      const int rr = r < lim ? r : lim;
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(base + rr * RB + c * 16),
                                       (__attribute__((address_space(3))) void*)(t + j * 256), 16, 0, 0);
    }
  }
};

// A lane's row in registers, split: operand s holds columns 16 s + 4 h + 0..3 and 16 s + 8 + 4 h + 0..3.
template <int D>
__device__ __forceinline__ void load_row_regs(const float* src, int row, int h, Split8* out) {
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    const float4 x = *reinterpret_cast<const float4*>(src + (int64_t)row * D + 16 * s + 4 * h);
    const float4 y = *reinterpret_cast<const float4*>(src + (int64_t)row * D + 16 * s + 8 + 4 * h);
    const float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    out[s] = split8(f);
  }
}

// The same rows, split once by the workgroup into LDS: part x (h, m, l) of operand s, 16 bytes a lane.
template <int D>
struct SplitLds {
  static constexpr int WORDS = 3 * (D / 16) * 256;  // 24 KB at D = 128, 12 KB at D = 64
  const uint32_t* p;
  int lane;
  __device__ __forceinline__ bf16x8 part(int s, int x) const {
    return *reinterpret_cast<const bf16x8*>(p + ((3 * s + x) * 64 + lane) * 4);
  }
  __device__ __forceinline__ Split8 operator[](int s) const { return Split8{part(s, 0), part(s, 1), part(s, 2)}; }
};
template <int D, int NF>
__device__ __forceinline__ SplitLds<D> put_row_split(uint32_t* dst, const float* src, int row, int lane, int f) {
#pragma unroll
  for (int s = f; s < D / 16; s += NF) {
    const float* r = src + (int64_t)row * D + 16 * s + 4 * (lane >> 5);
    const float4 x = *reinterpret_cast<const float4*>(r), y = *reinterpret_cast<const float4*>(r + 8);
    const float v[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    const Split8 o = split8(v);
    uint32_t* d = dst + (3 * s * 64 + lane) * 4;
    *reinterpret_cast<bf16x8*>(d) = o.h;
    *reinterpret_cast<bf16x8*>(d + 256) = o.m;
    *reinterpret_cast<bf16x8*>(d + 512) = o.l;
  }
  return SplitLds<D>{dst, lane};
}

// With two waves per SIMD (D = 64) the other wave fills the gaps of a step, and each step is closed
// off so that fewer operands are live; at D = 128 the compiler orders a whole product (S = 1000, 2
// heads 34.7 us forward, with closed steps 36.2). Scheduling groups that interleave every step's
// split with its MFMAs are 1 to 2% faster forward at D = 128 but take minutes to compile.
template <int D>
__device__ __forceinline__ void close_step() {
  if constexpr (D == 64) __builtin_amdgcn_sched_barrier(0);
}

// acc += tile (rows = m) x regs^T (rows = n) over D. The reads and the split of the next 16 columns
// run under the MFMAs of the current ones.
template <int D, typename Regs>
__device__ __forceinline__ f32x16 rows_product(const Tile32<D>& tl, const float* t, const Regs& regs, f32x16 acc) {
  auto get = [&](int s) __attribute__((always_inline)) {
    const float4 x = tl.row(t, 2 * s), y = tl.row(t, 2 * s + 1);
    const float f[8] = {x.x, x.y, x.z, x.w, y.x, y.y, y.z, y.w};
    return split8(f);
  };
  Split8 cur = get(0), op = regs[0];
#pragma unroll
  for (int s = 0; s < D / 16; ++s) {
    Split8 nxt = cur, opn = op;
    if (s + 1 < D / 16) nxt = get(s + 1), opn = regs[s + 1];
    acc = mfma_split(cur, op, acc);
    close_step<D>();
    cur = nxt, op = opn;
  }
  return acc;
}

// acc[d] += product over the tile's 32 rows of its columns and x (element i: row 8 (i / 4) + 4 h +
// i % 4). XA: x is the row operand (rows of the result come from x), else the column operand.
template <int D, bool XA>
__device__ __forceinline__ void cols_product(const Tile32<D>& tl, const float* t, f32x16 x, f32x16* acc) {
  constexpr int ND = D / 32;
  auto get = [&](int u, int d) __attribute__((always_inline)) {
    float f[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = tl.at(t, 8 * u + j, d);
    return split8(f);
  };
  Split8 cur = get(0, 0);
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    float f[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) f[j] = x[8 * u + j];
    const Split8 xs = split8(f);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int d = 0; d < ND; ++d) {
      Split8 nxt = cur;
      if (d + 1 < ND) nxt = get(u, d + 1);
      else if (u == 0) nxt = get(1, 0);
      acc[d] = XA ? mfma_split(xs, cur, acc[d]) : mfma_split(cur, xs, acc[d]);
      close_step<D>();
      cur = nxt;
    }
  }
}

// Rows after a query are masked by P = 0 and dS = 0, which keeps finite values out but not an infinity or a
// NaN (0 x NaN): on the tile that holds the diagonal, one non-finite row would reach the rows before it.
// A wave therefore looks that tile over before its products: non-finite elements are cleared, and the
// results of cols_product that an unmasked one belongs to are made infinite beforehand. (The products
// over D need no mark: a row with a non-finite element has a non-finite lse or Delta.) XA = false: the tile
// holds keys, masked after the query r32; XA = true: queries, masked before the key. The backward does so in its
// tile loop (4000 rows, 8 heads of 64 368 -> 372 us, others within 0.3%). In the forward that cost 3 to 5%;
// there the wave looks its sums over at the end and forms them again where it has to.
template <int D>
__device__ __forceinline__ bool tile_finite(const Tile32<D>& tl, const float* t) {
  float c = 0.0f;
#pragma unroll 4
  for (int kk = 0; kk < D / 8; ++kk) {
    const float4 x = tl.row(t, kk);  // 0 times a non-finite value is NaN
    c = __builtin_fmaf(x.x, 0.0f, __builtin_fmaf(x.y, 0.0f, __builtin_fmaf(x.z, 0.0f, __builtin_fmaf(x.w, 0.0f, c))));
  }
  return __builtin_amdgcn_ballot_w64(c != 0.0f) == 0;
}
template <int D>
__device__ __forceinline__ bool sums_finite(const f32x16* acc) {
  float c = 0.0f;
#pragma unroll
  for (int d = 0; d < D / 32; ++d)
#pragma unroll
    for (int i = 0; i < 16; ++i) c = __builtin_fmaf(acc[d][i], 0.0f, c);
  return __builtin_amdgcn_ballot_w64(c != 0.0f) == 0;
}
// Non-finite elements of the tile to 0; edge[c]: the first (XA: last) row with one in column 64 c + lane.
template <int D, bool XA>
__device__ __forceinline__ void clear_nonfinite(float* t, int lane, int* edge) {
#pragma unroll
  for (int c = 0; c < D / 64; ++c) {
    const int col = 64 * c + lane;
    edge[c] = XA ? -1 : 32;
#pragma unroll 1
    for (int k = 0; k < 32; ++k) {
      float* x = t + k * D + (((col >> 2) ^ (k & (D / 4 - 1))) << 2) + (col & 3);
      if (__builtin_isfinite(*x)) continue;
      *x = 0.0f;
      if (XA || edge[c] == 32) edge[c] = k;
    }
  }
}
// acc += 2^127 x 2^127 where the first (XA: last) cleared row of the column is unmasked, else 0 exactly.
template <int D, bool XA>
__device__ __forceinline__ void mark_nonfinite(const int* edge, int h, int r32, f32x16* acc) {
#pragma unroll
  for (int d = 0; d < D / 32; ++d) {
    const int e = __shfl(edge[d >> 1], 32 * (d & 1) + r32, 64);
#pragma unroll 1  // (unrolled, the comparisons are kept in registers across the tile loop)
    for (int u = 0; u < 2; ++u) {
      u16x8 bad, in;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int k = 8 * (2 * u + (j >> 2)) + 4 * h + (j & 3);
        bad[j] = k == e ? 0x7f00 : 0;
        in[j] = (XA ? k >= r32 : k <= r32) ? 0x7f00 : 0;
      }
      const bf16x8 x = __builtin_bit_cast(bf16x8, in), y = __builtin_bit_cast(bf16x8, bad);
      acc[d] = XA ? mfma_b16(x, y, acc[d]) : mfma_b16(y, x, acc[d]);
    }
  }
}
template <int D, bool XA>
__device__ __forceinline__ void contain(const Tile32<D>& tl, float* t, int lane, f32x16* acc) {
  if (tile_finite<D>(tl, t)) return;
  int edge[D / 64];
  clear_nonfinite<D, XA>(t, lane, edge);
  mark_nonfinite<D, XA>(edge, lane >> 5, lane & 31, acc);
}

// A wave's accumulators to LDS: unit u = 4 d + g holds elements 4 g .. 4 g + 3 of acc[d].
template <int D>
__device__ __forceinline__ void put_acc(float* dst, const f32x16* acc, int lane) {
#pragma unroll
  for (int d = 0; d < D / 32; ++d)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<float4*>(dst + ((4 * d + g) * 64 + lane) * 4) =
          make_float4(acc[d][4 * g], acc[d][4 * g + 1], acc[d][4 * g + 2], acc[d][4 * g + 3]);
}
__device__ __forceinline__ float4 get_unit(const float* src, int u, int lane) {
  return *reinterpret_cast<const float4*>(src + (u * 64 + lane) * 4);
}

// Workgroups in linear-id order take the longest blocks of every head first, and with a head
// count that is a multiple of 8 every block of a head lands on one XCD.
struct F32Pos {
  int rank;
  int64_t head;
};
__device__ __forceinline__ F32Pos f32_pos(int64_t lin, int64_t heads) { return F32Pos{(int)(lin / heads), lin % heads}; }

// ------------------------------------------------------------------ forward
template <int D, int NF>
__global__ void __launch_bounds__(64 * NF, D == 64 ? 2 : 1)
sdpa_fwd_f32(const float* __restrict__ Q, const float* __restrict__ K, const float* __restrict__ V,
             float* __restrict__ O, float* __restrict__ LSE, int S, float scale, int Hq, int Hs, int Gq) {
  using T = Tile32<D>;
  __shared__ __align__(16) float Kt[NF][32 * D], Vt[NF][32 * D];
  __shared__ float ms[NF][32], ls[NF][32];
  const int lane = threadIdx.x & 63, f = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = lane >> 5, r32 = lane & 31;
  const int nblk = (S + 31) / 32;
  const int64_t heads = (int64_t)gridDim.x / nblk;
  const F32Pos pos = f32_pos(blockIdx.x, heads);
  const int64_t bh = pos.head;
  const int qb = nblk - 1 - pos.rank, q0 = 32 * qb, myq = q0 + r32;
  const int64_t kvh = (bh / Hq) * Hs + (bh % Hq) / Gq;  // selection head: rows of ks, vs
  const float* Kh = K + kvh * S * D;
  const float* Vh = V + kvh * S * D;
  const float sl2 = scale * kLog2eF;
  float* kt = Kt[f];
  float* vt = Vt[f];
  const T tl(lane);
  f32x16 o[D / 32];
  float m, l;
  const int nt = qb + 1;  // key tiles 0 .. qb; only the last is masked
  auto pass = [&](auto again) __attribute__((always_inline)) {
    // (of a pass: its registers, kept for a second one, would be copied aside first: 1 us at D = 128)
    Split8 q[D / 16];
    load_row_regs<D>(Q + bh * S * D, myq < S ? myq : S - 1, h, q);
#pragma unroll
    for (int d = 0; d < D / 32; ++d) o[d] = f32x16{};
    // the running maximum of the unscaled logits starts at the lowest finite value: a masked logit
    // (-inf) of a row without any key yet then has weight exp2(-inf) = 0
    m = -FLT_MAX, l = 0.0f;
    if (f < nt) {
      T::load(kt, Kh, 32 * f, S, lane);
      T::load(vt, Vh, 32 * f, S, lane);
    }
    for (int t = f; t < nt; t += NF) {
      const int tn = t + NF < nt ? t + NF : t;  // the last tile is loaded once more, unused
      if (decltype(again)::value && t == nt - 1) {
        wait_loads<0>();
        contain<D, false>(tl, vt, lane, o);
      }
      wait_loads<T::NL>();  // the K tile has landed
      f32x16 s = rows_product<D>(tl, kt, q, f32x16{});
      wait_lds_reads();
      T::load(kt, Kh, 32 * tn, S, lane);
      if (t == nt - 1) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (32 * t + 8 * (i >> 2) + 4 * h + (i & 3) > myq) s[i] = -INFINITY;
      }
      float mx = s[0];
#pragma unroll
      for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
      mx = fmaxf(mx, __shfl_xor(mx, 32, 64));
      if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {
        const float mn = fmaxf(m, mx), al = __builtin_amdgcn_exp2f((m - mn) * sl2);
        l *= al;
#pragma unroll
        for (int d = 0; d < D / 32; ++d)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[d][i] *= al;
        m = mn;
      }
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = __builtin_amdgcn_exp2f((s[i] - m) * sl2);
      float sum = 0.0f;
#pragma unroll
      for (int i = 0; i < 16; ++i) sum += s[i];
      l += sum;
      wait_loads<T::NL>();  // the V tile has landed
      cols_product<D, false>(tl, vt, s, o);
      wait_lds_reads();
      T::load(vt, Vh, 32 * tn, S, lane);
    }
    wait_loads<0>();
  };
  pass(std::false_type{});
  // the wave of the masked tile forms its sums once more, with that tile contained, where they hold
  // what is not finite
  if (__builtin_expect(f == (nt - 1) % NF && !sums_finite<D>(o), 0)) pass(std::true_type{});
  l += __shfl_xor(l, 32, 64);
  put_acc<D>(kt, o, lane);
  if (h == 0) ms[f][r32] = m, ls[f][r32] = l;
  __syncthreads();
  float M = ms[0][r32], lt = 0.0f, w[NF];
#pragma unroll
  for (int x = 1; x < NF; ++x) M = fmaxf(M, ms[x][r32]);
#pragma unroll
  for (int x = 0; x < NF; ++x) {
    w[x] = __builtin_amdgcn_exp2f((ms[x][r32] - M) * sl2);  // 0 for a wave without a key of the row
    lt += w[x] * ls[x][r32];
  }
  if (myq >= S) return;
  constexpr int NU = D / 8 / NF;  // units of the output per wave
  const float inv = 1.0f / lt;
#pragma unroll
  for (int y = 0; y < NU; ++y) {
    const int u = f * NU + y;
    float4 a = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int x = 0; x < NF; ++x) {
      const float4 b = get_unit(Kt[x], u, lane);
      a.x += w[x] * b.x, a.y += w[x] * b.y, a.z += w[x] * b.z, a.w += w[x] * b.w;
    }
    *reinterpret_cast<float4*>(O + (bh * S + myq) * D + 8 * u + 4 * h) =
        make_float4(a.x * inv, a.y * inv, a.z * inv, a.w * inv);
  }
  if (f == 0 && h == 0) LSE[bh * S + myq] = M * scale + logf(lt);
}

// ------------------------------------------------------------------ backward
struct BwdF32 {
  const float *q, *k, *v, *go, *lse, *delta;
  float *dq, *dk, *dv;
  int64_t kblocks;  // dK/dV workgroups (the first of the launch); the rest are dQ workgroups
  int64_t kheads, qheads;
  int S, Hq, Hs, Gq;
  float scale;
};

// dQ of 32 query rows: dP^T = V dO^T (the chain starts from -Delta), S^T = K Q^T,
// dQ^T += K^T dS^T.
template <int D, int NF>
__device__ __forceinline__ void dq_block(const BwdF32& a, int64_t lin, float (*At)[32 * D], float (*Bt)[32 * D],
                                         uint32_t* sp, int lane, int f) {
  using T = Tile32<D>;
  const int h = lane >> 5, r32 = lane & 31, S = a.S;
  const int nblk = (S + 31) / 32;
  const F32Pos pos = f32_pos(lin, a.qheads);
  const int64_t bh = pos.head;
  const int qb = nblk - 1 - pos.rank, myq = 32 * qb + r32;
  const int64_t kvh = (bh / a.Hq) * a.Hs + (bh % a.Hq) / a.Gq;
  const float* Kh = a.k + kvh * S * D;
  const float* Vh = a.v + kvh * S * D;
  float* kt = At[f];
  float* vt = Bt[f];
  const T tl(lane);
  const int row = myq < S ? myq : S - 1;
  Split8 q[D / 16];
  load_row_regs<D>(a.q + bh * S * D, row, h, q);
  const SplitLds<D> go = put_row_split<D, NF>(sp, a.go + bh * S * D, row, lane, f);
  __syncthreads();
  const float lse = a.lse[bh * S + row], ndl = -a.delta[bh * S + row];
  f32x16 dq[D / 32];
#pragma unroll
  for (int d = 0; d < D / 32; ++d) dq[d] = f32x16{};
  const int nt = qb + 1;
  if (f < nt) {
    T::load(vt, Vh, 32 * f, S, lane);
    T::load(kt, Kh, 32 * f, S, lane);
  }
  for (int t = f; t < nt; t += NF) {
    const int tn = t + NF < nt ? t + NF : t;
    wait_loads<T::NL>();  // V
    f32x16 dp;
#pragma unroll
    for (int i = 0; i < 16; ++i) dp[i] = ndl;
    dp = rows_product<D>(tl, vt, go, dp);
    wait_lds_reads();
    T::load(vt, Vh, 32 * tn, S, lane);
    wait_loads<T::NL>();  // K
    if (t == nt - 1) contain<D, false>(tl, kt, lane, dq);
    f32x16 s = rows_product<D>(tl, kt, q, f32x16{});
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.scale, -lse) * kLog2eF);
      s[i] = t == nt - 1 && 32 * t + 8 * (i >> 2) + 4 * h + (i & 3) > myq ? 0.0f : p * dp[i];
    }
    cols_product<D, false>(tl, kt, s, dq);
    wait_lds_reads();
    T::load(kt, Kh, 32 * tn, S, lane);
  }
  wait_loads<0>();
  put_acc<D>(kt, dq, lane);
  __syncthreads();
  if (myq >= S) return;
  constexpr int NU = D / 8 / NF;
#pragma unroll
  for (int y = 0; y < NU; ++y) {
    const int u = f * NU + y;
    float4 x = get_unit(At[0], u, lane);
#pragma unroll
    for (int w = 1; w < NF; ++w) {
      const float4 b = get_unit(At[w], u, lane);
      x.x += b.x, x.y += b.y, x.z += b.z, x.w += b.w;
    }
    *reinterpret_cast<float4*>(a.dq + (bh * S + myq) * D + 8 * u + 4 * h) =
        make_float4(x.x * a.scale, x.y * a.scale, x.z * a.scale, x.w * a.scale);
  }
}

// dK, dV of 32 keys of a selection head, summed over its Gq query heads: dP = dO V^T (from
// -Delta), S = Q K^T, dV += P^T dO, dK += dS^T Q. A wave's tiles run over (head, query tile).
template <int D, int NF>
__device__ __forceinline__ void dkdv_block(const BwdF32& a, int64_t lin, float (*At)[32 * D], float (*Bt)[32 * D],
                                           float (*st)[64], uint32_t* sp, int lane, int f) {
  using T = Tile32<D>;
  const int h = lane >> 5, r32 = lane & 31, S = a.S;
  const F32Pos pos = f32_pos(lin, a.kheads);
  const int64_t bs = pos.head;
  const int kb = pos.rank, mykey = 32 * kb + r32;  // early keys meet the most queries: first
  const int64_t bh0 = (bs / a.Hs) * a.Hq + (bs % a.Hs) * a.Gq;
  float* qt = At[f];
  float* gt = Bt[f];
  float* stat = st[f];  // lse of the tile's rows, then -Delta
  const T tl(lane);
  const int row = mykey < S ? mykey : S - 1;
  Split8 k[D / 16];
  load_row_regs<D>(a.k + bs * S * D, row, h, k);
  const SplitLds<D> v = put_row_split<D, NF>(sp, a.v + bs * S * D, row, lane, f);
  __syncthreads();
  f32x16 dk[D / 32], dv[D / 32];
#pragma unroll
  for (int d = 0; d < D / 32; ++d) dk[d] = dv[d] = f32x16{};
  const int ntq = (S + 31) / 32 - kb;  // query tiles kb .. of one head; only the first is masked
  const int nt = ntq * a.Gq;
  float sx = 0.0f;  // lane l < 32: lse of row l of the next tile; l >= 32: Delta of row l - 32
  auto head_of = [&](int t) __attribute__((always_inline)) { return bh0 + t / ntq; };
  auto row_of = [&](int t) __attribute__((always_inline)) { return 32 * (kb + t % ntq); };
  auto load_go = [&](int t) __attribute__((always_inline)) {
    const int64_t b = head_of(t);
    const int r0 = row_of(t);
    T::load(gt, a.go + b * S * D, r0, S, lane);
    const int r = r0 + r32;
    sx = (h ? a.delta : a.lse)[b * S + (r < S ? r : S - 1)];
  };
  auto load_q = [&](int t) __attribute__((always_inline)) {
    T::load(qt, a.q + head_of(t) * S * D, row_of(t), S, lane);
  };
  if (f < nt) {
    load_go(f);
    load_q(f);
  }
  for (int t = f; t < nt; t += NF) {
    const int tn = t + NF < nt ? t + NF : t;
    const bool diag = t % ntq == 0;
    wait_loads<T::NL>();  // dO (and lse, Delta)
    if (diag) contain<D, true>(tl, gt, lane, dv);
    const bool in = row_of(t) + r32 < S;  // rows past S: P = 0
    stat[lane] = h ? (in ? -sx : 0.0f) : (in ? sx : INFINITY);
    f32x16 dp;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 d4 = *reinterpret_cast<const float4*>(stat + 32 + 8 * g + 4 * h);
      dp[4 * g] = d4.x, dp[4 * g + 1] = d4.y, dp[4 * g + 2] = d4.z, dp[4 * g + 3] = d4.w;
    }
    dp = rows_product<D>(tl, gt, v, dp);
    wait_loads<0>();  // Q
    if (diag) contain<D, true>(tl, qt, lane, dk);
    f32x16 s = rows_product<D>(tl, qt, k, f32x16{});
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const float4 l4 = *reinterpret_cast<const float4*>(stat + 8 * g + 4 * h);
      const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int i = 4 * g + j;
        const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[i], a.scale, -lv[j]) * kLog2eF);
        const bool masked = diag && 8 * g + 4 * h + j < r32;
        s[i] = masked ? 0.0f : p;
        dp[i] = masked ? 0.0f : p * dp[i];
      }
    }
    cols_product<D, true>(tl, gt, s, dv);
    wait_lds_reads();
    load_go(tn);
    cols_product<D, true>(tl, qt, dp, dk);
    wait_lds_reads();
    load_q(tn);
  }
  wait_loads<0>();
  put_acc<D>(qt, dk, lane);
  put_acc<D>(gt, dv, lane);
  __syncthreads();
  constexpr int NU = D / 8 / NF;
#pragma unroll
  for (int y = 0; y < NU; ++y) {
    const int u = f * NU + y;
    float4 x = get_unit(At[0], u, lane), z = get_unit(Bt[0], u, lane);
#pragma unroll
    for (int w = 1; w < NF; ++w) {
      const float4 b = get_unit(At[w], u, lane), c = get_unit(Bt[w], u, lane);
      x.x += b.x, x.y += b.y, x.z += b.z, x.w += b.w;
      z.x += c.x, z.y += c.y, z.z += c.z, z.w += c.w;
    }
    const float xs[4] = {x.x, x.y, x.z, x.w}, zs[4] = {z.x, z.y, z.z, z.w};
#pragma unroll
    for (int j = 0; j < 4; ++j) {  // C layout: key row 8 g + 4 h + j, column 32 d + l % 32
      const int key = 32 * kb + 8 * (u & 3) + 4 * h + j;
      if (key < S) {
        a.dk[(bs * S + key) * D + 32 * (u >> 2) + r32] = xs[j] * a.scale;
        a.dv[(bs * S + key) * D + 32 * (u >> 2) + r32] = zs[j];
      }
    }
  }
}

template <int D, int NF>
__global__ void __launch_bounds__(64 * NF, D == 64 ? 2 : 1) sdpa_bwd_f32(BwdF32 a) {
  __shared__ __align__(16) float At[NF][32 * D], Bt[NF][32 * D];
  __shared__ __align__(16) float st[NF][64];
  __shared__ __align__(16) uint32_t sp[SplitLds<D>::WORDS];
  const int lane = threadIdx.x & 63, f = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t lin = blockIdx.x;
  if (lin < a.kblocks) dkdv_block<D, NF>(a, lin, At, Bt, st, sp, lane, f);
  else dq_block<D, NF>(a, lin - a.kblocks, At, Bt, sp, lane, f);
}

}  // namespace lh

using namespace lh;

// Waves per workgroup at D = 64 (at D = 128 4, with 128 KB of tiles): 8 (the same 128 KB, one
// workgroup per CU) where the row blocks leave CUs idle, else 4 (64 KB, two per CU). Forward, 8 and 4
// waves: 284 blocks (S = 2257, 4 heads) 34.7 and 41.0 us, 497 43.1 and 46.4, 528 54.4 and 57.1, 568
// 52.2 and 50.8, 1000 133 and 124. Backward, over the blocks of dK/dV and dQ: 456 53.3 and 72.4, 568
// 82.3 and 96.7, 710 99.5 and 95.0, 1136 150 and 144.
static bool eight_waves_fwd(int64_t blocks) { return blocks <= 544; }
static bool eight_waves_bwd(int64_t blocks) { return blocks <= 640; }

hipError_t lh_launch_sdpa_fwd_f32(const LhShape& s, const void* qs, const void* ks, const void* vs, void* os,
                                  float* lse, hipStream_t st) {
  const int64_t blocks = (s.S + 31) / 32 * s.B * s.Hq;
  const dim3 grid((unsigned)blocks);
  auto q = (const float*)qs, k = (const float*)ks, v = (const float*)vs;
  if (s.D == 128)
    hipLaunchKernelGGL((sdpa_fwd_f32<128, 4>), grid, dim3(256), 0, st, q, k, v, (float*)os, lse, (int)s.S, s.scale,
                       s.Hq, s.Hs, s.Gq);
  else if (eight_waves_fwd(blocks))
    hipLaunchKernelGGL((sdpa_fwd_f32<64, 8>), grid, dim3(512), 0, st, q, k, v, (float*)os, lse, (int)s.S, s.scale,
                       s.Hq, s.Hs, s.Gq);
  else
    hipLaunchKernelGGL((sdpa_fwd_f32<64, 4>), grid, dim3(256), 0, st, q, k, v, (float*)os, lse, (int)s.S, s.scale,
                       s.Hq, s.Hs, s.Gq);
  return hipGetLastError();
}

hipError_t lh_launch_sdpa_bwd_f32(const LhShape& s, const void* qs, const void* ks, const void* vs, const void* dos,
                                  const float* lse, const float* delta, void* dqs, void* dks, void* dvs,
                                  hipStream_t st) {
  const int64_t nblk = (s.S + 31) / 32;
  BwdF32 a{(const float*)qs, (const float*)ks, (const float*)vs, (const float*)dos, lse, delta,
           (float*)dqs, (float*)dks, (float*)dvs, nblk * s.B * s.Hs, s.B * s.Hs, s.B * s.Hq,
           (int)s.S, s.Hq, s.Hs, s.Gq, s.scale};
  const int64_t blocks = nblk * (s.B * s.Hs + s.B * s.Hq);
  const dim3 grid((unsigned)blocks);
  if (s.D == 128) hipLaunchKernelGGL((sdpa_bwd_f32<128, 4>), grid, dim3(256), 0, st, a);
  else if (eight_waves_bwd(blocks)) hipLaunchKernelGGL((sdpa_bwd_f32<64, 8>), grid, dim3(512), 0, st, a);
  else hipLaunchKernelGGL((sdpa_bwd_f32<64, 4>), grid, dim3(256), 0, st, a);
  return hipGetLastError();
}
