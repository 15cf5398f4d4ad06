// k_pool_score.hip -- pyramid pooling (Sec. 3.3, Eq. pool) and norm scores (Sec. 3.4,
// Eqs. score-base and score-pool) in one streaming pass over Q, K and V.
//
// One launch covers the three tensors: the head slots of Q (Hq), K (Hkv) and V (Hkv) form one
// list, and a workgroup owns a range of base rows for a chunk of that list. The range is a
// multiple of p^(L-1), so every pyramid window lies inside it. Every window's sum is formed in
// fp64 in the order of its rows (its p children in order); the mean is rounded once to the storage
// dtype. Sums of bf16 (or fp32) values in fp64 are exact for the data this path sees, so the
// stored mean is the correctly rounded exact mean.
//
// Scores (Q and K only): rows are staged through LDS so that one thread computes one row's
// squared norm sequentially (c ascending, fp64; 16-byte LDS reads), takes the correctly rounded
// fp64 sqrt and rounds to fp32. The level-0 scores are then max-pooled up the levels.
//
// Two kernels: pool_leaf_kernel (p = 2, 3, 4) spreads the rows of a range over row groups;
// pool_score_kernel walks them. The rule between them is at the launch.
#include "lh_common.h"

namespace lh {

constexpr int kPoolRB = 8;  // rows staged per step
constexpr size_t kMaxLds = 160 * 1024;
constexpr int kLeafThreads = 256;  // threads per workgroup, unless p^(L-1) rows need more

struct PoolTensor {
  const void* x;  // [B, N, H, D]
  void* pyr;      // [B, R, H, D] or null
  float* s;       // [B, H, Ptot] or null
  int32_t H;
};

struct PoolArgs {
  PoolTensor t[3];
  int32_t slot1, slot2, nslots;  // head slots: [0, slot1) tensor 0, [slot1, slot2) tensor 1, rest 2
  int64_t N, R, Ptot;
  int32_t D, HW, WR, p, cpr_shift;
  int32_t epb[16];  // WR / p^l: level-l windows per workgroup
  int64_t off[17];
  double inv[16];  // 1 / p^l (exact when p is a power of two)
  double pwd[16];  // p^l
  int32_t pow2;
};

// acc / w, correctly rounded, for w = p^l with inv = RN(1 / w). For p a power of two the product
// is exact. Otherwise the quotient estimate is corrected by its exact remainder, which gives the
// correctly rounded quotient because inv is correctly rounded (Markstein's division theorem): 3
// fp64 operations where the compiler's division takes about 12.
__device__ __forceinline__ double quotient(double acc, double inv, double w, bool pow2) {
  const double q = acc * inv;
  if (pow2) return q;
  const double r = __builtin_fma(-q, w, acc);
  const double c = __builtin_fma(r, inv, q);
  return r == r ? c : q;  // an infinite sum stays infinite
}

template <typename T>
__device__ __forceinline__ void store_mean(T* dst, const double* acc, double inv, double w, bool pow2) {
  constexpr int CH = 16 / sizeof(T);
  if constexpr (sizeof(T) == 2) {
    uint32_t wd[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const double lo = quotient(acc[2 * c], inv, w, pow2);
      const double hi = quotient(acc[2 * c + 1], inv, w, pow2);
      wd[c] = (uint32_t)f64_to_bf16(lo) | ((uint32_t)f64_to_bf16(hi) << 16);
    }
    u32x4 o;
    o.x = wd[0], o.y = wd[1], o.z = wd[2], o.w = wd[3];
    store16_nt(dst, o);
  } else {
    float o[CH];
#pragma unroll
    for (int c = 0; c < CH; ++c) o[c] = (float)quotient(acc[c], inv, w, pow2);
    store_chunk_f32(reinterpret_cast<float*>(dst), o);
  }
}

// fp32 norm of an LDS row: 16-byte reads, squares (exact in fp64) summed in ascending order.
// AHEAD: four reads in flight at a time. For the walk, where a norm is on the chain of every step: pooling and
// scores of 21,504 rows, 1 head of 128, fp32, p = 8, L = 4 239 -> 184 us.
template <typename T, bool AHEAD>
__device__ __forceinline__ float row_norm(const T* row, int D) {
  constexpr int CH = 16 / sizeof(T);
  double s2 = 0.0;
  auto add = [&](int c) __attribute__((always_inline)) {
    const u32x4 w4 = *reinterpret_cast<const u32x4*>(row + c);
    const uint32_t u[4] = {w4.x, w4.y, w4.z, w4.w};
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if constexpr (sizeof(T) == 2) {
        const double lo = (double)__uint_as_float(u[e] << 16);
        const double hi = (double)__uint_as_float(u[e] & 0xffff0000u);
        s2 += lo * lo;
        s2 += hi * hi;
      } else {
        const double x = (double)__uint_as_float(u[e]);
        s2 += x * x;
      }
    }
  };
  if constexpr (AHEAD) {
#pragma unroll 4
    for (int c = 0; c < D; c += CH) add(c);
  } else {
    for (int c = 0; c < D; c += CH) add(c);
  }
  return (float)sqrt(s2);
}

template <typename T>
__device__ __forceinline__ void add_row(double* acc, const u32x4& w) {
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
  if constexpr (sizeof(T) == 2) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      acc[2 * i] += (double)__uint_as_float(u[i] << 16);
      acc[2 * i + 1] += (double)__uint_as_float(u[i] & 0xffff0000u);
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i] += (double)__uint_as_float(u[i]);
  }
}

// Max-pool cascade of nrc level-0 scores (rows in order) of head slot g2 of the block: the
// level-l window that a score completes is written, and its max carried one level up. The
// running state (mx, scnt, sent) carries over between calls.
template <int L, int LA>
__device__ __forceinline__ void cascade_rows(const PoolArgs& a, const float* nrm, int nrc, int col, int g2,
                                             int64_t b, float (&mx)[LA], int (&scnt)[LA + 1], int (&sent)[LA]) {
  const int t2i = g2 < a.slot1 ? 0 : g2 < a.slot2 ? 1 : 2;
  float* sb = a.t[t2i].s;
  if (!sb) return;
  const int h2 = g2 - (t2i == 0 ? 0 : t2i == 1 ? a.slot1 : a.slot2);
  float* srow = sb + (b * a.t[t2i].H + h2) * a.Ptot;
  for (int r = 0; r < nrc; ++r) {
    const float s0 = nrm[r * a.HW + col];
    mx[1] = mx[1] > s0 ? mx[1] : s0;
    ++scnt[1];
#pragma unroll
    for (int l = 1; l < L; ++l) {
      if (scnt[l] != a.p) break;
      scnt[l] = 0;
      srow[a.off[l] + (int64_t)blockIdx.x * a.epb[l] + sent[l]] = mx[l];
      ++sent[l];
      if (l + 1 < L) {
        const int ln = l + 1 < L ? l + 1 : l;
        mx[ln] = mx[ln] > mx[l] ? mx[ln] : mx[l];
        ++scnt[ln];
      }
      mx[l] = 0.0f;
    }
  }
}

// The walk: each thread owns one 16-byte column chunk of one head and walks the rows of the range in
// order, in steps of 8, with an fp64 running sum per level. When a level-l window closes, its mean
// is written and its sum added into the level-(l+1) sum. Window closings are tracked with
// per-level counters, which are the same for the whole workgroup, so no per-row division is
// needed. One thread per head slot (the block's last threads) max-pools the level-0 scores up the
// levels, one step behind: a step's cascade runs while the next step's norms are computed (two
// LDS score buffers).
// PF > 0: p == PF is known at compile time and kPoolRB is a multiple of it, so level-1
// windows close at fixed positions of every step. PF == 0: any p, checked row by row.
template <typename T, int L, int PF>
__global__ void __launch_bounds__(256) pool_score_kernel(PoolArgs a) {
  constexpr int CH = 16 / sizeof(T);
  constexpr int LA = L > 1 ? L : 2;
  static_assert(PF == 0 || kPoolRB % PF == 0, "steps must hold whole level-1 windows");
  extern __shared__ __align__(16) unsigned char smem[];
  const int D = a.D;
  const int tid = threadIdx.x;
  const int hs = tid >> a.cpr_shift, cc = tid & ((1 << a.cpr_shift) - 1);
  const int gs = blockIdx.y * a.HW + hs;  // global head slot
  const bool active = gs < a.nslots;
  const int ti = gs < a.slot1 ? 0 : gs < a.slot2 ? 1 : 2;
  const int h = gs - (ti == 0 ? 0 : ti == 1 ? a.slot1 : a.slot2);
  const PoolTensor& t0 = a.t[0];
  const PoolTensor& t1 = a.t[1];
  const PoolTensor& t2 = a.t[2];
  const T* x = reinterpret_cast<const T*>(ti == 0 ? t0.x : ti == 1 ? t1.x : t2.x);
  T* pyr = reinterpret_cast<T*>(ti == 0 ? t0.pyr : ti == 1 ? t1.pyr : t2.pyr);
  float* srow_base = ti == 0 ? t0.s : ti == 1 ? t1.s : t2.s;
  const int H = ti == 0 ? t0.H : ti == 1 ? t1.H : t2.H;
  const int64_t b = blockIdx.z;
  const int64_t j0 = (int64_t)blockIdx.x * a.WR;
  const int nrows = (int)((a.N - j0) < a.WR ? (a.N - j0) : a.WR);
  const bool do_pool = L > 1 && active && pyr != nullptr;
  const bool any_score = a.t[0].s != nullptr || a.t[1].s != nullptr || a.t[2].s != nullptr;

  // LDS: staged rows [RB][HW][D + pad] of T, then two buffers of level-0 scores [RB][HW].
  // rows padded by 16 bytes: 16-byte aligned, and the norm threads (one row each, consecutive
  // rows) read 16-byte chunks without bank conflicts
  const int rowT = D + 16 / (int)sizeof(T);
  T* tile = reinterpret_cast<T*>(smem);
  float* nrm_buf = reinterpret_cast<float*>(smem + (size_t)kPoolRB * a.HW * rowT * sizeof(T));
  // the cascade threads: the block's last HW threads, one per head slot
  const int ct = tid - ((int)blockDim.x - a.HW);
  const bool cthread = L > 1 && ct >= 0 && (int)blockIdx.y * a.HW + ct < a.nslots;
  int step = 0, nr_prev = 0;

  const T* xrow = x + ((b * a.N + j0) * H + h) * D + cc * CH;
  const int64_t xstride = (int64_t)H * D;
  T* prow[LA];
#pragma unroll
  for (int l = 1; l < L; ++l)
    prow[l] = pyr ? pyr + ((b * a.R + (a.off[l] - a.N) + (int64_t)blockIdx.x * a.epb[l]) * H + h) * D + cc * CH
                  : nullptr;
  const int64_t pstride = (int64_t)H * D;

  double acc[LA][CH];
#pragma unroll
  for (int l = 0; l < LA; ++l)
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[l][c] = 0.0;
  int cnt[LA + 1];  // rows (level 1) or closed windows (level l > 1) in the open level-l window
#pragma unroll
  for (int l = 0; l <= LA; ++l) cnt[l] = 0;
  // cascade state (used by the cascade threads)
  float mx[LA];
#pragma unroll
  for (int l = 0; l < LA; ++l) mx[l] = 0.0f;
  int scnt[LA + 1];
#pragma unroll
  for (int l = 0; l <= LA; ++l) scnt[l] = 0;
  int sent[LA];  // next entry index (within the workgroup) per level, for the scores
#pragma unroll
  for (int l = 0; l < LA; ++l) sent[l] = 0;

  // closes the level-1 window that just received its last row, and every window above it
  // that closes with it
  auto close_windows = [&]() {
#pragma unroll
    for (int l = 1; l < L; ++l) {
      if (l > 1 && cnt[l] != a.p) break;
      cnt[l] = 0;
      if (do_pool) {
        store_mean<T>(prow[l], acc[l], a.inv[l], a.pwd[l], a.pow2);
        prow[l] += pstride;
      }
      if (l + 1 < L) {
#pragma unroll
        for (int c = 0; c < CH; ++c) acc[l + 1 < L ? l + 1 : l][c] += acc[l][c];
        ++cnt[l + 1];
      }
#pragma unroll
      for (int c = 0; c < CH; ++c) acc[l][c] = 0.0;
    }
  };

  for (int rb = 0; rb < nrows; rb += kPoolRB) {
    const int nr = nrows - rb < kPoolRB ? nrows - rb : kPoolRB;
    // raw 16-byte chunks: converted to fp64 as they are summed (fewer live registers)
    u32x4 v[kPoolRB];
#pragma unroll
    for (int r = 0; r < kPoolRB; ++r) {
      if (r < nr && active) v[r] = load16_nt(xrow + (int64_t)(rb + r) * xstride);
      else v[r] = u32x4{0, 0, 0, 0};
    }
    if (any_score && active && srow_base) {
#pragma unroll
      for (int r = 0; r < kPoolRB; ++r)
        if (r < nr) *reinterpret_cast<u32x4*>(tile + ((size_t)r * a.HW + hs) * rowT + cc * CH) = v[r];
    }
    if (L > 1) {
      if constexpr (PF > 0) {
        // nr is a multiple of p here (rows per workgroup are a multiple of p^(L-1))
#pragma unroll
        for (int r = 0; r < kPoolRB; ++r) {
          if (r >= nr) break;
          add_row<T>(acc[1], v[r]);
          if (r % PF == PF - 1) close_windows();
        }
      } else {
#pragma unroll
        for (int r = 0; r < kPoolRB; ++r) {
          if (r >= nr) break;
          add_row<T>(acc[1], v[r]);
          if (++cnt[1] == a.p) close_windows();
        }
      }
    }
    if (any_score) {
      float* nrm = nrm_buf + (step & 1) * kPoolRB * a.HW;
      __syncthreads();
      // the previous step's cascade runs on the last threads while the first ones compute
      // this step's norms
      if (step > 0 && cthread)
        cascade_rows<L, LA>(a, nrm_buf + ((step - 1) & 1) * kPoolRB * a.HW, nr_prev, ct,
                            (int)blockIdx.y * a.HW + ct, b, mx, scnt, sent);
      // one thread per (row, head slot): sequential fp64 sum of squares, c ascending
      for (int e = tid; e < nr * a.HW; e += blockDim.x) {
        const int r = e / a.HW, hh = e - r * a.HW;
        const int g2 = blockIdx.y * a.HW + hh;
        if (g2 >= a.nslots) continue;
        const int t2i = g2 < a.slot1 ? 0 : g2 < a.slot2 ? 1 : 2;
        float* sb = t2i == 0 ? t0.s : t2i == 1 ? t1.s : t2.s;
        if (!sb) continue;
        const int h2 = g2 - (t2i == 0 ? 0 : t2i == 1 ? a.slot1 : a.slot2);
        const int H2 = t2i == 0 ? t0.H : t2i == 1 ? t1.H : t2.H;
        const float sc = row_norm<T, true>(tile + ((size_t)r * a.HW + hh) * rowT, D);
        nrm[r * a.HW + hh] = sc;
        sb[(b * H2 + h2) * a.Ptot + j0 + rb + r] = sc;
      }
      // this step's scores are complete and the previous cascade is done; `tile` may be
      // rewritten, and the next step's cascade reads this step's score buffer
      __syncthreads();
      nr_prev = nr;
    }
    ++step;
  }
  if (any_score && step > 0 && cthread)
    cascade_rows<L, LA>(a, nrm_buf + ((step - 1) & 1) * kPoolRB * a.HW, nr_prev, ct, (int)blockIdx.y * a.HW + ct,
                        b, mx, scnt, sent);
}

// ------------------------------------------------------------------ p = 2, 3, 4
// Row groups. A thread owns one 16-byte chunk of LR = p^A consecutive rows (a leaf) of one head
// slot: it closes the windows of levels 1 .. A itself. A workgroup holds RG leaves of each of its
// HW head slots, RG LR a multiple of p^(L-1); the sums of the higher levels are formed level by
// level through LDS from the leaves' sums, each window adding its p children in order, so every
// fp64 sum is the one a walk over the rows gives. The norms of BR rows of every leaf at a time go
// through LDS to one thread per row, and the scores' maxima go up level by level with the sums.
//
// Bound: HBM on long sequences; on short ones the latency of one workgroup's chain. A walk over
// at least 64 rows in steps of 8, with two barriers and a 128-term fp64 chain on part of the
// threads in each, took 3 to 7 us a step whatever the size of the problem. Here a workgroup's chain
// is LR / BR steps and L - 1 short levels. Walk -> leaves, pooling and scores: N = 8192, 8 heads, p
// = 4, L = 3 43 -> 19 us; 24,576, 12 / 4 heads of 64, p = 2, L = 6 73 -> 33; 32,805, 6 / 3 heads of
// 64, p = 3, L = 5 79 -> 33; 16,384, 1 head, p = 4, L = 6 627 -> 23; 524,288, 8 heads, L = 3 807 ->
// 730 (5.8 TB/s); 262,144, 32 / 8 heads, L = 5 893 -> 815. Slot chunks run fastest in the grid: the
// heads of one row are then read at about the same time (the last of these took 983 us with the
// row ranges fastest).

// The value of tensor t (0, 1, 2). By value: a choice among the arguments' addresses (as ?: on the
// members makes it) puts the whole argument block in scratch memory, 640 bytes a thread.
template <typename V>
__device__ __forceinline__ V of_tensor(int t, V x0, V x1, V x2) {
  const V y = t == 1 ? x1 : x2;
  return t == 0 ? x0 : y;
}

// Score row of head slot g, or null.
__device__ __forceinline__ float* score_row(const PoolArgs& a, int g, int64_t b) {
  if (g >= a.nslots) return nullptr;
  const int t = g < a.slot1 ? 0 : g < a.slot2 ? 1 : 2;
  const int h = g - of_tensor(t, 0, a.slot1, a.slot2);
  float* s = of_tensor(t, a.t[0].s, a.t[1].s, a.t[2].s);
  return s ? s + (b * of_tensor(t, a.t[0].H, a.t[1].H, a.t[2].H) + h) * a.Ptot : nullptr;
}

struct LeafArgs {
  PoolArgs a;
  int32_t RG, hw_shift;  // HW = 1 << hw_shift (a.HW)
  int32_t nchunk;        // chunks of HW head slots
  int32_t score;         // any tensor wants scores
  int32_t tile_bytes;    // LDS: staged rows (or leaf sums), then the scores
};

template <typename T, int P, int A, int BR, int L>
__global__ void __launch_bounds__(1024) pool_leaf_kernel(LeafArgs la) {
  constexpr int CH = 16 / sizeof(T);
  constexpr int LR = A == 1 ? P : P * P * (A == 3 ? P : 1);
  constexpr int LT = L - 1 < A ? L - 1 : A;  // levels closed by the thread
  static_assert(LR % BR == 0 && BR % P == 0, "a batch holds whole level-1 windows");
  extern __shared__ __align__(16) unsigned char smem[];
  const PoolArgs& a = la.a;
  const int D = a.D, HW = a.HW, RG = la.RG, NT = blockDim.x, tid = threadIdx.x;
  const int cc = tid & ((1 << a.cpr_shift) - 1), grp = tid >> a.cpr_shift;
  const int hs = grp & (HW - 1), rg = grp >> la.hw_shift;
  const uint32_t rblk = blockIdx.x / (uint32_t)la.nchunk;  // row range; the slot chunk runs fastest
  const int slot0 = (int)(blockIdx.x - rblk * la.nchunk) * HW, gs = slot0 + hs;
  const bool active = gs < a.nslots;
  const int64_t b = blockIdx.y;
  const int32_t N = (int32_t)a.N, R = (int32_t)a.R;
  const int32_t w0 = (int32_t)rblk * a.WR;  // first row of the workgroup
  const int32_t j0 = w0 + rg * LR;                // and of the thread's leaf
  const int ti = gs < a.slot1 ? 0 : gs < a.slot2 ? 1 : 2;
  const int h = gs - of_tensor(ti, 0, a.slot1, a.slot2);
  const T* x = reinterpret_cast<const T*>(of_tensor(ti, a.t[0].x, a.t[1].x, a.t[2].x));
  T* pyr = reinterpret_cast<T*>(of_tensor(ti, a.t[0].pyr, a.t[1].pyr, a.t[2].pyr));
  const bool scored = of_tensor(ti, a.t[0].s, a.t[1].s, a.t[2].s) != nullptr;
  const int H = of_tensor(ti, a.t[0].H, a.t[1].H, a.t[2].H);
  const int64_t stride = (int64_t)H * D;
  const T* xrow = x + ((b * a.N + j0) * H + h) * D + cc * CH;
  const int rowT = D + CH;  // staged rows are padded by 16 bytes
  T* tile = reinterpret_cast<T*>(smem);
  double* red = reinterpret_cast<double*>(smem);
  float* sc = reinterpret_cast<float*>(smem + la.tile_bytes);  // [HW][RG LR] scores of level 0, then 1, ..
  const int rows_wg = RG * LR;
  // entry (l, i) of the thread's head and chunk
  auto pyr_row = [=](int64_t off, int32_t i) __attribute__((always_inline)) {
    return pyr + ((b * (int64_t)R + (off - N) + i) * H + h) * D + cc * CH;
  };

  double acc[A + 1][CH];
#pragma unroll
  for (int l = 0; l <= A; ++l)
#pragma unroll
    for (int c = 0; c < CH; ++c) acc[l][c] = 0.0;
  const bool do_pool = L > 1 && active && pyr != nullptr;
#pragma unroll
  for (int b0 = 0; b0 < LR; b0 += BR) {
    u32x4 v[BR];
#pragma unroll
    for (int r = 0; r < BR; ++r)
      v[r] = (active && j0 + b0 + r < N) ? load16_nt(xrow + (int64_t)(b0 + r) * stride) : u32x4{0, 0, 0, 0};
    if (la.score && active && scored) {
#pragma unroll
      for (int r = 0; r < BR; ++r)
        *reinterpret_cast<u32x4*>(tile + (size_t)((hs * RG + rg) * BR + r) * rowT + cc * CH) = v[r];
    }
    if constexpr (L > 1) {
#pragma unroll
      for (int r = 0; r < BR; ++r) {
        add_row<T>(acc[1], v[r]);
        const int done = b0 + r + 1;  // rows of the leaf so far
        int span = 1;
#pragma unroll
        for (int l = 1; l <= LT; ++l) {
          span *= P;
          if (done % span != 0) break;
          if (do_pool && j0 + done <= N)
            store_mean<T>(pyr_row(a.off[l], (j0 + done) / span - 1), acc[l], a.inv[l], a.pwd[l], P != 3);
          if (l < LT) {
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[l + 1][c] += acc[l][c];
          }
          if (l < LT || LT < A) {
#pragma unroll
            for (int c = 0; c < CH; ++c) acc[l][c] = 0.0;
          }
        }
      }
    }
    if (la.score) {
      __syncthreads();
      // one thread per staged row; slot by slot, rows in order
      for (int e = tid; e < HW * RG * BR; e += NT) {
        const int s_ = e / (RG * BR), q = e - s_ * (RG * BR), g = q / BR, r = q - g * BR;
        float* srow = score_row(a, slot0 + s_, b);
        const int32_t j = w0 + g * LR + b0 + r;
        if (!srow || j >= N) continue;
        const float nrm = row_norm<T, false>(tile + (size_t)e * rowT, D);
        sc[s_ * rows_wg + g * LR + b0 + r] = nrm;
        srow[j] = nrm;
      }
      __syncthreads();  // the tile may be rewritten
    }
  }
  if constexpr (L > 1) {
    // maxima and, above the leaves, sums: level l from level l - 1
    float* sl = sc;
    int nw = rows_wg;  // windows of level l - 1 per head slot
    if constexpr (L - 1 > A) {
#pragma unroll
      for (int c = 0; c < CH; ++c) red[c * NT + tid] = acc[A][c];
    }
    int span = 1;
#pragma unroll
    for (int l = 1; l < L; ++l) {
      span *= P;
      const int n = nw / P;
      __syncthreads();
      float* sn = sl + HW * nw;
      if (la.score) {
        for (int e = tid; e < HW * n; e += NT) {
          const int s_ = e / n, i = e - s_ * n;
          float* srow = score_row(a, slot0 + s_, b);
          if (!srow || w0 + i * span >= N) continue;
          float mx = 0.0f;
#pragma unroll
          for (int r = 0; r < P; ++r) {
            const float y = sl[s_ * nw + i * P + r];
            mx = mx > y ? mx : y;
          }
          sn[s_ * n + i] = mx;
          srow[a.off[l] + w0 / span + i] = mx;
        }
      }
      if (L - 1 > A && l > A) {
        // thread (chunk, slot, window): the children's sums sit at their threads' places
        const int i = rg;  // window index in the slot
        double sum[CH];
        const bool mine = i < n;
        if (mine) {
#pragma unroll
          for (int c = 0; c < CH; ++c) sum[c] = 0.0;
#pragma unroll
          for (int r = 0; r < P; ++r)
#pragma unroll
            for (int c = 0; c < CH; ++c) sum[c] += red[c * NT + ((((i * P + r) << la.hw_shift) + hs) << a.cpr_shift) + cc];
        }
        __syncthreads();
        if (mine) {
#pragma unroll
          for (int c = 0; c < CH; ++c) red[c * NT + tid] = sum[c];
          if (do_pool && w0 + i * span < N)
            store_mean<T>(pyr_row(a.off[l], w0 / span + i), sum, a.inv[l], a.pwd[l], P != 3);
        }
      }
      sl = sn;
      nw = n;
    }
  }
}

// p^(L-1) rows fit a workgroup of leaves of LR rows, of the smallest head (D = 64).
template <typename T>
constexpr bool leaf_fits(int p, int LR, int L) {
  int64_t P = 1;
  for (int l = 1; l < L; ++l) P *= p;
  return P / LR * (64 * (int)sizeof(T) / 16) <= 1024;
}

// Launches the leaf kernel with leaves of p^A rows; false if a workgroup cannot hold p^(L-1) rows.
template <typename T, int P, int A, int BR>
static bool launch_leaf(const LhShape& s, PoolArgs a, hipStream_t st) {
  constexpr int LR = A == 1 ? P : P * P * (A == 3 ? P : 1);
  const int CPR = s.D * (int)sizeof(T) / 16;
  const int64_t rg_min = s.P > LR ? s.P / LR : 1;
  if (rg_min * CPR > 1024) return false;
  a.cpr_shift = CPR == 8 ? 3 : CPR == 16 ? 4 : 5;
  // head slots per workgroup: the largest power of two that fits 256 threads (rows of
  // neighbouring heads are contiguous) and leaves at most an eighth of the slots empty
  int sh = 0;
  for (int t = 1; t <= 4; ++t) {
    const int hw = 1 << t, padded = (a.nslots + hw - 1) / hw * hw;
    if (rg_min * CPR * hw <= kLeafThreads && padded * 8 <= a.nslots * 9) sh = t;
  }
  LeafArgs la;
  a.HW = 1 << sh;
  la.hw_shift = sh;
  la.nchunk = (a.nslots + a.HW - 1) / a.HW;
  const int64_t unit = rg_min * CPR << sh;
  la.RG = (int32_t)(rg_min * (unit >= kLeafThreads ? 1 : kLeafThreads / unit));
  a.WR = la.RG * LR;
  la.score = a.t[0].s || a.t[1].s || a.t[2].s;
  la.a = a;
  const int nt = (la.RG * CPR) << sh;
  const size_t staged = la.score ? (size_t)la.RG * a.HW * BR * (s.D * sizeof(T) + 16) : 0;
  const size_t sums = s.L - 1 > A ? (size_t)nt * (16 / sizeof(T)) * 8 : 0;
  const size_t tile = staged > sums ? staged : sums;
  la.tile_bytes = (int32_t)tile;
  size_t scores = 0;  // of every level of the workgroup's rows
  for (int l = 0, n = a.WR; l < s.L; ++l, n /= P) scores += (size_t)n * a.HW * sizeof(float);
  const size_t shm = tile + (la.score ? scores : 0);
  if (shm > kMaxLds) return false;
  const dim3 grid((unsigned)((s.N + a.WR - 1) / a.WR * la.nchunk), (unsigned)s.B);
  const dim3 block((unsigned)nt);
  constexpr int L0 = A == 3 && P > 2 ? 6 : 1;  // leaves of p^3 rows serve deep pyramids only
#define LH_LEAF_CASE(LL)                                                                             \
  case LL:                                                                                           \
    if constexpr (LL >= L0 && leaf_fits<T>(P, LR, LL))                                               \
      hipLaunchKernelGGL((pool_leaf_kernel<T, P, A, BR, LL>), grid, block, shm, st, la);             \
    break;
  switch (s.L) {
    LH_LEAF_CASE(1)
    LH_LEAF_CASE(2)
    LH_LEAF_CASE(3)
    LH_LEAF_CASE(4)
    LH_LEAF_CASE(5)
    LH_LEAF_CASE(6)
    LH_LEAF_CASE(7)
    default: LH_LEAF_CASE(8)
  }
#undef LH_LEAF_CASE
  return true;
}

template <typename T, int L>
static void launch_L(const PoolArgs& a, dim3 grid, dim3 block, size_t shm, hipStream_t st) {
  if constexpr (L >= 6) {
    if (a.p == 4) {
      hipLaunchKernelGGL((pool_score_kernel<T, L, 4>), grid, block, shm, st, a);
      return;
    }
  }
  hipLaunchKernelGGL((pool_score_kernel<T, L, 0>), grid, block, shm, st, a);
}

// Leaves of 16, 9 or 8 rows (p = 4, 3, 2); of 64 (p = 4) where p^(L-1) rows take more than 1024
// threads. The walk over p^(L-1) rows stays for p > 4, for pyramids too deep for a workgroup, and in
// bf16 where a workgroup of leaves would be one head slot of 1024 threads (L = 6, D = 128) although the
// walk fills the chip, three workgroups a CU, and its chunks of 16 slots are full to an eighth. Walk and
// leaves, us, by the walk's workgroups: 48 slots, 576 945 and 782; 672 960 and 903; 768 974 and 1034; 1024 1369
// and 1366; 2048 2525 and 2713; 4096 4899 and 5445; 16, 32, 64 and 80 slots alike (768 0.95 to 0.97 of
// the time, 4096 0.85 to 0.92); with chunks half or two thirds full, 24 slots, 768 878 and 768; 4096 4384 and
// 4072; 40 slots 4565 and 4536. In fp32 leaves are as fast or faster (48 slots, 1536 3190 and 3160; 24, 2048
// 3203 and 3097), and of 64 rows too (L = 7, N = 4,194,304, 48 slots 17.1 and 16.7 ms; D = 64 11.4 and 10.8).
template <typename T>
static bool launch_leaves(const LhShape& s, const PoolArgs& a, hipStream_t st) {
  if (s.p == 4) {
    const int64_t chunks = (a.nslots + 15) / 16, walk = s.N / s.P * chunks * s.B;
    const bool full = chunks * 16 * 8 <= a.nslots * 9;
    if (sizeof(T) == 2 && s.P / 16 * (s.D / 8) == 1024 && full && walk >= 720) return false;
    return launch_leaf<T, 4, 2, 8>(s, a, st) || (s.L >= 6 && launch_leaf<T, 4, 3, 8>(s, a, st));
  }
  if (s.p == 3) return launch_leaf<T, 3, 2, 9>(s, a, st);
  if (s.p == 2) return launch_leaf<T, 2, 3, 8>(s, a, st);
  return false;
}

template <typename T>
static hipError_t launch_T(const LhShape& s, PoolArgs& a, hipStream_t st) {
  if (launch_leaves<T>(s, a, st)) return hipGetLastError();
  const int CH = 16 / sizeof(T);
  const int CPR = s.D / CH;
  int cs = 0;
  while ((1 << cs) < CPR) ++cs;
  a.cpr_shift = cs;
  a.HW = a.nslots < 256 / CPR ? a.nslots : 256 / CPR;
  if (a.HW < 1) a.HW = 1;
  // rows per workgroup: the smallest multiple of p^(L-1) that is >= 64
  int64_t W = s.P;
  while (W < 64) W += s.P;
  a.WR = (int32_t)W;
  for (int l = 0; l < 16; ++l) a.epb[l] = l < s.L ? (int32_t)(W / s.pw[l]) : 0;
  dim3 grid((unsigned)((s.N + W - 1) / W), (unsigned)((a.nslots + a.HW - 1) / a.HW), (unsigned)s.B);
  dim3 block((unsigned)(a.HW * CPR));
  const bool score = a.t[0].s || a.t[1].s || a.t[2].s;
  const int rowT = s.D + 16 / (int)sizeof(T);
  size_t shm = score ? (size_t)kPoolRB * a.HW * rowT * sizeof(T) + 2 * (size_t)kPoolRB * a.HW * sizeof(float) : 0;
  switch (s.L) {
    case 1: launch_L<T, 1>(a, grid, block, shm, st); break;
    case 2: launch_L<T, 2>(a, grid, block, shm, st); break;
    case 3: launch_L<T, 3>(a, grid, block, shm, st); break;
    case 4: launch_L<T, 4>(a, grid, block, shm, st); break;
    case 5: launch_L<T, 5>(a, grid, block, shm, st); break;
    case 6: launch_L<T, 6>(a, grid, block, shm, st); break;
    case 7: launch_L<T, 7>(a, grid, block, shm, st); break;
    case 8: launch_L<T, 8>(a, grid, block, shm, st); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace lh

using namespace lh;

hipError_t lh_launch_pool_score(const LhShape& s, const void* q, const void* k, const void* v,
                                void* qpyr, void* kpyr, void* vpyr, float* s_qk, float* s_kq,
                                hipStream_t st) {
  PoolArgs a = {};
  const PoolTensor jobs[3] = {{q, qpyr, s_qk, s.Hq}, {k, kpyr, s_kq, s.Hkv}, {v, vpyr, nullptr, s.Hkv}};
  int n = 0;
  for (const PoolTensor& j : jobs) {
    PoolTensor t = j;
    if (s.L == 1) t.pyr = nullptr;
    if (!t.x || (!t.pyr && !t.s)) continue;
    a.t[n++] = t;
  }
  if (n == 0) return hipSuccess;
  for (int i = n; i < 3; ++i) a.t[i] = PoolTensor{nullptr, nullptr, nullptr, 0};
  a.slot1 = a.t[0].H;
  a.slot2 = a.slot1 + a.t[1].H;
  a.nslots = a.slot2 + a.t[2].H;
  a.N = s.N;
  a.R = s.R;
  a.Ptot = s.Ptot;
  a.D = s.D;
  a.p = s.p;
  for (int l = 0; l < 16; ++l) {
    a.inv[l] = l < s.L ? 1.0 / (double)s.pw[l] : 0.0;
    a.pwd[l] = l < s.L ? (double)s.pw[l] : 1.0;
  }
  a.pow2 = (s.p & (s.p - 1)) == 0;
  for (int l = 0; l < 17; ++l) a.off[l] = s.off[l];
  return s.dtype == LH_BF16 ? launch_T<bf16_t>(s, a, st) : launch_T<float>(s, a, st);
}
