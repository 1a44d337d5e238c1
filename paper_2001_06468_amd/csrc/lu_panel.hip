// Panel of the partial-pivoting LU with its rows in registers.
//
// A 64-column panel of at most 8192 rows is factored in sub-panels of
// W columns, one launch each.  Workgroup 0 holds every row of the sub-panel in
// registers (R rows x W columns per thread: the register file of a CU is
// 512 KB, its LDS 160 KB), so a pivot decision needs workgroup barriers and no
// grid-wide one; the other workgroups apply the previous sub-panel to the
// columns right of this one, two whole columns each, so that work is off the
// critical path.  Workgroup 0 applies the previous sub-panel to its own columns
// itself: a launch depends on the launch before it only through finished
// columns.
//
// Rows are not moved between registers when they are interchanged: a thread
// keeps the rows it loaded, the rows among the first W that lost their place
// remember their position, and finished pivot rows go straight to memory.  The
// multipliers are stored column by column as they are formed; the displaced
// rows (W at most) are stored once more at their final position at the end.
//
// What bounds it: the pivot chain.  Per column: the largest entry of a thread's
// R rows, of its wave (DPP), of the eight waves (LDS), one reciprocal, the
// broadcast of the pivot row, R fused updates per column left.
// Pivots and factors are those of the column-by-column elimination (largest
// magnitude, lowest row on ties; every entry takes its updates in increasing
// pivot order; multipliers are correctly rounded quotients, except that of an entry so small
// (below about 1e-291 in FP64, 2e-31 in FP32) that its remainder is subnormal, which
// may be off by one more rounding).
//
// Measured, FP64, per launch of W columns: 19.9 us (W = 16) at 512 rows, 21.9 us
// at 1024, 24.1 us at 1536, 12.7 us (W = 8) at 2048, 15.5 us at 3072, 19.0 us at
// 4096, i.e. 1.2 to 2.4 us a column; one grid-wide barrier per column took 4.4 us
// (600 rows) to 5.5 us (3000 rows).  Nearly all of it is issue and latency of
// dependent instructions on one or two waves per SIMD (with the update on one side of a
// branch, which copied every register twice, and addresses formed per column: 22.1, 23.5,
// 26.8, 13.9, 16.8 and 21.8 us).  Measured equal or slower: a rolled loop with the next column searched
// ahead (one barrier and one LDS read a column, but twice the fused updates), four
// waves of twice the rows, the interchange done in registers (copies at every
// branch), 32 columns at 512 rows.
#include <algorithm>
#include <type_traits>
#include <utility>

#include "nrs_internal.h"

namespace nrs {

namespace {

constexpr int kPT = 512;   // threads of a panel workgroup

__device__ inline uint32_t max8_u32(uint32_t v) {   // over each group of 8 lanes
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0, (int)v, 0xB1, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0, (int)v, 0x4E, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0, (int)v, 0x141, 0xF, 0xF, false));
  return v;
}

// Maximum over the wave (ALL) or over lanes 0..7, as a uniform value.
template <bool ALL>
__device__ inline uint32_t group_max(uint32_t v) {
  v = max8_u32(v);
  if (!ALL) return (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0, (int)v, 0x140, 0xF, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0, (int)v, 0x142, 0xA, 0xF, false));
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)0, (int)v, 0x143, 0xC, 0xF, false));
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// Lane with the largest (hi, lo) pair, the lowest idx on ties.  The low word
// and the index are looked at only where the high word does not decide.
template <bool ALL>
__device__ inline int best_lane(uint32_t hi, uint32_t lo, int idx) {
  constexpr uint64_t kMask = ALL ? ~0ull : 0xffull;
  const uint32_t mh = group_max<ALL>(hi);
  uint64_t b = __ballot(hi == mh) & kMask;
  if (b & (b - 1)) {
    const uint32_t ml = group_max<ALL>(hi == mh ? lo : 0u);
    const bool in = hi == mh && lo == ml;
    b = __ballot(in) & kMask;
    if (b & (b - 1)) {
      const uint32_t key = in ? 0x7fffffffu - (uint32_t)idx : 0u;
      const uint32_t mi = group_max<ALL>(key);
      b = __ballot(in && key == mi) & kMask;
    }
  }
  return __builtin_ctzll(b);
}

__device__ inline void split_key(double v, uint32_t& hi, uint32_t& lo) {
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  hi = (uint32_t)(b >> 32);
  lo = (uint32_t)b;
}
__device__ inline void split_key(float v, uint32_t& hi, uint32_t& lo) {
  hi = __float_as_uint(v);
  lo = 0u;
}

__device__ inline float lane_value(float v, int lane) {
  return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ inline double lane_value(double v, int lane) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffll), lane);
  const int hi = __builtin_amdgcn_readlane((int)(b >> 32), lane);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// |piv| (hi: its high word) far enough from the ends of the range that 1/piv is a normal
// number and the corrected quotient below can neither overflow nor lose the reciprocal's
// accuracy: about 1e-279 to 1e279 in FP64, 1e-29 to 1e29 in FP32
template <class T>
__device__ inline bool plain_pivot(uint32_t hi);
template <>
__device__ inline bool plain_pivot<double>(uint32_t hi) { return hi - 0x06000000u < 0x73e00000u; }
template <>
__device__ inline bool plain_pivot<float>(uint32_t hi) { return hi - 0x0f000000u < 0x61000000u; }

// Element access through a buffer resource: offsets at or past the resource's
// size read zero and store nothing, so rows past the panel need no branch.
template <class T>
struct Column {
  __amdgpu_buffer_rsrc_t rs;
  __device__ inline Column(const T* p, int64_t rows)
      : rs(__builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), (short)0,
                                             (int)(rows * (int64_t)sizeof(T)), 0x00020000)) {}
  __device__ inline T get(int row) const;
  __device__ inline void put(int row, T v) const;
};
template <>
__device__ inline double Column<double>::get(int row) const {
  const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, row * 8, 0, 0);
  return __longlong_as_double((long long)(((uint64_t)v[1] << 32) | v[0]));
}
template <>
__device__ inline float Column<float>::get(int row) const {
  return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, row * 4, 0, 0));
}
template <>
__device__ inline void Column<double>::put(int row, double v) const {
  typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
  const uint64_t b = (uint64_t)__double_as_longlong(v);
  const u32x2 w = {(uint32_t)b, (uint32_t)(b >> 32)};
  __builtin_amdgcn_raw_buffer_store_b64(w, rs, row * 8, 0, 0);
}
template <>
__device__ inline void Column<float>::put(int row, float v) const {
  __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rs, row * 4, 0, 0);
}

// lane n of each row of 16 lanes, in all of them
template <int n>
__device__ inline float row16_bcast(float v) {
  return __int_as_float(
      __builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + n, 0xF, 0xF, false));
}
template <int n>
__device__ inline double row16_bcast(double v) {
  const long long b = __double_as_longlong(v);
  const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffll), 0x150 + n, 0xF, 0xF, false);
  const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x150 + n, 0xF, 0xF, false);
  return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

template <class T, int W>
struct PanelLds {
  int4 cand[2][kPT / 64];    // by column parity: (high, low word of the entry, position, row)
  T row[2][W];               // pivot row
  T L[W * W];                // previous sub-panel's unit lower block, column-major
  T u[W * W];                // its U rows on this workgroup's columns, [row][column]
};

// x <- L^-1 x for the unit lower W x W block in S.L, one column per row of 16
// lanes (lane q: entry q).  Entry Q leaves the entries up to it as they are, by a
// select: a zero multiplier would make them NaN where it is infinite.
template <class T, int W, int... Q>
__device__ inline T lower_solve16(const PanelLds<T, W>& S, T x, int q,
                                  std::integer_sequence<int, Q...>) {
  T l[W];
#pragma unroll
  for (int t = 0; t < W; ++t) l[t] = (q > t && q < W) ? S.L[t * W + q] : T(0);
  const auto step = [&](auto at) {
    constexpr int t = decltype(at)::value;
    const T v = x - l[t] * row16_bcast<t>(x);
    x = q > t ? v : x;
  };
  (step(std::integral_constant<int, Q>{}), ...);
  return x;
}

// Columns col0 .. col0+nc-1 (nc <= C), rows kb .. n-1, into registers with the
// previous sub-panel (columns and rows from kb - W) applied: interchanges,
// unit lower solve of its W rows (left in S.u), rank-W update.  Thread t holds
// rows kb + r kPT + t; rows past n are zero.
template <class T, int R, int W, int C>
__device__ inline void load_columns(PanelLds<T, W>& S, T (&a)[R][C], int64_t n, int64_t kb,
                                    int64_t col0, int nc, bool prev, const T* __restrict__ A,
                                    int64_t lda, const int32_t* __restrict__ ipiv) {
  const int tid = threadIdx.x, lane = tid & 63, wid = tid >> 6;
  const int64_t m = n - kb;
  if (!prev) {
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const Column<T> col(A + kb + (col0 + c) * lda, c < nc ? m : 0);
#pragma unroll
      for (int r = 0; r < R; ++r) a[r][c] = col.get(r * kPT + tid);
    }
    return;
  }
  const int64_t base = kb - W;
  // positions relative to base: where the rows that the W interchanges leave at
  // the pivot positions and at the top W positions came from
  const int pl = lane < W ? (int)(ipiv[base + lane] - base) : -1;
  for (int e = tid; e < W * W; e += kPT)
    S.L[e] = A[base + (e & (W - 1)) + (base + e / W) * lda];
  int from_p = pl, from_t = lane;
#pragma unroll
  for (int j = W - 1; j >= 0; --j) {
    const int pj = __builtin_amdgcn_readlane(pl, j);
    from_p = from_p == j ? pj : (from_p == pj ? j : from_p);
    from_t = from_t == j ? pj : (from_t == pj ? j : from_t);
  }
  int src[R];
#pragma unroll
  for (int r = 0; r < R; ++r) src[r] = r * kPT + tid + W;
#pragma unroll
  for (int j = 0; j < W; ++j) {
    const int i = __builtin_amdgcn_readlane(pl, j) - W;
    if (i >= 0 && ((i >> 6) & (kPT / 64 - 1)) == wid) {
      const int f = __builtin_amdgcn_readlane(from_p, j);
#pragma unroll
      for (int r = 0; r < R; ++r)
        if (r == i / kPT && lane == (i & 63)) src[r] = f;
    }
  }
#pragma unroll
  for (int c = 0; c < C; ++c) {
    const Column<T> col(A + base + (col0 + c) * lda, c < nc ? m + W : 0);
#pragma unroll
    for (int r = 0; r < R; ++r) a[r][c] = col.get(src[r]);
  }
  // the top W rows: 16 lanes per column
  const int ft = __shfl(from_t, lane & 15);
  T x = T(0);
  const int xc = tid >> 4, xq = tid & 15;
  if (xc < nc && xq < W) x = A[base + ft + (col0 + xc) * lda];
  constexpr int D = 2;
  T l[D][R];   // multipliers of the next D pivot columns
#pragma unroll
  for (int t = 0; t < D; ++t) {
    const Column<T> lc(A + kb + (base + t) * lda, m);
#pragma unroll
    for (int r = 0; r < R; ++r) l[t][r] = lc.get(r * kPT + tid);
  }
  __syncthreads();
  if (wid < (C * 16 + 63) / 64) {
    x = lower_solve16<T, W>(S, x, xq, std::make_integer_sequence<int, W>{});
    if (xc < C && xq < W) S.u[xq * C + xc] = x;
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < W; ++t) {
    T lt[R];
#pragma unroll
    for (int r = 0; r < R; ++r) lt[r] = l[t % D][r];
    if (t + D < W) {
      const Column<T> lc(A + kb + (base + t + D) * lda, m);
#pragma unroll
      for (int r = 0; r < R; ++r) l[t % D][r] = lc.get(r * kPT + tid);
    }
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const T u = S.u[t * C + c];
#pragma unroll
      for (int r = 0; r < R; ++r) a[r][c] -= lt[r] * u;
    }
  }
}

// The previous sub-panel's U rows on columns col0 .. col0+nc-1 (S.u).
template <class T, int W, int C>
__device__ inline void store_u(const PanelLds<T, W>& S, int64_t kb, int64_t col0, int nc,
                               T* __restrict__ A, int64_t lda) {
  for (int e = threadIdx.x; e < W * nc; e += kPT)
    A[kb - W + (e & (W - 1)) + (col0 + e / W) * lda] = S.u[(e & (W - 1)) * C + e / W];
}

// Row r (uniform) of this lane to LDS: one branch per row.  The empty asm
// statements differ, so the compiler cannot merge the branches into an indexed
// access (which would put the whole array into scratch memory).
template <class T, int R, int W, int Q>
__device__ inline void put_row_at(T* dst, const T (&a)[R][W], int r) {
  if (r == Q) {
#pragma unroll
    for (int c = 0; c < W; ++c) dst[c] = a[Q][c];
    asm volatile("; row %0" ::"n"(Q));
  }
}
template <class T, int R, int W, int... Q>
__device__ inline void put_row(T* dst, const T (&a)[R][W], int r,
                               std::integer_sequence<int, Q...>) {
  (put_row_at<T, R, W, Q>(dst, a, r), ...);
}

// Column j of the sub-panel: pivot search, multipliers, rank-1 update of the
// columns right of it.  j is a compile-time constant, so that the columns stay
// in registers.  pos: position of this thread's first row (-1 once it is a
// pivot); the other rows never move.  A pivot row eliminates itself (its
// multiplier is 1), so finished rows are zero and need no mask.
template <class T, int R, int W, int j>
__device__ inline void eliminate_column(PanelLds<T, W>& S, T (&a)[R][W], int& pos, int wv,
                                        int64_t m, int64_t kb, T*& colp, T* __restrict__ rowp,
                                        int64_t lda, int32_t* __restrict__ ipiv,
                                        int32_t* __restrict__ sing) {
  if (j >= wv) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wid = __builtin_amdgcn_readfirstlane(tid >> 6);
  // this thread's largest entry, the lowest row on ties (NaN is never chosen)
  T best = T(0);
  int br = 0;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const T v = fabs(a[r][j]);
    if (v > best) {
      best = v;
      br = r;
    }
  }
  const int at = br == 0 ? pos : br * kPT + tid;
  uint32_t hi, lo;
  split_key(best, hi, lo);
  const int wl = best_lane<true>(hi, lo, at);
  if (lane == wl) S.cand[j & 1][wid] = make_int4((int)hi, (int)lo, at, br * kPT + tid);
  __syncthreads();
  const int4 cd = S.cand[j & 1][lane & 7];
  const int pw = best_lane<false>((uint32_t)cd.x, (uint32_t)cd.y, cd.z);
  const int khi = __builtin_amdgcn_readlane(cd.x, pw);
  const int klo = __builtin_amdgcn_readlane(cd.y, pw);
  int p = __builtin_amdgcn_readlane(cd.z, pw);
  const int g = __builtin_amdgcn_readlane(cd.w, pw);
  // no entry but zeros and NaN: row j stays, and the matrix counts as singular (whether
  // the zero or the NaN lies in row j)
  const bool none = (khi | klo) == 0;
  if (none) {
    p = j;
    if (pos == j) {
#pragma unroll
      for (int c = 0; c < W; ++c) S.row[j & 1][c] = a[0][c];
    }
  } else if (((g >> 6) & (kPT / 64 - 1)) == wid && lane == (g & 63)) {
    put_row(S.row[j & 1], a, g / kPT, std::make_integer_sequence<int, R>{});
  }
  const bool is_piv = (none ? pos : tid) == (none ? j : g);
  __syncthreads();
  const T ul = S.row[j & 1][lane & (W - 1)];
  const T uz = none ? T(0) : ul;   // nothing is eliminated without a pivot
  T u[W];
#pragma unroll
  for (int c = j; c < W; ++c) u[c] = lane_value(uz, c);
  const T piv = u[j];
  if (wid == 0) {
    // the pivot row is final: its multipliers and its U part
    if (lane < wv) rowp[j] = ul;
    if (lane == j) {
      ipiv[kb + j] = (int32_t)(kb + p);
      if (none) atomicOr(sing, 1);
    }
  }
  // One path for all columns: with the update on one side of a branch only, the whole
  // of a[][] was copied to other registers and back for each column.
  if (plain_pivot<T>((uint32_t)khi)) {
    // quotient by the reciprocal, corrected by its remainder: correctly rounded
    // where the remainder is a normal number (or zero)
    const T inv = T(1) / piv;
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const T q = a[r][j] * inv;
      a[r][j] = fma(fma(-q, piv, a[r][j]), inv, q);
    }
  } else if (!none) {
#pragma unroll
    for (int r = 0; r < R; ++r) a[r][j] = a[r][j] / piv;
  }
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const T l = none ? T(0) : a[r][j];
#pragma unroll
    for (int c = j + 1; c < W; ++c) a[r][c] -= l * u[c];
  }
  if (none) {
    asm volatile("; no pivot");   // a branch, not two selects per column
    if (is_piv) {
#pragma unroll
      for (int c = j + 1; c < W; ++c) a[0][c] = T(0);
    }
  }
  pos = is_piv ? -1 : (pos == j ? p : pos);
  // the first W rows are stored when they become pivots or at the end; what a
  // pivot row stores here is overwritten by the row that takes its place
  const Column<T> col(colp, m);
  colp += lda;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    if (r == 0) {
      if (tid >= W) col.put(tid, a[0][j]);
    } else {
      col.put(r * kPT + tid, a[r][j]);
    }
  }
}

template <class T, int R, int W, int... J>
__device__ inline void eliminate(PanelLds<T, W>& S, T (&a)[R][W], int& pos, int wv, int64_t m,
                                 int64_t kb, T* __restrict__ A, int64_t lda,
                                 int32_t* __restrict__ ipiv, int32_t* __restrict__ sing,
                                 std::integer_sequence<int, J...>) {
  T* colp = A + kb + kb * lda;                           // column j, from row kb
  T* rowp = A + kb + (kb + (threadIdx.x & 63)) * lda;    // this lane's column of row kb + j
  (eliminate_column<T, R, W, J>(S, a, pos, wv, m, kb, colp, rowp, lda, ipiv, sing), ...);
}

// Factors columns kb .. kb+wv-1 (rows kb .. n-1) after applying the sub-panel
// before them; workgroups 1, 2, ... apply it to columns kb+wv .. kend-1.
template <class T, int R, int W>
__global__ __launch_bounds__(kPT) void k_panel_reg(int64_t n, int64_t kb, int wv, int prev,
                                                   int64_t kend, T* __restrict__ A, int64_t lda,
                                                   int32_t* __restrict__ ipiv,
                                                   int32_t* __restrict__ sing) {
  __shared__ __align__(16) PanelLds<T, W> S;
  const int tid = threadIdx.x;
  const int64_t m = n - kb;
  if (blockIdx.x > 0) {
    T a[R][2];
    const int64_t col0 = kb + wv + 2 * (int64_t)(blockIdx.x - 1);
    const int nc = (int)min<int64_t>(2, kend - col0);
    load_columns<T, R, W, 2>(S, a, n, kb, col0, nc, true, A, lda, ipiv);
    // every load of this workgroup's columns has landed before any store
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const Column<T> col(A + kb + (col0 + c) * lda, c < nc ? m : 0);
#pragma unroll
      for (int r = 0; r < R; ++r) col.put(r * kPT + tid, a[r][c]);
    }
    store_u<T, W, 2>(S, kb, col0, nc, A, lda);
    return;
  }
  T a[R][W];
  load_columns<T, R, W, W>(S, a, n, kb, kb, wv, prev != 0, A, lda, ipiv);
  // every load of these columns has landed before any store (the first store
  // comes after a barrier)
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  int pos = tid;
  eliminate<T, R, W>(S, a, pos, wv, m, kb, A, lda, ipiv, sing,
                     std::make_integer_sequence<int, W>{});
  if (prev) store_u<T, W, W>(S, kb, kb, wv, A, lda);
  // rows that lost their place, over what was stored there before
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's stores are done
  __syncthreads();
  if (tid < W && pos >= wv && pos < m) {
#pragma unroll
    for (int c = 0; c < W; ++c)
      if (c < wv) A[kb + pos + (kb + c) * lda] = a[0][c];
  }
}

template <class T, int R, int W>
hipError_t run_panel(int64_t n, int64_t k, int jb, T* A, int64_t lda, int32_t* ipiv,
                     int32_t* sing, hipStream_t s) {
  const int64_t kend = k + jb;
  for (int64_t kb = k; kb < kend; kb += W) {
    const int wv = (int)std::min<int64_t>(W, kend - kb);
    const int prev = kb > k;
    const unsigned help = prev ? (unsigned)((kend - kb - wv + 1) / 2) : 0u;
    hipLaunchKernelGGL((k_panel_reg<T, R, W>), dim3(1 + help), dim3(kPT), 0, s, n, kb, wv, prev,
                       kend, A, lda, ipiv, sing);
  }
  return hipGetLastError();
}

template <int V>
using ic = std::integral_constant<int, V>;

// Rows per thread and columns per sub-panel for an m-row panel: as wide as the
// registers allow (R W <= 64 doubles), since every sub-panel pays its launch and
// its loads.  f(R, W); false if m is too large.
template <class F>
bool panel_shape(int64_t m, F f) {
  if (m <= 1 * kPT) return f(ic<1>{}, ic<16>{}), true;
  if (m <= 2 * kPT) return f(ic<2>{}, ic<16>{}), true;
  if (m <= 3 * kPT) return f(ic<3>{}, ic<16>{}), true;
  if (m <= 4 * kPT) return f(ic<4>{}, ic<8>{}), true;
  if (m <= 6 * kPT) return f(ic<6>{}, ic<8>{}), true;
  if (m <= 8 * kPT) return f(ic<8>{}, ic<8>{}), true;
  if (m <= 16 * kPT) return f(ic<16>{}, ic<4>{}), true;
  return false;
}

}  // namespace

// Sub-panel width for m rows (0: too many rows for the registers of a CU).
int panel_reg_width(int64_t m) {
  int w = 0;
  panel_shape(m, [&](auto, auto W) { w = decltype(W)::value; });
  return w;
}

// Columns k .. k+jb-1 over rows k .. n-1.  Inside the panel, a sub-panel's
// interchanges have been applied to the columns right of it only: columns of
// earlier sub-panels are left to k_laswp_trsm.
template <class T>
hipError_t launch_panel_reg(int64_t n, int64_t k, int jb, T* A, int64_t lda, int32_t* ipiv,
                            int32_t* sing, hipStream_t s) {
  hipError_t e = hipErrorInvalidValue;
  panel_shape(n - k, [&](auto R, auto W) {
    e = run_panel<T, decltype(R)::value, decltype(W)::value>(n, k, jb, A, lda, ipiv, sing, s);
  });
  return e;
}

template hipError_t launch_panel_reg<float>(int64_t, int64_t, int, float*, int64_t, int32_t*,
                                            int32_t*, hipStream_t);
template hipError_t launch_panel_reg<double>(int64_t, int64_t, int, double*, int64_t, int32_t*,
                                             int32_t*, hipStream_t);

}  // namespace nrs
