// Geometry at time t, nearest-neighbour map and the nu-sorted (CSR) layout of
// the quadrature points.
#include <type_traits>

#include "nrs_internal.h"

namespace nrs {

namespace {

// Body-frame wave displacement and derivatives of one point.
__device__ inline void wave_terms(const double* __restrict__ wave, int p, double s, double t,
                                  double d[3], double dds[3], double ddt[3]) {
  const double* wp = wave + 6 * p;
  const double beta = wp[0], A0 = wp[1], A1 = wp[2], k = wp[3], om = wp[4], phi = wp[5];
  const double th = k * s - om * t + phi;
  double sn, cs;
  sincos(th, &sn, &cs);
  const double amp = A0 + A1 * s;
  d[0] = beta * s;
  d[1] = amp * sn;
  d[2] = 0.0;
  dds[0] = beta;
  dds[1] = A1 * sn + amp * k * cs;
  dds[2] = 0.0;
  ddt[0] = 0.0;
  ddt[1] = -om * amp * cs;
  ddt[2] = 0.0;
}

// One point set of a scene for k_geometry.  mode 0: force points ->
// positions and prescribed velocities; mode 1: quadrature points ->
// positions and weights.
struct GeomSet {
  int64_t n;
  int32_t mode;
  const double* xi;
  const int32_t* body;
  const int32_t* part;
  const double* s;
  const double* aux;
  double* pos;
  double* out2;
};

__device__ inline void geometry_point(const GeomSet& g, int64_t i, int32_t M, int32_t P,
                                      const double* __restrict__ wave,
                                      const double* __restrict__ Y, double t) {
  const int64_t n = g.n;
  const int mode = g.mode;
  const double* __restrict__ xi = g.xi;
  const int32_t* __restrict__ body = g.body;
  const int32_t* __restrict__ part = g.part;
  const double* __restrict__ s = g.s;
  const double* __restrict__ aux = g.aux;
  double* __restrict__ pos = g.pos;
  double* __restrict__ out2 = g.out2;
  double p[3] = {xi[i], xi[n + i], xi[2 * n + i]};
  double d[3] = {0, 0, 0}, dds[3] = {0, 0, 0}, ddt[3] = {0, 0, 0};
  // out-of-range indices are treated as "none" (no wave / fixed point)
  const int pi = (part[i] >= 0 && part[i] < P) ? part[i] : -1;
  if (pi >= 0) {
    wave_terms(wave, pi, s[i], t, d, dds, ddt);
    p[0] += d[0];
    p[1] += d[1];
    p[2] += d[2];
  }
  const int b = (body[i] >= 0 && body[i] < M) ? body[i] : -1;
  double q[3], v[3];
  if (b >= 0) {
    const double* Yb = Y + 12 * b;
    for (int r = 0; r < 3; ++r) {
      q[r] = Yb[r] + (Yb[3 + 3 * r] * p[0] + Yb[4 + 3 * r] * p[1] + Yb[5 + 3 * r] * p[2]);
      v[r] = Yb[3 + 3 * r] * ddt[0] + Yb[4 + 3 * r] * ddt[1] + Yb[5 + 3 * r] * ddt[2];
    }
  } else {
    q[0] = p[0];
    q[1] = p[1];
    q[2] = p[2];
    v[0] = v[1] = v[2] = 0.0;
  }
  if (pos) {
    pos[i] = q[0];
    pos[n + i] = q[1];
    pos[2 * n + i] = q[2];
  }
  if (out2) {
    if (mode == 0) {
      if (b < 0) {
        v[0] = aux[i];
        v[1] = aux[n + i];
        v[2] = aux[2 * n + i];
      }
      out2[i] = v[0];
      out2[n + i] = v[1];
      out2[2 * n + i] = v[2];
    } else {
      double w = aux[i];
      if (pi >= 0) w *= sqrt(dds[0] * dds[0] + dds[1] * dds[1] + dds[2] * dds[2]);
      out2[i] = w;
    }
  }
}

// Both point sets of a scene in one launch: the first nb0 workgroups take
// set 0 (force points), the rest set 1 (quadrature points).
__global__ void k_geometry(GeomSet g0, GeomSet g1, int64_t nb0, int32_t M, int32_t P,
                           const double* __restrict__ wave, const double* __restrict__ Y,
                           double t) {
  const bool first = blockIdx.x < nb0;
  const GeomSet& g = first ? g0 : g1;
  const int64_t i = (blockIdx.x - (first ? 0 : nb0)) * (int64_t)blockDim.x + threadIdx.x;
  if (i >= g.n) return;
  geometry_point(g, i, M, P, wave, Y, t);
}

// kNnSplit consecutive lanes per quadrature point, each over every kNnSplit-th
// force point of the point's group, in increasing order, then the smallest
// (distance, index) of them.  Squared distance without contraction so that the
// result equals the (dx*dx + dy*dy) + dz*dz of a plain FP64 evaluation; the first
// force point stands until one is strictly nearer (also where its distance is
// not a number).
// What bounds it: one lane's chain of dependent FP64 operations when a group is
// small (a filament's 40 points), FP64 issue when it is large.  With one thread per
// quadrature point over force points in LDS, 10,000 points in groups of 40
// took 14.5 us (40 workgroups; 4.4 us so), 32,000 points in one group of 2000
// 207 us (98 us so), 74,000 in one of 4624 537 us (227 us so; 382 us while every
// lane tested every point's own range).
constexpr int kNnBlock = 256;
constexpr int kNnSplit = 8;
// kPer points per lane group share the loads of a force point; one point where
// more would leave SIMDs without a wave (kNnManyQ).
constexpr int64_t kNnManyQ = 32768;
template <int kPer>
__global__ __launch_bounds__(kNnBlock) void k_nearest(int64_t N, const double* __restrict__ x,
                                                      GroupTable gt, int64_t Q,
                                                      const double* __restrict__ X,
                                                      const int32_t* __restrict__ groupX,
                                                      int32_t* __restrict__ nu) {
#pragma clang fp contract(off)
  const int64_t q0 = (blockIdx.x * (int64_t)kNnBlock + threadIdx.x) / kNnSplit * kPer;
  const int sub = threadIdx.x % kNnSplit;
  int lo[kPer], hi[kPer], ulo = 0x7fffffff, uhi = 0;   // each point's group, all of them
  double qx[kPer], qy[kPer], qz[kPer], best[kPer];
  int arg[kPer];
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int64_t q = q0 + e;
    lo[e] = hi[e] = 0;
    qx[e] = qy[e] = qz[e] = 0.0;
    best[e] = __builtin_huge_val();
    arg[e] = 0x7fffffff;
    if (q < Q) {
      const int g = groupX[q];
      if (g >= 0 && g < gt.G) {
        lo[e] = gt.off[g];
        hi[e] = gt.off[g + 1];
      }
      qx[e] = X[q];
      qy[e] = X[Q + q];
      qz[e] = X[2 * Q + q];
    }
    if (hi[e] > lo[e]) {
      ulo = min(ulo, lo[e]);
      uhi = max(uhi, hi[e]);
    }
  }
  if (uhi == 0) ulo = 0;   // no point of this lane group has candidates
  // every lane starts from the first force point (not a number: nothing is nearer)
  bool mixed = false;
  int64_t own = 0;   // candidates of the points, each its group's
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    mixed = mixed || lo[e] != ulo || hi[e] != uhi;
    own += hi[e] - lo[e];
    if (hi[e] > lo[e]) {
      const int j = lo[e];
      const double dx = x[j] - qx[e];
      const double dy = x[N + j] - qy[e];
      const double dz = x[2 * N + j] - qz[e];
      const double d2 = dx * dx + dy * dy + dz * dz;
      best[e] = d2 == d2 ? d2 : -1.0;
      arg[e] = j;
    }
  }
  const auto nearer = [&](int e, int j, double px, double py, double pz, bool in) {
#pragma clang fp contract(off)
    const double dx = px - qx[e];
    const double dy = py - qy[e];
    const double dz = pz - qz[e];
    const double d2 = dx * dx + dy * dy + dz * dz;
    if (d2 < best[e] && in) {
      best[e] = d2;
      arg[e] = j;
    }
  };
  const auto scan = [&](auto all) {
#pragma unroll 4
    for (int j = ulo + sub; j < uhi; j += kNnSplit) {
      const double px = x[j], py = x[N + j], pz = x[2 * N + j];
#pragma unroll
      for (int e = 0; e < kPer; ++e)
        nearer(e, j, px, py, pz, decltype(all)::value || (j >= lo[e] && j < hi[e]));
    }
  };
  if (kPer == 1 || !__any(mixed)) {
    scan(std::true_type{});   // each lane's points share one group
  } else if (!__any(kPer * (int64_t)(uhi - ulo) > 2 * own)) {
    // neighbouring groups: all points over the range that holds them, which shares the
    // loads and takes at most twice the distances (100,000 points that alternate between
    // two groups of 1000: 113 us, 167 us point by point)
    scan(std::false_type{});
  } else {
    // distant groups: point by point, or the force points between them would be walked
    // too (200,000 points in random order of 120 groups of 160: 54 us, 1885 us)
#pragma unroll
    for (int e = 0; e < kPer; ++e)
#pragma unroll 4
      for (int j = lo[e] + sub; j < hi[e]; j += kNnSplit)
        nearer(e, j, x[j], x[N + j], x[2 * N + j], true);
  }
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
#pragma unroll
    for (int o = 1; o < kNnSplit; o <<= 1) {
      const double ob = __shfl_xor(best[e], o, 64);
      const int oa = __shfl_xor(arg[e], o, 64);
      if (ob < best[e] || (ob == best[e] && oa < arg[e])) {
        best[e] = ob;
        arg[e] = oa;
      }
    }
    if (q0 + e < Q && sub == 0) nu[q0 + e] = hi[e] > lo[e] ? arg[e] : -1;
  }
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

__global__ void k_fill_f64(double* p, double v, int64_t n) {
  const int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

// Quadrature points whose nu is outside [0, N) are left out of the layout and
// counted in cnt[N + 1] (reported as an argument error by the caller).
__global__ void k_csr_count(int64_t N, int64_t Q, const int32_t* __restrict__ nu, int32_t* cnt) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q < Q) {
    const int32_t v = nu[q];
    if (v >= 0 && v < N)
      atomicAdd(&cnt[v], 1);
    else
      atomicAdd(&cnt[N + 1], 1);
  }
}

// Exclusive scan of cnt[0..N) into seg[0..N]; cnt becomes the scatter cursor.
// st (may be NULL): argument error when some nu was outside [0, N) (counted
// in cnt[N + 1]).
constexpr int kScanBlock = 1024;

// Exclusive scan of one value per thread over a kScanBlock workgroup: a
// shuffle scan inside each wavefront, then the wavefronts' totals scanned by
// wavefront 0 (two barriers); *total receives the sum over the workgroup.
__device__ inline int32_t block_exclusive_scan(int32_t v, int32_t* wtot, int32_t* total) {
  const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
  int32_t x = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int32_t y = __shfl_up(x, off, 64);
    if (lane >= off) x += y;
  }
  if (lane == 63) wtot[wv] = x;
  __syncthreads();
  if (wv == 0) {
    int32_t t = lane < kScanBlock / 64 ? wtot[lane] : 0;
#pragma unroll
    for (int off = 1; off < kScanBlock / 64; off <<= 1) {
      const int32_t y = __shfl_up(t, off, 64);
      if (lane >= off) t += y;
    }
    if (lane < kScanBlock / 64) wtot[lane] = t;
  }
  __syncthreads();
  *total = wtot[kScanBlock / 64 - 1];
  return x - v + (wv ? wtot[wv - 1] : 0);
}

__global__ __launch_bounds__(kScanBlock) void k_csr_scan(int64_t N, int32_t* cnt, int32_t* seg,
                                                         SolveState* st) {
  if (threadIdx.x == 0 && st && cnt[N + 1] > 0) {
    st->nonfinite = 2;
    st->failed = 1;
    st->stop = 1;
  }
  __shared__ int32_t wtot[kScanBlock / 64];
  const int tid = threadIdx.x;
  const int64_t per = (N + kScanBlock - 1) / kScanBlock;
  const int64_t a = tid * per, b = min<int64_t>(N, a + per);
  int32_t sum = 0;
  for (int64_t i = a; i < b; ++i) sum += cnt[i];
  int32_t total;
  int32_t run = block_exclusive_scan(sum, wtot, &total);
  for (int64_t i = a; i < b; ++i) {
    const int32_t c = cnt[i];
    seg[i] = run;
    cnt[i] = run;
    run += c;
  }
  if (tid == kScanBlock - 1) seg[N] = total;
}

__global__ void k_csr_scatter(int64_t N, int64_t Q, const int32_t* __restrict__ nu,
                              int32_t* cursor, int32_t* perm) {
  const int64_t q = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (q < Q) {
    const int32_t v = nu[q];
    if (v >= 0 && v < N) {
      const int pos = atomicAdd(&cursor[v], 1);
      perm[pos] = (int32_t)q;
    }
  }
}

// Per segment (one wavefront each): order the members by original index
// (deterministic layout), pack the sorted coordinates and sum the patch
// weight.  A member's place is the number of members with a smaller index
// (the indices are distinct), found by comparing against every member
// broadcast from its lane; segments longer than 256 members (not met by
// the workloads) are sorted by insertion in lane 0.
constexpr int kFinishWaves = 4;
__device__ inline double csr_store(int64_t Q, int64_t n, int pos, int q, const double* __restrict__ X,
                                   const double* __restrict__ w, int32_t* __restrict__ perm,
                                   int32_t* __restrict__ nus, double4* __restrict__ X64,
                                   float4* __restrict__ X32hi, float4* __restrict__ X32lo) {
  const double px = X[q], py = X[Q + q], pz = X[2 * Q + q];
  const double wq = w ? w[q] : 1.0;
  perm[pos] = q;
  nus[pos] = (int32_t)n;
  X64[pos] = make_double4(px, py, pz, wq);
  const float hx = (float)px, hy = (float)py, hz = (float)pz;
  X32hi[pos] = make_float4(hx, hy, hz, (float)wq);
  X32lo[pos] = make_float4((float)(px - (double)hx), (float)(py - (double)hy),
                           (float)(pz - (double)hz), 0.0f);
  return wq;
}

__global__ __launch_bounds__(kFinishWaves * 64) void k_csr_finish(
    int64_t N, int64_t Q, const int32_t* __restrict__ seg, int32_t* __restrict__ perm,
    const double* __restrict__ X, const double* __restrict__ w, int32_t* __restrict__ nus,
    double4* __restrict__ X64, float4* __restrict__ X32hi, float4* __restrict__ X32lo,
    double* __restrict__ W) {
  // weights by sorted position, so that the patch weight is summed in an
  // order that does not depend on the (atomic, unordered) scatter
  __shared__ double s_w[kFinishWaves][256];
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const int64_t n = (int64_t)blockIdx.x * kFinishWaves + wv;
  if (n >= N) return;
  const int a = seg[n], len = seg[n + 1] - a;
  double wsum = 0.0;
  if (len <= 256) {
    int key[4];
#pragma unroll
    for (int c = 0; c < 4; ++c) key[c] = c * 64 + lane < len ? perm[a + c * 64 + lane] : 0x7fffffff;
    int rank[4] = {0, 0, 0, 0};
#pragma unroll
    for (int cj = 0; cj < 4; ++cj) {
      if (cj * 64 < len) {   // wave-uniform
        const int top = min(64, len - cj * 64);
        for (int jj = 0; jj < top; ++jj) {
          const int kj = __shfl(key[cj], jj, 64);
#pragma unroll
          for (int c = 0; c < 4; ++c) rank[c] += kj < key[c] ? 1 : 0;
        }
      }
    }
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c * 64 + lane < len)
        s_w[wv][rank[c]] = csr_store(Q, n, a + rank[c], key[c], X, w, perm, nus, X64, X32hi, X32lo);
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    // lane l adds sorted places l, l + 64, ...; then a fixed tree over lanes
#pragma unroll
    for (int c = 0; c < 4; ++c)
      if (c * 64 + lane < len) wsum += s_w[wv][c * 64 + lane];
  } else if (lane == 0) {
    for (int i = a + 1; i < a + len; ++i) {
      const int32_t k = perm[i];
      int j = i - 1;
      while (j >= a && perm[j] > k) {
        perm[j + 1] = perm[j];
        --j;
      }
      perm[j + 1] = k;
    }
    for (int i = a; i < a + len; ++i) wsum += csr_store(Q, n, i, perm[i], X, w, perm, nus, X64, X32hi, X32lo);
  }
#pragma unroll
  for (int o = 32; o >= 1; o >>= 1) wsum += __shfl_xor(wsum, o, 64);
  if (lane == 0) W[n] = wsum;
}

// The whole layout in one launch for N <= kCsrSmallN and Q <= kCsrSmallQ: a workgroup
// owns kSegPts consecutive force points, reads every nu, counts the points of
// lower force points (its place in the layout, so workgroups need nothing from
// each other) and lists its own in order of their index, which is the order of the
// layout: nothing is sorted.  Every wave takes a contiguous share of the
// quadrature points and keeps its list in LDS (kSegCap entries; a wave that finds
// more reads its share a second time instead).
// What bounds it: the latency of reading nu, eight loads in flight per lane.
// A count, scan and scatter in one workgroup followed by a sort per force
// point took 8.2 + 4.7 us for 10,000 points (10.8 us so) and 25 + 6 us for 40,000
// (15.8 us so).
constexpr int64_t kCsrSmallN = 8192;
constexpr int64_t kCsrSmallQ = 1 << 17;
constexpr int kSegPts = 16;
constexpr int kSegWaves = 16;
constexpr int kSegCap = 512;
constexpr int kSegBatch = 8;
constexpr int kSegW = 64;

__device__ __forceinline__ void csr_segments(
    int32_t block, int64_t N, int64_t Q, const int32_t* __restrict__ nu, const double* __restrict__ X,
    const double* __restrict__ w, int32_t* __restrict__ seg, int32_t* __restrict__ perm,
    int32_t* __restrict__ nus, double4* __restrict__ X64, float4* __restrict__ X32hi,
    float4* __restrict__ X32lo, double* __restrict__ W, SolveState* st) {
  __shared__ int32_t list[kSegWaves][kSegCap];    // q + (force point - n0) 2^20
  __shared__ int16_t rank[kSegWaves][kSegCap];    // place among the wave's of that force point
  __shared__ int32_t cnt[kSegWaves][kSegPts];     // members, then where each wave's start
  __shared__ double sw[kSegPts][kSegW];           // weights by place (short segments)
  __shared__ int32_t below[kSegWaves], len[kSegWaves];
  __shared__ int32_t base[kSegPts + 1];
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const uint64_t lower = (1ull << lane) - 1;
  const int32_t n0 = block * kSegPts;
  const int32_t n1 = (int32_t)min<int64_t>(N, n0 + kSegPts);
  const int32_t per = ((int32_t)Q + kSegWaves * 64 - 1) / (kSegWaves * 64) * 64;
  const int32_t qa = min((int32_t)Q, wv * per), qb = min((int32_t)Q, qa + per);
  // calls f(q, nu[q] or N past the share) for the 64 points from q on, for all of them
  auto scan = [&](auto f) {
    for (int32_t q = qa; q < qb; q += 64 * kSegBatch) {
      int32_t v[kSegBatch];
#pragma unroll
      for (int e = 0; e < kSegBatch; ++e) {
        const int32_t qe = q + 64 * e + lane;
        v[e] = qe < qb ? nu[qe] : (int32_t)N;
      }
#pragma unroll
      for (int e = 0; e < kSegBatch; ++e) f(q + 64 * e + lane, v[e]);
    }
  };
  int32_t lo = 0, found = 0, bad = 0;   // wave-uniform (but bad)
  int32_t next = 0;   // lane k < kSegPts: members of force point n0 + k so far
  scan([&](int32_t q, int32_t v) {
    lo += __popcll(__ballot(v >= 0 && v < n0));
    const bool hit = v >= n0 && v < n1;
    bad |= q < qb && (v < 0 || v >= N);
    const uint64_t m = __ballot(hit);
    if (m) {
      const int at = found + __popcll(m & lower);
      int32_t before = 0;
      for (uint64_t left = m; left;) {   // one force point at a time
        const int32_t k = __builtin_amdgcn_readlane(v, __builtin_ctzll(left));
        const uint64_t mk = __ballot(hit && v == k);
        if (v == k) before = __builtin_amdgcn_readlane(next, k - n0) + __popcll(mk & lower);
        if (lane == k - n0) next += __popcll(mk);
        left &= ~mk;
      }
      if (hit && at < kSegCap) {
        list[wv][at] = q | (v - n0) << 20;
        rank[wv][at] = (int16_t)before;
      }
      found += __popcll(m);
    }
  });
  if (lane < kSegPts) cnt[wv][lane] = next;
  if (lane == 0) {
    below[wv] = lo;
    len[wv] = found;
  }
  if (block == 0 && st && bad) {
    st->nonfinite = 2;
    st->failed = 1;
    st->stop = 1;
  }
  __syncthreads();
  if (wv == 0) {
    int32_t first = 0, mine = 0;
#pragma unroll
    for (int k = 0; k < kSegWaves; ++k) {
      first += below[k];
      if (lane < kSegPts) mine += cnt[k][lane];
    }
    int32_t incl = mine;
#pragma unroll
    for (int o = 1; o < kSegPts; o <<= 1) {
      const int32_t y = __shfl_up(incl, o, 64);
      if (lane >= o) incl += y;
    }
    if (lane < kSegPts) {
      int32_t at = first + incl - mine;
      base[lane] = at;
      if (n0 + lane < n1) seg[n0 + lane] = at;
      if (lane == kSegPts - 1) base[kSegPts] = at + mine;
      if (n0 + lane == N - 1) seg[N] = at + mine;
#pragma unroll
      for (int k = 0; k < kSegWaves; ++k) {
        const int32_t c = cnt[k][lane];
        cnt[k][lane] = at;
        at += c;
      }
    }
  }
  __syncthreads();
  // every thread stores records of every list (a force point's members mostly lie in
  // one wave's share)
  const int32_t lens = len[lane & (kSegWaves - 1)];
  const bool tooLong = __any(lens > kSegCap);
#pragma unroll 1
  for (int k = 0; k < kSegWaves; ++k) {
    const int32_t c = __builtin_amdgcn_readlane(lens, k);
    if (c > kSegCap) continue;
    for (int32_t i = threadIdx.x; i < c; i += kSegWaves * 64) {
      const int32_t v = list[k][i], p = v >> 20, at = cnt[k][p] + rank[k][i];
      const double wq = csr_store(Q, n0 + p, at, v & ((1 << 20) - 1), X, w, perm, nus, X64, X32hi,
                                  X32lo);
      if (at - base[p] < kSegW) sw[p][at - base[p]] = wq;
    }
  }
  if (found > kSegCap) {   // this wave's list was too short: its share once more
    next = lane < kSegPts ? cnt[wv][lane] : 0;
    scan([&](int32_t q, int32_t v) {
      const bool hit = v >= n0 && v < n1;
      for (uint64_t left = __ballot(hit); left;) {
        const int32_t k = __builtin_amdgcn_readlane(v, __builtin_ctzll(left));
        const uint64_t mk = __ballot(hit && v == k);
        const int32_t at = __builtin_amdgcn_readlane(next, k - n0) + __popcll(mk & lower);
        if (hit && v == k)
          csr_store(Q, k, at, q, X, w, perm, nus, X64, X32hi, X32lo);
        if (lane == k - n0) next += __popcll(mk);
        left &= ~mk;
      }
    });
  }
  const int32_t longest = base[min(lane, kSegPts - 1) + 1] - base[min(lane, kSegPts - 1)];
  const bool fromLds = !tooLong && !__any(longest > kSegW);   // the same in every wave
  if (!fromLds) __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's records are stored
  __syncthreads();
  // patch weights: lane l adds places l, l + 64, ...; then a fixed tree over lanes
  for (int k = wv; k < n1 - n0; k += kSegWaves) {
    double sum = 0.0;
    const int32_t c = base[k + 1] - base[k];
    for (int32_t i = lane; i < c; i += 64) sum += fromLds ? sw[k][i] : X64[base[k] + i].w;
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) sum += __shfl_xor(sum, o, 64);
    if (lane == 0) W[n0 + k] = sum;
  }
}

__global__ __launch_bounds__(kSegWaves * 64) void k_csr_segments(
    int64_t N, int64_t Q, const int32_t* __restrict__ nu, const double* __restrict__ X,
    const double* __restrict__ w, int32_t* __restrict__ seg, int32_t* __restrict__ perm,
    int32_t* __restrict__ nus, double4* __restrict__ X64, float4* __restrict__ X32hi,
    float4* __restrict__ X32lo, double* __restrict__ W, SolveState* st) {
  csr_segments((int32_t)blockIdx.x, N, Q, nu, X, w, seg, perm, nus, X64, X32hi, X32lo, W, st);
}

__global__ __launch_bounds__(kSegWaves * 64) void k_csr_segments_batch(
    const BatchSys* __restrict__ sys, const int64_t* __restrict__ first, int32_t s0, int32_t s1) {
  const int64_t g = first[s0] + blockIdx.x;
  const int32_t s = batch_find(first, s0, s1, g);
  const BatchSys& y = sys[s];
  csr_segments((int32_t)(g - first[s]), y.N, y.Q, as_global(y.nu), as_global(y.X), as_global(y.w),
               as_global(y.seg), as_global(y.perm), as_global(y.nus), as_global(y.X64),
               as_global(y.X32hi), as_global(y.X32lo), as_global(y.W), as_global(y.st));
}

inline dim3 grid1(int64_t n, int b) { return dim3((unsigned)((n + b - 1) / b)); }

}  // namespace

hipError_t launch_geometry(const nrs_scene& sc, double t, const double* Y, double* x, double* X,
                           double* w, double* u, hipStream_t s) {
  GeomSet g0 = {(sc.N > 0 && (x || u)) ? sc.N : 0, 0, sc.xi, sc.body, sc.part, sc.s, sc.ufix, x, u};
  GeomSet g1 = {(sc.Q > 0 && (X || w)) ? sc.Q : 0, 1, sc.Xi, sc.bodyX, sc.partX, sc.sX, sc.w0, X, w};
  const int64_t nb0 = (g0.n + 255) / 256, nb1 = (g1.n + 255) / 256;
  if (nb0 + nb1 == 0) return hipSuccess;
  hipLaunchKernelGGL(k_geometry, dim3((unsigned)(nb0 + nb1)), dim3(256), 0, s, g0, g1, nb0, sc.M,
                     sc.P, sc.wave, Y, t);
  return hipGetLastError();
}

hipError_t launch_nearest(int64_t N, const double* x, const GroupTable& gt, int64_t Q,
                          const double* X, const int32_t* groupX, int32_t* nu, hipStream_t s) {
  if (Q == 0) return hipSuccess;
  if (Q < kNnManyQ)
    hipLaunchKernelGGL(k_nearest<1>, grid1(Q * kNnSplit, kNnBlock), dim3(kNnBlock), 0, s, N, x, gt,
                       Q, X, groupX, nu);
  else
    hipLaunchKernelGGL(k_nearest<4>, grid1((Q + 3) / 4 * kNnSplit, kNnBlock), dim3(kNnBlock), 0, s,
                       N, x, gt, Q, X, groupX, nu);
  return hipGetLastError();
}

hipError_t launch_fill_i32(int32_t* p, int32_t v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_i32, grid1(n, 256), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t launch_fill_f64(double* p, double v, int64_t n, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_fill_f64, grid1(n, 256), dim3(256), 0, s, p, v, n);
  return hipGetLastError();
}

hipError_t launch_build_csr(int64_t N, int64_t Q, const double* X, const double* w,
                            const int32_t* nu, Sorted& srt, SolveState* st, hipStream_t s) {
  if (N <= kCsrSmallN && Q <= kCsrSmallQ) {
    hipLaunchKernelGGL(k_csr_segments, dim3((unsigned)((N + kSegPts - 1) / kSegPts)),
                       dim3(kSegWaves * 64), 0, s, N, Q, nu, X, w, srt.seg, srt.perm, srt.nus,
                       srt.X64, srt.X32hi, srt.X32lo, srt.W, st);
    return hipGetLastError();
  }
  hipError_t e = launch_fill_i32(srt.cnt, 0, N + 2, s);
  if (e != hipSuccess) return e;
  if (Q > 0) {
    hipLaunchKernelGGL(k_csr_count, grid1(Q, 256), dim3(256), 0, s, N, Q, nu, srt.cnt);
  }
  hipLaunchKernelGGL(k_csr_scan, dim3(1), dim3(kScanBlock), 0, s, N, srt.cnt, srt.seg, st);
  if (Q > 0) {
    hipLaunchKernelGGL(k_csr_scatter, grid1(Q, 256), dim3(256), 0, s, N, Q, nu, srt.cnt,
                       srt.perm);
  }
  hipLaunchKernelGGL(k_csr_finish, dim3((unsigned)((N + kFinishWaves - 1) / kFinishWaves)),
                     dim3(kFinishWaves * 64), 0, s, N, Q, srt.seg, srt.perm, X, w, srt.nus, srt.X64,
                     srt.X32hi, srt.X32lo, srt.W);
  return hipGetLastError();
}

int64_t batch_blocks_points(const BatchSys& y) {
  return y.N <= kCsrSmallN && y.Q <= kCsrSmallQ ? (y.N + kSegPts - 1) / kSegPts : 0;
}

hipError_t launch_csr_batch(const BatchSet& bs, hipStream_t s) {
  return batch_launch(bs, kBatchCsr, [&](const int64_t* first, int32_t s0, int32_t s1, unsigned g) {
    hipLaunchKernelGGL(k_csr_segments_batch, dim3(g), dim3(kSegWaves * 64), 0, s, bs.sys, first, s0,
                       s1);
  });
}

}  // namespace nrs
