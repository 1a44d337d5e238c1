// Fused NEAREST operator assembly (Sec. 3 eqs. 18, 21-23 and the matrix view
// after them), rigid-body blocks of the swimming problem (Sec. 2, Sec. 4),
// right-hand side, and the matrix-free FP64 product used by refinement.
//
// Mapping: one lane per collocation row m, lanes of a wave take consecutive m
// so that every store of A (column-major) is a contiguous 64-element run.  A
// workgroup owns a strip of kTN force points n; the quadrature points of each
// n are contiguous in the nu-sorted layout, so the inner loop walks one
// segment with wave-uniform (scalar) loads and sums the segment in registers:
// the segmented reduction over nu needs no cross-lane traffic and the dense
// 3N x 3Q stokeslet matrix is never formed.
#include <algorithm>
#include <type_traits>

#include "nrs_internal.h"

namespace nrs {

namespace {

// Launch shapes (rows per workgroup, force points per strip); every shape
// computes each entry with the same operations, so the choice (made by the
// autotuner) never changes a result.
constexpr int kShapeBlk[kAsmShapes] = {64, 64, 64, 128, 128, 128, 256, 256, 256};
constexpr int kShapeTN[kAsmShapes] = {4, 8, 16, 4, 8, 16, 4, 8, 16};
// In the smallest shape each of four waves takes one force point of the strip, in the
// others every wave takes the whole strip for 64 rows of its own: small matrices leave SIMDs idle
// unless a wave has one force point only.
constexpr bool asm_split(int blk, int tn) { return blk == 64 && tn == 4; }
constexpr int asm_threads(int blk, int tn) { return asm_split(blk, tn) ? 64 * tn : blk; }

// Component j of e_i x r.
__device__ inline double cross_unit(int i, int j, const double r[3]) {
  // (e_i x r)_j = eps_{j i k} r_k
  if (i == j) return 0.0;
  const int k = 3 - i - j;
  // eps_{j i k} = +1 for cyclic (j,i,k)
  const bool cyc = (j == 0 && i == 1) || (j == 1 && i == 2) || (j == 2 && i == 0);
  return cyc ? r[k] : -r[k];
}

// The rigid-body rows and columns of the swimming problem, written by extra
// workgroups of the assembly launch.  Task t < 3N M: row `row` of the
// velocity equations and body s = t / 3N, its six entries in columns
// 3N + 6s .. 3N + 6s + 5 (-1 for U_j on its own component, -(e_i x r_m)_j
// for Omega_i, zero for other bodies).  Task 3N M + t', t' < n M: column
// col = t' / M and body s = t' % M, the six entries of rows 3N + 6s ..
// (force rows W_m delta_jk, moment rows W_m (r_m x e_k)_i for the body's
// points, zero elsewhere and in the rigid-rigid block).  r_m = x_m - x0.
struct RigidArgs {
  int64_t N;
  int32_t M;
  const int32_t* body;
  const double* x;
  const double* Y;
  const double* W;
};

template <class T>
__device__ inline void rigid_task(int64_t t, const RigidArgs& g, T* __restrict__ A, int64_t lda) {
  const int64_t N = g.N, M = g.M, n = 3 * N + 6 * M;
  const int64_t ta = 3 * N * M;
  if (t < ta) {
    const int s = (int)(t / (3 * N));
    const int64_t row = t - (int64_t)s * 3 * N;
    const int j = (int)(row / N);
    const int64_t m = row - j * N;
    const bool own = g.body[m] == s;
    double r[3] = {0.0, 0.0, 0.0};
    if (own) {
      r[0] = g.x[m] - g.Y[12 * s + 0];
      r[1] = g.x[N + m] - g.Y[12 * s + 1];
      r[2] = g.x[2 * N + m] - g.Y[12 * s + 2];
    }
    T* col = A + (3 * N + 6 * (int64_t)s) * lda + row;
    for (int c = 0; c < 6; ++c) {
      double v = 0.0;
      if (own) v = c < 3 ? (c == j ? -1.0 : 0.0) : -cross_unit(c - 3, j, r);
      col[c * lda] = (T)v;
    }
    return;
  }
  t -= ta;
  if (t >= n * M) return;
  const int64_t col = t / M;
  const int s = (int)(t - col * M);
  T* out = A + col * lda + 3 * N + 6 * (int64_t)s;
  if (col < 3 * N) {
    const int k = (int)(col / N);
    const int64_t m = col - k * N;
    if (g.body[m] == s) {
      const double r[3] = {g.x[m] - g.Y[12 * s], g.x[N + m] - g.Y[12 * s + 1],
                           g.x[2 * N + m] - g.Y[12 * s + 2]};
      const double wm = g.W[m];
      for (int c = 0; c < 6; ++c)
        // (r x e_k)_i = -(e_k x r)_i
        out[c] = (T)(c < 3 ? (c == k ? wm : 0.0) : -wm * cross_unit(k, c - 3, r));
      return;
    }
  }
  for (int c = 0; c < 6; ++c) out[c] = (T)0.0;
}

// Workgroups past the force-point strips (blockIdx.y >= strips) take the
// rigid-body tasks, one consecutive task per thread.
template <class T, int kAsmBlock, int kTN>
__device__ inline bool rigid_part(const RigidArgs& g, T* __restrict__ A, int64_t lda) {
  const int64_t strips = (g.N + kTN - 1) / kTN;
  if ((int64_t)blockIdx.y < strips) return false;
  const int64_t t = (((int64_t)blockIdx.y - strips) * gridDim.x + blockIdx.x) *
                        asm_threads(kAsmBlock, kTN) + threadIdx.x;
  if (g.M > 0) rigid_task<T>(t, g, A, lda);
  return true;
}

// Row of this thread and its force points [n0, nend).
template <int kAsmBlock, int kTN>
__device__ inline int64_t asm_share(int64_t N, int64_t& n0, int64_t& nend) {
  n0 = (int64_t)blockIdx.y * kTN;
  if (asm_split(kAsmBlock, kTN)) {
    n0 += __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    nend = min<int64_t>(N, n0 + 1);
    return blockIdx.x * (int64_t)kAsmBlock + (threadIdx.x & 63);
  }
  nend = min<int64_t>(N, n0 + kTN);
  return blockIdx.x * (int64_t)kAsmBlock + threadIdx.x;
}

// FP32 form: coordinates carried as hi + lo floats so that r = x_m - X_q keeps
// FP32 relative accuracy even when |r| << |x|.
template <int kAsmBlock, int kTN>
__global__ __launch_bounds__(asm_threads(kAsmBlock, kTN)) void k_assemble32(
    int64_t N, const double* __restrict__ x, const int32_t* __restrict__ seg,
    const float4* __restrict__ Xhi, const float4* __restrict__ Xlo, float eps2, float scale,
    float* __restrict__ A, int64_t lda, RigidArgs rg) {
  if (rigid_part<float, kAsmBlock, kTN>(rg, A, lda)) return;
  int64_t n0, nend;
  const int64_t m = asm_share<kAsmBlock, kTN>(N, n0, nend);
  const bool live = m < N;
  float xh = 0, yh = 0, zh = 0, xl = 0, yl = 0, zl = 0;
  if (live) {
    const double px = x[m], py = x[N + m], pz = x[2 * N + m];
    xh = (float)px;
    yh = (float)py;
    zh = (float)pz;
    xl = (float)(px - (double)xh);
    yl = (float)(py - (double)yh);
    zl = (float)(pz - (double)zh);
  }
  for (int64_t n = n0; n < nend; ++n) {
    const int a = seg[n], b = seg[n + 1];
    float a00 = 0, a11 = 0, a22 = 0, a01 = 0, a02 = 0, a12 = 0;
    for (int p = a; p < b; ++p) {
      const float4 h = Xhi[p];
      const float4 l = Xlo[p];
      const float rx = (xh - h.x) + (xl - l.x);
      const float ry = (yh - h.y) + (yl - l.y);
      const float rz = (zh - h.z) + (zl - l.z);
      const float d = rx * rx + ry * ry + rz * rz + eps2;
      const float rho = __builtin_amdgcn_rsqf(d);
      const float t = h.w * (rho * rho * rho);
      const float s = (d + eps2) * t;
      const float tx = t * rx, ty = t * ry, tz = t * rz;
      a00 += s + tx * rx;
      a11 += s + ty * ry;
      a22 += s + tz * rz;
      a01 += tx * ry;
      a02 += tx * rz;
      a12 += ty * rz;
    }
    if (live) {
      float* c0 = A + n * lda;
      float* c1 = A + (N + n) * lda;
      float* c2 = A + (2 * N + n) * lda;
      c0[m] = scale * a00;
      c0[N + m] = scale * a01;
      c0[2 * N + m] = scale * a02;
      c1[m] = scale * a01;
      c1[N + m] = scale * a11;
      c1[2 * N + m] = scale * a12;
      c2[m] = scale * a02;
      c2[N + m] = scale * a12;
      c2[2 * N + m] = scale * a22;
    }
  }
}

template <int kAsmBlock, int kTN>
__global__ __launch_bounds__(asm_threads(kAsmBlock, kTN)) void k_assemble64(
    int64_t N, const double* __restrict__ x, const int32_t* __restrict__ seg,
    const double4* __restrict__ X64, double eps2, double scale, double* __restrict__ A,
    int64_t lda, RigidArgs rg) {
  if (rigid_part<double, kAsmBlock, kTN>(rg, A, lda)) return;
  int64_t n0, nend;
  const int64_t m = asm_share<kAsmBlock, kTN>(N, n0, nend);
  const bool live = m < N;
  double px = 0, py = 0, pz = 0;
  if (live) {
    px = x[m];
    py = x[N + m];
    pz = x[2 * N + m];
  }
  for (int64_t n = n0; n < nend; ++n) {
    const int a = seg[n], b = seg[n + 1];
    double a00 = 0, a11 = 0, a22 = 0, a01 = 0, a02 = 0, a12 = 0;
    for (int p = a; p < b; ++p) {
      const double4 q = X64[p];
      const double rx = px - q.x, ry = py - q.y, rz = pz - q.z;
      const double d = rx * rx + ry * ry + rz * rz + eps2;
      const double rho = rsqrt_refined(d);
      const double t = q.w * (rho * rho * rho);
      const double s = (d + eps2) * t;
      const double tx = t * rx, ty = t * ry, tz = t * rz;
      a00 += s + tx * rx;
      a11 += s + ty * ry;
      a22 += s + tz * rz;
      a01 += tx * ry;
      a02 += tx * rz;
      a12 += ty * rz;
    }
    if (live) {
      double* c0 = A + n * lda;
      double* c1 = A + (N + n) * lda;
      double* c2 = A + (2 * N + n) * lda;
      c0[m] = scale * a00;
      c0[N + m] = scale * a01;
      c0[2 * N + m] = scale * a02;
      c1[m] = scale * a01;
      c1[N + m] = scale * a11;
      c1[2 * N + m] = scale * a12;
      c2[m] = scale * a02;
      c2[N + m] = scale * a12;
      c2[2 * N + m] = scale * a22;
    }
  }
}

// b = [u; f_ext or 0]; with b32 != NULL also its FP32 copy; with st != NULL
// also the body-index check (body[m] in [-1, M), else an argument error).
__device__ inline void rhs_entry(int64_t i, int64_t N, int32_t M, const double* __restrict__ u,
                                 const double* __restrict__ ft, double* __restrict__ b,
                                 float* __restrict__ b32, const int32_t* __restrict__ body,
                                 SolveState* st) {
  const int64_t n = 3 * N + 6 * (int64_t)M;
  if (st && i < N && (body[i] < -1 || body[i] >= M)) {
    st->nonfinite = 2;
    st->failed = 1;
    st->stop = 1;
  }
  if (i >= n) return;
  const double v = i < 3 * N ? u[i] : (ft ? ft[i - 3 * N] : 0.0);
  b[i] = v;
  if (b32) b32[i] = (float)v;
}

constexpr int kRhsThreads = 256;
__global__ void k_rhs(int64_t N, int32_t M, const double* __restrict__ u,
                      const double* __restrict__ ft, double* __restrict__ b,
                      float* __restrict__ b32, const int32_t* __restrict__ body, SolveState* st) {
  rhs_entry(blockIdx.x * (int64_t)kRhsThreads + threadIdx.x, N, M, u, ft, b, b32, body, st);
}

__global__ void k_rhs_batch(const BatchSys* __restrict__ sys, const int64_t* __restrict__ first,
                            int32_t s0, int32_t s1) {
  const int64_t g = first[s0] + blockIdx.x;
  const int32_t s = batch_find(first, s0, s1, g);
  const BatchSys& y = sys[s];
  rhs_entry((g - first[s]) * kRhsThreads + threadIdx.x, y.N, y.M, as_global(y.u), as_global(y.ft),
            as_global(y.b), as_global(y.r32), as_global(y.body), as_global(y.st));
}

// Pair sum of the matrix-free product: chunk partial sums of the flow of the
// force densities f at the N force points (one per lane).  The sources are the
// nu-sorted quadrature points, so a wave reads a 32-byte record (position and
// weight) per pair by scalar load and a force density once per segment, and no
// pass gathers sources first.  Workgroups are dealt to the eight XCDs in turn; with
// at least eight chunks, workgroup 8 (pb + pblocks k) + x takes block pb of 64
// points and chunk 8k + x, so an XCD's L2 holds its eighth of the sources.  Wave w
// sums a contiguous quarter of its chunk, the four wave sums are added in a fixed
// order.
// What bounds it: FP64 issue (24 instructions and a quarter-rate reciprocal square
// root per pair, 3 per segment), and below about 10^7 pairs the launch and the scalar
// loads' latency, hence the short chunks of apply_plan().  The factor of a segment's
// force density is summed over the segment and applied once (kPerSegment): applied pair by
// pair, 26 instructions, 13,000 x 130,000 pairs took 1687 us a call (1600 us so; 1615 us
// with gathered records).  Segments of one or two points lose by it (4000 of one point
// 34.8 -> 36.6 us, of two 46.9 -> 48.4 us, of four 75.4 -> 74.9 us), hence the rule
// pair_per_segment().  Against gathering 64-byte source records first and the tracers'
// chunks of 256 sources (mean over calls, converged ones that exit included): one
// filament (40 x 400 pairs) 16.5 -> 5.7 us, 25 filaments (1000 x 10,000) 21.6 -> 13.8
// us, 100 filaments (4000 x 40,000) 100.8 -> 99.8 us.
constexpr int kPairThreads = 256;
constexpr int kPairWaves = kPairThreads / 64;
__host__ __device__ inline bool pair_per_segment(int64_t N, int64_t Q) { return Q >= 4 * N; }

template <bool kPerSegment>
__device__ __forceinline__ void apply_pairs(
    int64_t block, int64_t N, int64_t pblocks, int32_t chunks, int64_t chunk,
    const double* __restrict__ x, const int32_t* __restrict__ seg,
    const int32_t* __restrict__ nus, const double4* __restrict__ X64,
    const double* __restrict__ f, double eps2, double* __restrict__ part) {
  __shared__ double red[3][kPairWaves][64];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int32_t ch;
  int64_t pb;
  if (chunks >= 8) {
    const int64_t j = block >> 3;
    pb = j % pblocks;
    ch = 8 * (int32_t)(j / pblocks) + (int32_t)(block & 7);
    if (ch >= chunks) return;
  } else {
    ch = (int32_t)(block % chunks);
    pb = block / chunks;
  }
  const int64_t m = pb * 64 + lane;
  double px = 0.0, py = 0.0, pz = 0.0;
  if (m < N) {
    px = x[m];
    py = x[N + m];
    pz = x[2 * N + m];
  }
  // this wave's sorted sources [a, b), wave-uniform (points outside every segment
  // are not in the layout: seg[N] of them at most Q)
  const int64_t total = seg[N];
  const int64_t q0 = min<int64_t>(total, (int64_t)ch * chunk);
  const int64_t q1 = min<int64_t>(total, q0 + chunk);
  const int64_t per = (q1 - q0 + kPairWaves - 1) / kPairWaves;
  const int64_t a64 = min<int64_t>(q1, q0 + w * per);
  const int b = __builtin_amdgcn_readfirstlane((int)min<int64_t>(q1, a64 + per));
  int p = __builtin_amdgcn_readfirstlane((int)a64);
  double ux = 0.0, uy = 0.0, uz = 0.0;
  if (p < b) {
    int n = __builtin_amdgcn_readfirstlane(nus[p]);
    double gx = f[n], gy = f[N + n], gz = f[2 * N + n];
    int e = min(b, seg[n + 1]);
    for (;;) {
      // the next segment's force density, loaded beside this one's sources
      const int64_t nn = n + 1 < N ? n + 1 : n;
      const double hx = f[nn], hy = f[N + nn], hz = f[2 * N + nn];
      const int en = seg[nn + 1];
      double ag = 0.0;   // the segment's factor of g (kPerSegment)
#pragma unroll 2
      for (; p < e; ++p) {
        const double4 s = X64[p];
        const double rx = px - s.x, ry = py - s.y, rz = pz - s.z;
        const double d = fma(rz, rz, fma(ry, ry, fma(rx, rx, eps2)));
        const double r = rsqrt_refined(d);                // (|r|^2 + eps^2)^(-1/2)
        const double wr = s.w * r;
        const double t = wr * (r * r);                    // w (|r|^2 + eps^2)^(-3/2)
        const double be = t * fma(rz, gz, fma(ry, gy, rx * gx));
        const double al = fma(t, eps2, wr);               // (|r|^2 + 2 eps^2) t
        ux = fma(be, rx, ux);
        uy = fma(be, ry, uy);
        uz = fma(be, rz, uz);
        if (kPerSegment) {
          ag += al;
        } else {
          ux = fma(al, gx, ux);
          uy = fma(al, gy, uy);
          uz = fma(al, gz, uz);
        }
      }
      if (kPerSegment) {
        ux = fma(ag, gx, ux);
        uy = fma(ag, gy, uy);
        uz = fma(ag, gz, uz);
      }
      if (p >= b) break;
      n = n + 1;
      gx = hx;
      gy = hy;
      gz = hz;
      e = min(b, en);
    }
  }
  red[0][w][lane] = ux;
  red[1][w][lane] = uy;
  red[2][w][lane] = uz;
  __syncthreads();
  if (w < 3 && m < N) {
    double acc = 0.0;
#pragma unroll
    for (int k = 0; k < kPairWaves; ++k) acc += red[w][k][lane];
    part[(int64_t)ch * 3 * N + w * N + m] = acc;
  }
}

template <bool kPerSegment>
__global__ __launch_bounds__(kPairThreads) void k_apply_pairs(
    int64_t N, int64_t pblocks, int32_t chunks, int64_t chunk, const double* __restrict__ x,
    const int32_t* __restrict__ seg, const int32_t* __restrict__ nus,
    const double4* __restrict__ X64, const double* __restrict__ f, double eps2,
    double* __restrict__ part, const int32_t* __restrict__ stop) {
  if (stop && *stop) return;
  apply_pairs<kPerSegment>(blockIdx.x, N, pblocks, chunks, chunk, x, seg, nus, X64, f, eps2, part);
}

__global__ __launch_bounds__(kPairThreads) void k_apply_pairs_batch(
    const BatchSys* __restrict__ sys, const int64_t* __restrict__ first, int32_t s0, int32_t s1,
    int force) {
  const int64_t g = first[s0] + blockIdx.x;
  const int32_t s = batch_find(first, s0, s1, g);
  const BatchSys& y = sys[s];
  if (!force && as_global(y.st)->stop) return;
  const auto pairs = [&](auto per) {
    apply_pairs<decltype(per)::value>(g - first[s], y.N, y.pblocks, y.chunks, y.chunk,
                                      as_global(y.x), as_global(y.seg), as_global(y.nus),
                                      as_global(y.X64), as_global(y.sol), y.eps2,
                                      as_global(y.part));
  };
  if (pair_per_segment(y.N, y.Q))
    pairs(std::true_type{});
  else
    pairs(std::false_type{});
}

constexpr int kApplyThreads = 1024, kApplyWaves = kApplyThreads / 64;

// Stage 2 for the 3N velocity rows: sum the chunks in a fixed order (wave w
// takes a contiguous sixteenth of them with four running sums), scale,
// subtract the rigid-body motion U + Omega x r_m of free-body points.
// What bounds it: the latency of one round of loads of the partial sums, hence sixteen waves
// (1000 force points, 104 chunks: 5.4 us with four waves, 4.0 us so).
__device__ inline void apply_velocity_rows(int64_t block, int64_t N, int32_t M, int32_t chunks,
                                           const double* __restrict__ part, double scale,
                                           const double* __restrict__ x,
                                           const int32_t* __restrict__ body,
                                           const double* __restrict__ Y,
                                           const double* __restrict__ v, double* __restrict__ y) {
  __shared__ double red[kApplyWaves][64];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  const int64_t row = block * 64 + lane;
  const int per = (chunks + kApplyWaves - 1) / kApplyWaves;
  const int c0 = w * per, c1 = min(chunks, c0 + per);
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  if (row < 3 * N) {
    const double* p = part + row;
    int c = c0;
    for (; c + 7 < c1; c += 8) {   // eight loads in flight
      double t[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) t[q] = p[(int64_t)(c + q) * 3 * N];
#pragma unroll
      for (int q = 0; q < 8; ++q) a[q & 3] += t[q];
    }
    double t[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) t[q] = c + q < c1 ? p[(int64_t)(c + q) * 3 * N] : 0.0;
#pragma unroll
    for (int q = 0; q < 8; ++q) a[q & 3] += t[q];
  }
  red[w][lane] = (a[0] + a[1]) + (a[2] + a[3]);
  __syncthreads();
  if (w != 0 || row >= 3 * N) return;
  double acc = 0.0;
#pragma unroll
  for (int q = 0; q < kApplyWaves; ++q) acc += red[q][lane];
  acc *= scale;
  const int j = (int)(row / N);
  const int64_t m = row - j * N;
  const int b = (body[m] >= 0 && body[m] < M) ? body[m] : -1;
  if (b >= 0) {
    const double r[3] = {x[m] - Y[12 * b], x[N + m] - Y[12 * b + 1], x[2 * N + m] - Y[12 * b + 2]};
    const double* uw = v + 3 * N + 6 * b;
    acc -= uw[j];
    for (int i = 0; i < 3; ++i) acc -= uw[3 + i] * cross_unit(i, j, r);
  }
  y[row] = acc;
}

// Stage 2 for the 6M rigid rows of body s: one workgroup, fixed-order
// reduction of W_m f_m and W_m r_m x f_m.
__device__ inline void apply_body_rows(int s, int64_t N, const int32_t* __restrict__ body,
                                       const double* __restrict__ x,
                                       const double* __restrict__ Y,
                                       const double* __restrict__ W,
                                       const double* __restrict__ v, double* __restrict__ y) {
  __shared__ double red[kApplyWaves][8];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  for (int64_t m = threadIdx.x; m < N; m += kApplyThreads) {
    if (body[m] != s) continue;
    const double f[3] = {W[m] * v[m], W[m] * v[N + m], W[m] * v[2 * N + m]};
    const double r[3] = {x[m] - Y[12 * s], x[N + m] - Y[12 * s + 1], x[2 * N + m] - Y[12 * s + 2]};
    acc[0] += f[0];
    acc[1] += f[1];
    acc[2] += f[2];
    acc[3] += r[1] * f[2] - r[2] * f[1];
    acc[4] += r[2] * f[0] - r[0] * f[2];
    acc[5] += r[0] * f[1] - r[1] * f[0];
  }
  const double t = wave_sum8(acc);
  if ((lane & 7) == 0) red[w][wave_sum8_of(lane)] = t;
  __syncthreads();
  if (threadIdx.x < 6) {
    double sum = 0.0;
#pragma unroll
    for (int q = 0; q < kApplyWaves; ++q) sum += red[q][threadIdx.x];
    y[3 * N + 6 * s + threadIdx.x] = sum;
  }
}

// Stage 2 of the product in one launch: workgroups [0, rowblocks) take the
// velocity rows, workgroup rowblocks + s the rigid rows of body s.
__device__ __forceinline__ void apply_stage2(
    int64_t block, int64_t N, int32_t M, int32_t chunks, const double* __restrict__ part,
    double scale, const double* __restrict__ x, const int32_t* __restrict__ body,
    const double* __restrict__ Y, const double* __restrict__ W, const double* __restrict__ v,
    double* __restrict__ y) {
  const int64_t rowblocks = (3 * N + 63) / 64;
  if (block >= rowblocks) {
    apply_body_rows((int)(block - rowblocks), N, body, x, Y, W, v, y);
    return;
  }
  apply_velocity_rows(block, N, M, chunks, part, scale, x, body, Y, v, y);
}

__global__ __launch_bounds__(kApplyThreads) void k_apply_stage2(
    int64_t N, int32_t M, int32_t chunks, const double* __restrict__ part, double scale,
    const double* __restrict__ x, const int32_t* __restrict__ body,
    const double* __restrict__ Y, const double* __restrict__ W, const double* __restrict__ v,
    double* __restrict__ y, const int32_t* __restrict__ stop) {
  if (stop && *stop) return;
  apply_stage2(blockIdx.x, N, M, chunks, part, scale, x, body, Y, W, v, y);
}

__global__ __launch_bounds__(kApplyThreads) void k_apply_stage2_batch(
    const BatchSys* __restrict__ sys, const int64_t* __restrict__ first, int32_t s0, int32_t s1,
    int force) {
  const int64_t g = first[s0] + blockIdx.x;
  const int32_t s = batch_find(first, s0, s1, g);
  const BatchSys& y = sys[s];
  if (!force && as_global(y.st)->stop) return;
  apply_stage2(g - first[s], y.N, y.M, y.chunks, as_global(y.part), y.scale, as_global(y.x),
               as_global(y.body), as_global(y.Y), as_global(y.W), as_global(y.sol),
               as_global(y.Ax));
}

inline dim3 grid1(int64_t n, int b) { return dim3((unsigned)((n + b - 1) / b)); }

// Grid: x = row blocks of BLK, y = strips of TN force points, then enough
// extra y rows of workgroups for the rigid-body tasks.
template <int BLK, int TN>
dim3 asm_grid(const nrs_problem& pb) {
  const int64_t N = pb.N, M = pb.M, n = 3 * N + 6 * M;
  const int64_t gx = (N + BLK - 1) / BLK, strips = (N + TN - 1) / TN;
  const int64_t tasks = 3 * N * M + n * M;
  const int64_t row = gx * asm_threads(BLK, TN);
  const int64_t extra = (tasks + row - 1) / row;
  return dim3((unsigned)gx, (unsigned)(strips + extra));
}
inline RigidArgs rigid_args(const nrs_problem& pb, const Sorted& srt) {
  return RigidArgs{pb.N, pb.M, pb.body, pb.x, pb.Y, srt.W};
}
template <int BLK, int TN>
void asm32(const nrs_problem& pb, const Sorted& srt, float* A, int64_t lda, float scale,
           hipStream_t s) {
  const dim3 g = asm_grid<BLK, TN>(pb);
  hipLaunchKernelGGL((k_assemble32<BLK, TN>), g, dim3(asm_threads(BLK, TN)), 0, s, pb.N, pb.x,
                     srt.seg, srt.X32hi, srt.X32lo, (float)(pb.eps * pb.eps), scale, A, lda,
                     rigid_args(pb, srt));
}
template <int BLK, int TN>
void asm64(const nrs_problem& pb, const Sorted& srt, double* A, int64_t lda, double scale,
           hipStream_t s) {
  const dim3 g = asm_grid<BLK, TN>(pb);
  hipLaunchKernelGGL((k_assemble64<BLK, TN>), g, dim3(asm_threads(BLK, TN)), 0, s, pb.N, pb.x,
                     srt.seg, srt.X64, pb.eps * pb.eps, scale, A, lda, rigid_args(pb, srt));
}

template <class T>
void asm_dispatch(int shape, const nrs_problem& pb, const Sorted& srt, T* A, int64_t lda, T scale,
                  hipStream_t s);
#define NRS_ASM_CASES(F)                                                                        \
  switch (shape) {                                                                             \
    case 0: F<64, 4>(pb, srt, A, lda, scale, s); break;                                        \
    case 1: F<64, 8>(pb, srt, A, lda, scale, s); break;                                        \
    case 2: F<64, 16>(pb, srt, A, lda, scale, s); break;                                       \
    case 3: F<128, 4>(pb, srt, A, lda, scale, s); break;                                       \
    case 4: F<128, 8>(pb, srt, A, lda, scale, s); break;                                       \
    case 5: F<128, 16>(pb, srt, A, lda, scale, s); break;                                      \
    case 6: F<256, 4>(pb, srt, A, lda, scale, s); break;                                       \
    case 7: F<256, 8>(pb, srt, A, lda, scale, s); break;                                       \
    default: F<256, 16>(pb, srt, A, lda, scale, s); break;                                     \
  }
template <>
void asm_dispatch<float>(int shape, const nrs_problem& pb, const Sorted& srt, float* A,
                         int64_t lda, float scale, hipStream_t s) {
  NRS_ASM_CASES(asm32)
}
template <>
void asm_dispatch<double>(int shape, const nrs_problem& pb, const Sorted& srt, double* A,
                          int64_t lda, double scale, hipStream_t s) {
  NRS_ASM_CASES(asm64)
}
#undef NRS_ASM_CASES

}  // namespace

// Shape of a problem that is not tuned.  Small matrices need every wave they can get,
// large ones long stores.  Measured, us per nrs_assemble call with 10 quadrature points per
// force point, 64 x 4 / 128 x 4 / 256 x 4 (best of the other six):
//   FP32 N = 40: 10.6 / 16.0 / 16.7 (22.2); 1000: 24.2 / 25.1 / 25.7 (29.9); 1500: 35.8 / 34.3 /
//   35.2 (37.3); 2100: 50.7 / 48.4 / 50.3 (52.9); 3100: 111 / 96 / 94 (100); 4500: 303 / 268 /
//   236 (244); 6000: 429 / 375 / 363 (370); 8000: 700 / 637 / 628 (635)
//   FP64 N = 40: 11.2 / 18.2 / 18.9 (24.6); 1000: 28.5 / 30.7 / 31.7 (36.2); 2100: 78 / 80 / 78
//   (87); 3100: 209 / 214 / 198 (206); 4500: 435 / 399 / 373 (379); 5200: 477 / 462 / 470 (465);
//   6000: 627 / 607 / 615 (608); 8000: 1084 / 1063 / 1076 (1061)
int32_t asm_untuned_shape(int64_t N, int bits) {
  if (N <= 1536) return 0;
  if (N <= 3072 || (bits == 64 && N > 5000)) return 3;
  return 6;
}

void asm_shape_dims(int32_t shape, int32_t* blk, int32_t* tn) {
  *blk = kShapeBlk[shape];
  *tn = kShapeTN[shape];
}

template <class T>
hipError_t launch_assemble(const nrs_problem& pb, const Sorted& srt, T* A, int64_t lda,
                           hipStream_t s, int32_t shape) {
  const int64_t N = pb.N;
  const int64_t n = 3 * N + 6 * (int64_t)pb.M;
  const T scale = (T)(1.0 / (8.0 * kPi * pb.mu));
  // one launch: the fused operator and, in extra workgroups, the rigid-body
  // rows and columns
  if (shape < 0) shape = asm_untuned_shape(N, 8 * (int)sizeof(T));
  if (N > 0) asm_dispatch<T>(shape, pb, srt, A, lda, scale, s);
  (void)n;
  return hipGetLastError();
}
template hipError_t launch_assemble<float>(const nrs_problem&, const Sorted&, float*, int64_t,
                                           hipStream_t, int32_t);
template hipError_t launch_assemble<double>(const nrs_problem&, const Sorted&, double*, int64_t,
                                            hipStream_t, int32_t);

hipError_t launch_rhs(int64_t N, int32_t M, const double* u, const double* ftext, double* b,
                      hipStream_t s, float* b32, const int32_t* body, SolveState* st) {
  const int64_t n = 3 * N + 6 * (int64_t)M;
  hipLaunchKernelGGL(k_rhs, grid1(std::max(n, st ? N : 0), kRhsThreads), dim3(kRhsThreads), 0, s,
                     N, M, u, ftext, b, b32, body, st);
  return hipGetLastError();
}

hipError_t launch_rhs_batch(const BatchSet& bs, hipStream_t s) {
  return batch_launch(bs, kBatchRhs, [&](const int64_t* first, int32_t s0, int32_t s1, unsigned g) {
    hipLaunchKernelGGL(k_rhs_batch, dim3(g), dim3(kRhsThreads), 0, s, bs.sys, first, s0, s1);
  });
}

// Chunks of the pair sum: 2048 workgroups (eight per CU) while the sources give
// every chunk at least kMinChunk of them.
FieldPlan apply_plan(int64_t N, int64_t Q) {
  constexpr int64_t kMinChunk = 96;
  FieldPlan fp;
  fp.pblocks = (N + 63) / 64;
  int64_t c = 2048 / std::max<int64_t>(fp.pblocks, 1);
  c = std::min<int64_t>(c, std::max<int64_t>(1, Q / kMinChunk));
  c = std::max<int64_t>(1, std::min<int64_t>(c, 1024));
  if (c >= 8) c -= c % 8;  // whole rounds of the eight XCDs
  fp.cap = (int32_t)c;
  fp.chunk = (Q + c - 1) / c;
  fp.chunks = (int32_t)((Q + fp.chunk - 1) / fp.chunk);
  return fp;
}

// Workgroups of the pair sum: whole rounds of the eight XCDs from eight chunks on.
static int64_t pair_blocks(int64_t pblocks, int32_t chunks) {
  return pblocks * (chunks >= 8 ? 8 * ((chunks + 7) / 8) : chunks);
}

// Matrix-free FP64 product: the velocity rows are the flow of the force
// densities v at the force points (chunk partial sums over the nu-sorted sources),
// then the fixed-order chunk sum with the rigid-body motion and the balance rows
// in one launch (k_apply_stage2).  `chunks` bounds the partial buffer (at least
// apply_plan(N, Q).cap).
hipError_t launch_apply(const nrs_problem& pb, const Sorted& srt, const double* v, double* y,
                        double* part, int32_t chunks, const int32_t* stop, hipStream_t s) {
  const int64_t N = pb.N, Q = pb.Q;
  if (N > 0) {
    const FieldPlan fp = apply_plan(N, Q);
    if (fp.chunks > chunks) return hipErrorInvalidValue;
    hipLaunchKernelGGL(pair_per_segment(N, Q) ? k_apply_pairs<true> : k_apply_pairs<false>,
                       dim3((unsigned)pair_blocks(fp.pblocks, fp.chunks)), dim3(kPairThreads), 0, s,
                       N, fp.pblocks, fp.chunks, fp.chunk, pb.x, srt.seg, srt.nus, srt.X64, v,
                       pb.eps * pb.eps, part, stop);
    const unsigned blocks = (unsigned)((3 * N + 63) / 64 + pb.M);
    hipLaunchKernelGGL(k_apply_stage2, dim3(blocks), dim3(kApplyThreads), 0, s, N, pb.M,
                       fp.chunks, part, 1.0 / (8.0 * kPi * pb.mu), pb.x, pb.body, pb.Y, srt.W, v,
                       y, stop);
  }
  return hipGetLastError();
}

// The same for every system of a batch, Ax at sol, in two launches (96 systems of orders
// 300..6000: about 1.0 ms, as the FP64 rate of the pair sum gives).
hipError_t launch_apply_batch(const BatchSet& bs, int force, hipStream_t s) {
  hipError_t e =
      batch_launch(bs, kBatchPairs, [&](const int64_t* first, int32_t s0, int32_t s1, unsigned g) {
        hipLaunchKernelGGL(k_apply_pairs_batch, dim3(g), dim3(kPairThreads), 0, s, bs.sys, first,
                           s0, s1, force);
      });
  if (e != hipSuccess) return e;
  return batch_launch(bs, kBatchRows, [&](const int64_t* first, int32_t s0, int32_t s1, unsigned g) {
    hipLaunchKernelGGL(k_apply_stage2_batch, dim3(g), dim3(kApplyThreads), 0, s, bs.sys, first, s0,
                       s1, force);
  });
}

int64_t batch_blocks_assemble(int kind, const BatchSys& y) {
  switch (kind) {
    case kBatchRhs: return (std::max(y.n, y.N) + kRhsThreads - 1) / kRhsThreads;
    case kBatchPairs: return pair_blocks(y.pblocks, y.chunks);
    default: return (3 * y.N + 63) / 64 + y.M;   // kBatchRows
  }
}

}  // namespace nrs
