// Device kernels of the hierarchy, smoother, V-cycle and CG (paper §2.1, §2.2, §3.1,
// §4.1), shared by single-instance and batched solves.
//
// A level of a batch holds several independent instances.  Their block rows are
// contiguous "segments"; the segments that are smoothed (active) come first, the
// ones whose coarsest level this is (terminal) last.  Per-instance quantities
// (Lanczos coefficients, lambda_hat, Chebyshev coefficients, CG scalars) are looked
// up from the row by a binary search of the segment offsets.  All reductions are
// deterministic: fixed chunks summed in a fixed order.
#pragma once

#include <cmath>

#include "spmv_core.hpp"

namespace blk {

constexpr int kMaxCheb = 16;
constexpr int kMaxLanczos = 64;

struct LevelScalars {
  double alpha[kMaxLanczos];
  double beta[kMaxLanczos];
  double inv_b, ratio;            // Lanczos: 1 / b_k and b_k / b_(k-1) of the current step
  double lam;                     // lambda_hat
  double coef[1 + 2 * kMaxCheb];  // 1/theta, then (c1, c2) per Chebyshev step
  double tmp[4];
  float coef_f[1 + 2 * kMaxCheb];  // the same coefficients rounded to FP32
};

// Chebyshev coefficient t in the arithmetic type of the smoother
template <class TA>
__device__ __forceinline__ TA cheb_coef(const LevelScalars& S, int t) {
  if constexpr (sizeof(TA) == 4) return S.coef_f[t];
  else return static_cast<TA>(S.coef[t]);
}

// segment of row `row` among off[0..n] (off[0] = 0 <= row < off[n])
__device__ __forceinline__ int seg_of(const int32_t* __restrict__ off, int n, int row) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (off[mid] <= row) lo = mid; else hi = mid;
  }
  return lo;
}

__device__ __forceinline__ uint64_t splitmix64(uint64_t z) {
  z += 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ---------------------------------------------------------------------------
// Segmented dot products.  A chunk is a row range inside one segment; workgroup c
// sums chunk c for every right-hand side q into partial[c * NR + q].
// ---------------------------------------------------------------------------
template <int NR, class T, class TB = T>
__global__ __launch_bounds__(256) void seg_dot_kernel(const T* __restrict__ a, const TB* __restrict__ b,
                                                      const int32_t* __restrict__ lo, const int32_t* __restrict__ hi,
                                                      double* __restrict__ partial) {
  __shared__ double lds[4 * NR];
  const int c = blockIdx.x;
  double acc[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) acc[q] = 0.0;
  for (int i = lo[c] + threadIdx.x; i < hi[c]; i += 256) {
#pragma unroll
    for (int q = 0; q < NR; ++q)
      acc[q] = fmadd(static_cast<double>(a[static_cast<size_t>(i) * NR + q]),
                     static_cast<double>(b[static_cast<size_t>(i) * NR + q]), acc[q]);
  }
#pragma unroll
  for (int q = 0; q < NR; ++q) {
    acc[q] = group_sum<64>(acc[q]);
    if ((threadIdx.x & 63) == 0) lds[(threadIdx.x >> 6) * NR + q] = acc[q];
  }
  __syncthreads();
  if (threadIdx.x < NR) {
    const int q = threadIdx.x;
    partial[static_cast<size_t>(c) * NR + q] = ((lds[q] + lds[NR + q]) + lds[2 * NR + q]) + lds[3 * NR + q];
  }
}

// Output (segment s, rhs q) = sum of partial[c * nr + q] over the chunks c of s,
// workgroup per output, fixed assignment and tree; then op(s, q, sum).
template <class Op>
__global__ __launch_bounds__(256) void seg_finish_kernel(const double* __restrict__ partial,
                                                         const int32_t* __restrict__ seg_ptr, int nr, Op op) {
  __shared__ double lds[4];
  const int sg = blockIdx.x / nr, q = blockIdx.x % nr;
  double v = 0.0;
  for (int c = seg_ptr[sg] + threadIdx.x; c < seg_ptr[sg + 1]; c += 256) v += partial[static_cast<size_t>(c) * nr + q];
  const double s = block_sum_256(v, lds);
  if (threadIdx.x == 0) op(sg, q, s);
}

// Lanczos scalars of segment s: which < 0 -> tmp[0] = sqrt(v); else beta[which] = sqrt(v)
struct OpLzSqrt {
  LevelScalars* sc;
  int which;
  __device__ void operator()(int s, int, double v) const {
    const double r = sqrt(v > 0.0 ? v : 0.0);
    if (which < 0) sc[s].tmp[0] = r; else sc[s].beta[which] = r;
  }
};
struct OpLzAlpha {
  LevelScalars* sc;
  int step;
  __device__ void operator()(int s, int, double v) const { sc[s].alpha[step] = v; }
};
// The refresh's Lanczos keeps its vectors unnormalised, U = b u and Y = b y with
// b = sqrt(U.Y): the norm after step `step` (-1: the start vector's) and the two factors
// the next product needs.  A zero norm counts as 1.
struct OpLzNorm {
  LevelScalars* sc;
  int step;
  __device__ void operator()(int s, int, double v) const {
    LevelScalars& S = sc[s];
    const double r = sqrt(v > 0.0 ? v : 0.0), b = r > 0.0 ? r : 1.0;
    if (step >= 0) S.beta[step] = r;
    S.ratio = step < 0 ? 0.0 : r * S.inv_b;
    S.inv_b = 1.0 / b;
  }
};
// alpha = u.wy from U.wy
struct OpLzDot {
  LevelScalars* sc;
  int step;
  __device__ void operator()(int s, int, double v) const { sc[s].alpha[step] = v * sc[s].inv_b; }
};

// ---------------------------------------------------------------------------
// Block-diagonal inverse (point-block Jacobi, paper §4.1)
// ---------------------------------------------------------------------------
template <int BS, class TM, class TD>
__global__ __launch_bounds__(256) void dinv_kernel(int nbr, const int32_t* __restrict__ rp, const int32_t* __restrict__ ci,
                            const TM* __restrict__ val, TD* __restrict__ dinv, int32_t* __restrict__ diag_idx,
                            int* flag) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nbr) return;
  // the diagonal block: binary search in the row's ascending column indices
  int kd = -1;
  for (int lo = rp[r], hi = rp[r + 1]; lo < hi;) {
    const int mid = (lo + hi) >> 1;
    const int c = ci[mid];
    if (c == r) { kd = mid; break; }
    if (c < r) lo = mid + 1; else hi = mid;
  }
  diag_idx[r] = kd;
  double a[BS][2 * BS];
#pragma unroll
  for (int i = 0; i < BS; ++i) {
#pragma unroll
    for (int j = 0; j < BS; ++j) {
      a[i][j] = kd >= 0 ? ld<double>(val + static_cast<size_t>(kd) * BS * BS + i * BS + j) : 0.0;
      a[i][BS + j] = (i == j) ? 1.0 : 0.0;
    }
  }
  // Gauss-Jordan with partial pivoting, fully unrolled: the pivot row is exchanged with
  // row c by selects, so every index is a compile-time constant and the array stays in
  // registers (indexing it by the run-time pivot put it in scratch memory)
  bool ok = kd >= 0;
#pragma unroll
  for (int c = 0; c < BS; ++c) {
    int p = c;
    double best = fabs(a[c][c]);
#pragma unroll
    for (int i = c + 1; i < BS; ++i)
      if (fabs(a[i][c]) > best) { best = fabs(a[i][c]); p = i; }
    ok = ok && best > 0.0;
#pragma unroll
    for (int i = c + 1; i < BS; ++i) {
      const bool sw = i == p;
#pragma unroll
      for (int j = 0; j < 2 * BS; ++j) {
        const double t = a[c][j];
        a[c][j] = sw ? a[i][j] : t;
        a[i][j] = sw ? t : a[i][j];
      }
    }
    const double inv = ok ? 1.0 / a[c][c] : 0.0;
#pragma unroll
    for (int j = 0; j < 2 * BS; ++j) a[c][j] *= inv;
#pragma unroll
    for (int i = 0; i < BS; ++i) {
      if (i == c) continue;
      const double f = a[i][c];
#pragma unroll
      for (int j = 0; j < 2 * BS; ++j) a[i][j] -= f * a[c][j];
    }
  }
  if (!ok) atomicExch(flag, 1);
  TD* o = dinv + static_cast<size_t>(r) * BS * BS;
  for (int i = 0; i < BS; ++i)
    for (int j = 0; j < BS; ++j) o[i * BS + j] = static_cast<TD>(ok ? a[i][BS + j] : (i == j ? 1.0 : 0.0));
}

// ---------------------------------------------------------------------------
// Lanczos (D inner product on D^-1 A), one recurrence per active segment.
// sc points at this level's first LevelScalars; segment s uses sc[s].
// ---------------------------------------------------------------------------

// v from splitmix64 of the instance-local scalar index, Dv = diag-block(A) v; workgroup c
// takes the rows of chunk c and, with partial set, sums their v.Dv
template <int BS, class TM, class TV>
__global__ __launch_bounds__(256) void lanczos_start_kernel(const int32_t* __restrict__ lo,
                                                            const int32_t* __restrict__ hi,
                                                            const int32_t* __restrict__ off, int nseg, uint64_t seed,
                                                            const TM* __restrict__ val,
                                                            const int32_t* __restrict__ diag_idx, TV* __restrict__ v,
                                                            TV* __restrict__ Dv, double* __restrict__ partial) {
  __shared__ double lds[4];
  const int c = blockIdx.x, r1 = hi[c] / BS;
  double acc = 0.0;
  for (int r = lo[c] / BS + threadIdx.x; r < r1; r += 256) {
    const int sg = seg_of(off, nseg, r);
    const int64_t local = static_cast<int64_t>(r - off[sg]) * BS;
    double vv[BS];
    for (int j = 0; j < BS; ++j) {
      const uint64_t z = splitmix64(seed ^ static_cast<uint64_t>(local + j));
      vv[j] = static_cast<double>(static_cast<TV>(2.0 * (static_cast<double>(z >> 11) * 0x1.0p-53) - 1.0));
      v[static_cast<size_t>(r) * BS + j] = static_cast<TV>(vv[j]);
    }
    const int kd = diag_idx[r];
    for (int i = 0; i < BS; ++i) {
      double sv = 0.0;
      if (kd >= 0)
        for (int j = 0; j < BS; ++j) sv += ld<double>(val + static_cast<size_t>(kd) * BS * BS + i * BS + j) * vv[j];
      const TV dv = static_cast<TV>(sv);
      Dv[static_cast<size_t>(r) * BS + i] = dv;
      acc = fmadd(vv[i], static_cast<double>(dv), acc);
    }
  }
  if (partial) {
    const double t = block_sum_256(acc, lds);
    if (threadIdx.x == 0) partial[c] = t;
  }
}

// (ao, bo) = (a, b) / s_seg with s_seg = sc[seg].tmp[0] (start) or sc[seg].beta[step]
template <int BS, class TV>
__global__ void lanczos_scale_kernel(int nbr, const int32_t* __restrict__ off, int nseg,
                                     const LevelScalars* __restrict__ sc, int which, const TV* __restrict__ a,
                                     const TV* __restrict__ b, TV* __restrict__ ao, TV* __restrict__ bo) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nbr) return;
  const int sg = seg_of(off, nseg, r);
  double s = which < 0 ? sc[sg].tmp[0] : sc[sg].beta[which];
  if (!(s > 0.0)) s = 1.0;
  const double inv = 1.0 / s;
  for (int j = 0; j < BS; ++j) {
    const size_t o = static_cast<size_t>(r) * BS + j;
    ao[o] = static_cast<TV>(static_cast<double>(a[o]) * inv);
    bo[o] = static_cast<TV>(static_cast<double>(b[o]) * inv);
  }
}

// wy -= alpha y ; U = Dinv wy ; partial[c] = U.wy over the rows of chunk c (y = Y / b).
// One pass over wy, Y and Dinv: the norm's dot product reads nothing again.
template <int BS, class TV>
__global__ __launch_bounds__(256) void lanczos_orth_kernel(const int32_t* __restrict__ lo,
                                                           const int32_t* __restrict__ hi,
                                                           const int32_t* __restrict__ off, int nseg,
                                                           const LevelScalars* __restrict__ sc, int step,
                                                           const TV* __restrict__ Y, TV* __restrict__ wy,
                                                           const TV* __restrict__ dinv, TV* __restrict__ U,
                                                           double* __restrict__ partial) {
  __shared__ double lds[4];
  const int c = blockIdx.x, r0 = lo[c] / BS, r1 = hi[c] / BS;
  const LevelScalars& S = sc[seg_of(off, nseg, r0)];  // a chunk lies in one segment
  const double al = S.alpha[step] * S.inv_b;
  double acc = 0.0;
  for (int r = r0 + threadIdx.x; r < r1; r += 256) {
    double w[BS];
    for (int j = 0; j < BS; ++j) {
      const size_t o = static_cast<size_t>(r) * BS + j;
      const TV wt = static_cast<TV>(static_cast<double>(wy[o]) - al * static_cast<double>(Y[o]));
      wy[o] = wt;
      w[j] = static_cast<double>(wt);
    }
    const TV* D = dinv + static_cast<size_t>(r) * BS * BS;
    for (int i = 0; i < BS; ++i) {
      double z = 0.0;
      for (int j = 0; j < BS; ++j) z += static_cast<double>(D[i * BS + j]) * w[j];
      const TV u = static_cast<TV>(z);
      U[static_cast<size_t>(r) * BS + i] = u;
      acc = fmadd(static_cast<double>(u), w[i], acc);
    }
  }
  const double t = block_sum_256(acc, lds);
  if (threadIdx.x == 0) partial[c] = t;
}

// SpMV epilogue of one Lanczos step on the unnormalised vectors: wy = (A U) / b_k -
// b_k y_(k-1), in place over Y_(k-1) (no previous vector on step 0).  With DOT (one
// segment), also the partial sums of U.wy.  One right-hand side, BR <= G: lane i < BR owns
// output i.
template <class TV, class TA, bool DOT>
struct EpiLanczos {
  static constexpr bool kReduce = DOT;
  const TV* U;
  TV* wy;
  const LevelScalars* sc;
  const int32_t* off;
  int nseg;
  int step;
  double* partial = nullptr;
  template <int BR, int NR, int G>
  __device__ __forceinline__ RowVals<double, 4> prefetch(bool active, int row) const {
    static_assert(lane_owned<BR * NR, G>(), "Lanczos epilogue expects BR * NR <= G");
    RowVals<double, 4> p;
#pragma unroll
    for (int t = 0; t < 4; ++t) p.v[t] = 0.0;
    const int lane = static_cast<int>(threadIdx.x) % G;
    if (active && lane < BR * NR) {
      const LevelScalars& S = sc[DOT ? 0 : seg_of(off, nseg, row)];
      const size_t o = static_cast<size_t>(row) * (BR * NR) + lane;
      p.v[0] = S.inv_b;
      if (step > 0) {
        p.v[1] = S.ratio;
        p.v[2] = static_cast<double>(wy[o]);
      }
      if (DOT) p.v[3] = static_cast<double>(U[o]);
    }
    return p;
  }
  template <int BR, int NR, int G>
  __device__ __forceinline__ double apply(bool active, int row, int lane, const TA (&s)[BR * NR],
                                          const RowVals<double, 4>& pre) const {
    if (!active || lane >= BR * NR) return 0.0;
    const TV w = static_cast<TV>(static_cast<double>(pick<BR * NR>(s, lane)) * pre.v[0] - pre.v[1] * pre.v[2]);
    wy[static_cast<size_t>(row) * (BR * NR) + lane] = w;
    return DOT ? pre.v[3] * static_cast<double>(w) : 0.0;
  }
};

// Largest eigenvalue of each segment's tridiagonal T_k by Sturm counts, then the
// Chebyshev coefficients (Saad, Alg. 12.1) for [lo*lam, hi*lam].  One wave per segment: its
// 64 lanes count at 64 points of the interval, which narrows it 65 times a round, so ten
// rounds of k dependent divisions take the place of bisection's fifty (66 -> 12 us).
__global__ __launch_bounds__(64) void lanczos_finish_kernel(LevelScalars* sc, int k, const double* user_lam, double lo,
                                                            double hi, int degree) {
  const int sg = blockIdx.x, lane = threadIdx.x;
  LevelScalars* S = sc + sg;
  double lam;
  if (user_lam != nullptr) {
    lam = user_lam[sg];
  } else {
    __shared__ double al[kMaxLanczos], b2[kMaxLanczos];
    int m = k;
    for (int j = 0; j < k - 1; ++j)
      if (!(S->beta[j] > 0.0)) { m = j + 1; break; }
    if (lane < m) {
      al[lane] = S->alpha[lane];
      b2[lane] = lane < m - 1 ? S->beta[lane] * S->beta[lane] : 0.0;
    }
    double gl = 1e300, gh = -1e300;
    for (int i = 0; i < m; ++i) {
      const double o = (i > 0 ? fabs(S->beta[i - 1]) : 0.0) + (i < m - 1 ? fabs(S->beta[i]) : 0.0);
      gl = fmin(gl, S->alpha[i] - o);
      gh = fmax(gh, S->alpha[i] + o);
    }
    __syncthreads();
    double a = gl, b = gh;
    for (int it = 0; it < 64; ++it) {
      const double x = a + (b - a) * ((lane + 1) * (1.0 / 65.0));
      const bool inside = x > a && x < b;
      if (__ballot(inside) == 0) {  // the points round to the ends: bisect what is left
        const double mid = 0.5 * (a + b);
        if (!(mid > a && mid < b)) break;
      }
      const double t = __ballot(inside) == 0 ? 0.5 * (a + b) : x;
      int cnt = 0;
      double q = al[0] - t;
      if (q < 0) cnt++;
      for (int i = 1; i < m; ++i) {
        const double qq = (q != 0.0) ? q : 1e-300;
        q = al[i] - t - b2[i - 1] / qq;
        if (q < 0) cnt++;
      }
      // the points rise with the lane: the first one above every eigenvalue ends the interval
      const unsigned long long above = __ballot(t >= b || (t > a && cnt == m));
      const int f = above ? __ffsll(above) - 1 : 64;
      const double bn = __shfl(t, f < 64 ? f : 63), an = __shfl(t, f > 0 ? f - 1 : 0);
      if (f < 64) b = fmin(b, bn);
      if (f > 0) a = fmax(a, an);
    }
    lam = 0.5 * (a + b);
  }
  if (lane != 0) return;
  S->lam = lam;
  const double ea = lo * lam, eb = hi * lam;
  const double theta = 0.5 * (eb + ea), delta = 0.5 * (eb - ea);
  const double sigma = theta / delta;
  double rho = 1.0 / sigma;
  S->coef[0] = 1.0 / theta;
  for (int t = 1; t < degree; ++t) {
    const double rho1 = 1.0 / (2.0 * sigma - rho);
    S->coef[1 + 2 * (t - 1)] = rho1 * rho;
    S->coef[2 + 2 * (t - 1)] = 2.0 * rho1 / delta;
    rho = rho1;
  }
  for (int t = 0; t < 2 * degree - 1; ++t) S->coef_f[t] = static_cast<float>(S->coef[t]);
}

// ---------------------------------------------------------------------------
// Chebyshev / point-block Jacobi (paper §4.1 pbjacobi inside Saad's Chebyshev)
// ---------------------------------------------------------------------------

// d = Dinv f / theta_seg (zero-guess start), NR right-hand sides; row_seg (NULL for
// one segment) gives the segment of each row
template <int BS, int NR, class TV>
__global__ void cheb0_kernel(int nbr, const uint16_t* __restrict__ row_seg, const LevelScalars* __restrict__ sc,
                             const TV* __restrict__ f, const TV* __restrict__ dinv, TV* __restrict__ out) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nbr) return;
  const TV it = cheb_coef<TV>(sc[row_seg ? row_seg[r] : 0], 0);
  TV fv[BS * NR];
  for (int t = 0; t < BS * NR; ++t) fv[t] = f[static_cast<size_t>(r) * BS * NR + t];
  const TV* D = dinv + static_cast<size_t>(r) * BS * BS;
  for (int i = 0; i < BS; ++i)
    for (int q = 0; q < NR; ++q) {
      TV z = 0;
      for (int j = 0; j < BS; ++j) z = fmadd(D[i * BS + j], fv[j * NR + q], z);
      out[static_cast<size_t>(r) * BS * NR + i * NR + q] = z * it;
    }
}

enum SmoothMode { M_RESID = 0, M_INITX = 1, M_STEP = 2 };

// s = A * (gathered vector); per-row Chebyshev coefficients from the row's segment.
//   RESID : r_out = f - s
//   INITX : r = f - s ; d = Dinv r / theta ; x_out = x_in + d   (writes r, d, x_out)
//   STEP  : r = f - s (f = current r) ; d' = c1 d_in + c2 Dinv r ; x_out = x_in + d'
// One right-hand side: lane i < BR owns output i; it loads f_i, d_i, x_i, row i of
// Dinv and the two coefficients before the product (their latency then hides behind
// the block loads), and the residual entries reach the other owners by shuffles.
// Eight right-hand sides: a lane holds its columns of all BR entries, so D^-1 r stays
// inside the lane; its operands are loaded after the product.
template <int MODE, class TV, class TA>
struct EpiSmooth {
  static constexpr bool kReduce = false;
  const TV* f;
  TV* r_out;
  const TV* d_in;
  TV* d_out;
  const TV* x_in;
  TV* x_out;
  const TV* dinv;
  const LevelScalars* sc;
  const uint16_t* row_seg;  // segment of each row, NULL for one segment
  int step;
  double* partial = nullptr;

  template <int BR, int NR, int G>
  static constexpr int pre_len() { return 3 + BR; }

  __device__ __forceinline__ const LevelScalars& scal(int row) const { return sc[row_seg ? row_seg[row] : 0]; }

  // own-row operands of one right-hand side, all in the arithmetic type (the
  // coefficients come pre-rounded), so nothing has to be converted, and waited for,
  // before the product
  template <int BR, int NR, int G>
  struct Pre {
    RowVals<TA, 3 + BR> a;
    TA c1, c2;
  };

  // The loads are unconditional (lanes >= BR and rows past the end read valid
  // addresses of the same row / row 0 and their values are never stored), so no
  // branch separates them from the product's loads.
  template <int BR, int NR, int G>
  __device__ __forceinline__ Pre<BR, NR, G> prefetch(bool active, int row) const {
    static_assert(NR == 1 && lane_owned<BR, G>(), "one right-hand side with BR <= G");
    Pre<BR, NR, G> p;
#pragma unroll
    for (int t = 0; t < 3 + BR; ++t) p.a.v[t] = TA(0);
    p.c1 = TA(0);
    p.c2 = TA(0);
    const int lane = min(static_cast<int>(threadIdx.x) % G, BR - 1);
    const int rr = active ? row : 0;
    const size_t o = static_cast<size_t>(rr) * BR + lane;
    p.a.v[0] = ld<TA>(f + o);
    if (MODE == M_STEP) p.a.v[1] = ld<TA>(d_in + o);
    if (MODE != M_RESID) {
      p.a.v[2] = ld<TA>(x_in + o);
      const TV* D = dinv + static_cast<size_t>(rr) * (BR * BR) + lane * BR;
#pragma unroll
      for (int j = 0; j < BR; ++j) p.a.v[3 + j] = ld<TA>(D + j);
      const LevelScalars& S = scal(rr);
      if (MODE == M_INITX) {
        p.c2 = cheb_coef<TA>(S, 0);
      } else {
        p.c1 = cheb_coef<TA>(S, 1 + 2 * step);
        p.c2 = cheb_coef<TA>(S, 2 + 2 * step);
      }
    }
    return p;
  }

  template <int BR, int NR, int G>
  __device__ __forceinline__ double apply(bool active, int row, int lane, const TA (&s)[BR * NR],
                                          const Pre<BR, NR, G>& pre) const {
    if (!active) return 0.0;
    // every lane of the group takes part in the shuffles; lanes >= BR carry zeros
    const TA r = pre.a.v[0] - pick<BR>(s, lane < BR ? lane : 0);
    const size_t o = static_cast<size_t>(row) * BR + lane;
    if (MODE == M_RESID) {
      if (lane < BR) r_out[o] = static_cast<TV>(r);
      return 0.0;
    }
    TA z = TA(0);
#pragma unroll
    for (int j = 0; j < BR; ++j) z = fmadd(pre.a.v[3 + j], __shfl(r, j, G), z);
    TA dn = pre.c2 * z;
    if (MODE == M_STEP) dn = fmadd(pre.c1, pre.a.v[1], dn);
    if (lane < BR) {
      x_out[o] = static_cast<TV>(pre.a.v[2] + dn);
      if (r_out) r_out[o] = static_cast<TV>(r);
      if (d_out) d_out[o] = static_cast<TV>(dn);
    }
    return 0.0;
  }

  // eight right-hand sides: every lane holds its CPL columns of the row's BR sums and
  // forms the residual of all of them; slot `slot` finishes rows slot, slot + S, ...
  template <int BR, int S, int CPL>
  __device__ __forceinline__ void apply8(int row, int slot, int cl, const TA (&s)[BR][CPL]) const {
    const size_t base = static_cast<size_t>(row) * (BR * 8) + cl * CPL;
    TA r[BR][CPL];
#pragma unroll
    for (int i = 0; i < BR; ++i) {
      if (MODE == M_RESID && i % S != slot) continue;
      TA fv[CPL];
      ld_cols<TA>(f + base + i * 8, fv);
#pragma unroll
      for (int q = 0; q < CPL; ++q) r[i][q] = fv[q] - s[i][q];
      if (MODE == M_RESID) st_cols(r_out + base + i * 8, r[i]);
    }
    if (MODE == M_RESID) return;
    // r_out may be f: every lane of the row has read f before any of them stores
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const LevelScalars& L = scal(row);
    const TA c1 = MODE == M_STEP ? cheb_coef<TA>(L, 1 + 2 * step) : TA(0);
    const TA c2 = MODE == M_STEP ? cheb_coef<TA>(L, 2 + 2 * step) : cheb_coef<TA>(L, 0);
    const TV* D = dinv + static_cast<size_t>(row) * (BR * BR);
#pragma unroll
    for (int i = 0; i < BR; ++i) {
      if (i % S != slot) continue;
      const size_t o = base + i * 8;
      TA xi[CPL], di[CPL], dn[CPL];
      ld_cols<TA>(x_in + o, xi);
      if (MODE == M_STEP) ld_cols<TA>(d_in + o, di);
#pragma unroll
      for (int q = 0; q < CPL; ++q) {
        TA z = TA(0);
#pragma unroll
        for (int j = 0; j < BR; ++j) z = fmadd(ld<TA>(D + i * BR + j), r[j][q], z);
        dn[q] = c2 * z;
        if (MODE == M_STEP) dn[q] = fmadd(c1, di[q], dn[q]);
        xi[q] += dn[q];
      }
      st_cols(x_out + o, xi);
      if (r_out) st_cols(r_out + o, r[i]);
      if (d_out) st_cols(d_out + o, dn);
    }
  }
};

// ---------------------------------------------------------------------------
// Prolongator smoothing (cold setup, paper §2.2) with the weight omega of the row's
// segment (omega_scale / lambda_hat, or a learned weight):
//   P_ib = [agg(i) == b] P~_i - omega Dinv_i sum_{j in A_i, agg(j) == b} A_ij P~_j
// ---------------------------------------------------------------------------
template <int BS, int NC>
__global__ void smooth_p_kernel(int nbr, const int32_t* __restrict__ a_rp, const int32_t* __restrict__ a_ci,
                                const double* __restrict__ a_v, const int32_t* __restrict__ agg,
                                const double* __restrict__ pt, const double* __restrict__ dinv,
                                const int32_t* __restrict__ off, int nseg, const double* __restrict__ omega_seg,
                                const int32_t* __restrict__ p_rp, const int32_t* __restrict__ p_ci,
                                double* __restrict__ p_v) {
  const int64_t gidx = blockIdx.x * static_cast<int64_t>(blockDim.x) + threadIdx.x;
  const int64_t nnz = p_rp[nbr];
  if (gidx >= nnz) return;
  int lo = 0, hi = nbr;
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (p_rp[mid] <= gidx) lo = mid; else hi = mid;
  }
  const int i = lo;
  const int b = p_ci[gidx];
  double acc[BS * NC];
  for (int t = 0; t < BS * NC; ++t) acc[t] = 0.0;
  for (int k = a_rp[i]; k < a_rp[i + 1]; ++k) {
    const int j = a_ci[k];
    if (agg[j] != b) continue;
    const double* ab = a_v + static_cast<size_t>(k) * BS * BS;
    const double* pb = pt + static_cast<size_t>(j) * BS * NC;
    for (int r = 0; r < BS; ++r)
      for (int m = 0; m < BS; ++m) {
        const double a = ab[r * BS + m];
        for (int c = 0; c < NC; ++c) acc[r * NC + c] += a * pb[m * NC + c];
      }
  }
  const double omega = omega_seg[seg_of(off, nseg, i)];
  const double* D = dinv + static_cast<size_t>(i) * BS * BS;
  double* o = p_v + static_cast<size_t>(gidx) * BS * NC;
  for (int r = 0; r < BS; ++r)
    for (int c = 0; c < NC; ++c) {
      double z = 0.0;
      for (int m = 0; m < BS; ++m) z += D[r * BS + m] * acc[m * NC + c];
      const double base = (agg[i] == b) ? pt[static_cast<size_t>(i) * BS * NC + r * NC + c] : 0.0;
      o[r * NC + c] = base - omega * z;
    }
}

// ---------------------------------------------------------------------------
// Dense coarse solves (FP64) of all terminal segments of a level at once:
// expansion, then the inverse Cholesky factor panel by panel.  Segment t (blockIdx.y) owns
// an n_t x n_t row-major matrix at mats + mat_off[t]; tiles of kT x kT, and tiles
// that stick out of the matrix act as identity-padded.
// ---------------------------------------------------------------------------
constexpr int kT = 32;

// block rows [row0_t, row0_t + nrows_t) of the level matrix, columns shifted by row0_t
template <class TM>
__global__ void expand_dense_kernel(const int32_t* __restrict__ seg_row0, const int32_t* __restrict__ seg_nrows,
                                    const int64_t* __restrict__ mat_off, int bs, const int32_t* __restrict__ rp,
                                    const int32_t* __restrict__ ci, const TM* __restrict__ val,
                                    double* __restrict__ mats) {
  const int t = blockIdx.y;
  const int r = blockIdx.x;
  const int nr = seg_nrows[t], r0 = seg_row0[t];
  if (r >= nr) return;
  const int n = nr * bs;
  double* M = mats + mat_off[t];
  for (int k = rp[r0 + r]; k < rp[r0 + r + 1]; ++k) {
    const int c = ci[k] - r0;
    if (c < 0 || c >= nr) continue;
    for (int e = threadIdx.x; e < bs * bs; e += blockDim.x) {
      const int i = e / bs, j = e % bs;
      M[static_cast<size_t>(r * bs + i) * n + c * bs + j] = ld<double>(val + static_cast<size_t>(k) * bs * bs + e);
    }
  }
}

__device__ __forceinline__ double mat_at(const double* M, int n, int i, int j) {
  if (i < n && j < n) return M[static_cast<size_t>(i) * n + j];
  return (i == j) ? 1.0 : 0.0;
}

__device__ __forceinline__ int tiles_of(int n) { return (n + kT - 1) / kT; }

using f64x4 = double __attribute__((ext_vector_type(4)));

// Quadrant `w` (16 x 16, one per wave) of X W^T for 32 x 32 tiles in LDS, added to or
// taken from c: eight v_mfma_f64_16x16x4_f64.  Lane l feeds X[i][q] and W[i][q] of row
// l % 16 at q = l / 16 and ends with rows l / 16 + 4 v, column l % 16 of the quadrant.
template <bool kSub>
__device__ __forceinline__ f64x4 mul_nt(const double (*X)[kT + 1], const double (*W)[kT + 1], int w, int l, f64x4 c) {
  const int i = 16 * (w >> 1) + (l & 15), j = 16 * (w & 1) + (l & 15), q0 = l >> 4;
#pragma unroll
  for (int q = 0; q < kT; q += 4) {
    const double a = X[i][q + q0];
    c = __builtin_amdgcn_mfma_f64_16x16x4f64(kSub ? -a : a, W[j][q + q0], c, 0, 0, 0);
  }
  return c;
}

__device__ __forceinline__ double read_lane(double v, int lane) {
  union { double d; int i[2]; } u;
  u.d = v;
  u.i[0] = __builtin_amdgcn_readlane(u.i[0], lane);
  u.i[1] = __builtin_amdgcn_readlane(u.i[1], lane);
  return u.d;
}

// Inverse Cholesky factor of the SPD tile D (lower triangle read) by one wave, in
// registers: lane r < 32 holds row r of D, lane 32 + j column j of the identity.  Step c
// scales entry c by 1/L_cc and takes L_jc times it from entry j > c in both halves: the
// rows become L, the columns L^-1.  No barrier and no division (1/sqrt from the hardware's
// estimate, 5e-8 off, by one third-order step).  A non-positive pivot sets *flag and counts as 1.
__device__ __forceinline__ void invert_tile(const double (*D)[kT + 1], double (*Y)[kT + 1], int* flag) {
  const int l = threadIdx.x & 63, r = l & 31;
  double v[kT];
#pragma unroll
  for (int j = 0; j < kT; ++j) v[j] = l < 32 ? D[r][j] : (j == r ? 1.0 : 0.0);
#pragma unroll
  for (int c = 0; c < kT; ++c) {
    double d = read_lane(v[c], c);
    if (!(d > 0.0)) {
      if (l == 0) *flag = 1;
      d = 1.0;
    }
    double y = __builtin_amdgcn_rsq(d);
    const double e = fma(-d * y, y, 1.0);
    y = fma(y * e, fma(e, 0.375, 0.5), y);
    const double m = v[c] * y;
    v[c] = m;
#pragma unroll
    for (int j = c + 1; j < kT; ++j) v[j] = fma(-m, read_lane(m, j), v[j]);
  }
  if (l >= 32) {
#pragma unroll
    for (int i = 0; i < kT; ++i) Y[i][r] = v[i];
  }
}

// Inverse Cholesky factor Y = L^-1 (and Y^T) of every terminal segment's matrix, one
// launch per 32-column panel k (and one, k = -1, for the first diagonal tile).  The
// factorisation and the forward substitution on the identity advance together: tile
// (a, b), b > k, of M holds A's lower part for a >= b and, for a <= k, the transposed
// right-hand side S_ba^T, and step k takes V_a V_b^T from it, with V_a = M_ak L_kk^-T
// (V_k = L_kk^-T).  V_a is L_ak below the diagonal and Y_ka^T above it; nothing else of L
// is ever stored.  Every workgroup forms the V it needs itself from the column k of M and
// the inverse diagonal tile, which the previous launch left in Y; the one with tile
// (k + 1, k + 1), first in the grid, also inverts it for the next launch.  Within a launch
// no tile is read that another workgroup writes.
// The chain of diagonal tiles bounds it: 13 us a panel, half of it the tile's inversion;
// the products run on the matrix cores.  750 dofs (24 panels): 0.33 ms, against 2.28 ms
// for separate panel, update, inverse and transposition launches with the tiles
// factored in LDS.
__global__ __launch_bounds__(256) void chol_inverse_kernel(double* __restrict__ mats, double* __restrict__ Ys,
                                                           double* __restrict__ Yts,
                                                           const int64_t* __restrict__ mat_off,
                                                           const int32_t* __restrict__ ndof, int k, int* flag) {
  __shared__ double W[kT][kT + 1], X[kT][kT + 1], Z[kT][kT + 1], Va[kT][kT + 1], Vb[kT][kT + 1];
  const int n = ndof[blockIdx.y];
  const int nt = tiles_of(n);
  if (k >= nt) return;  // uniform over the block, as every return below
  double* M = mats + mat_off[blockIdx.y];
  double* Y = Ys + mat_off[blockIdx.y];
  double* Yt = Yts + mat_off[blockIdx.y];
  const int tid = threadIdx.x, w = tid >> 6, l = tid & 63;
  auto load = [&](double (*T)[kT + 1], const double* P, int ti, int tj) {
#pragma unroll
    for (int e = tid; e < kT * kT; e += 256) T[e / kT][e % kT] = mat_at(P, n, ti * kT + e / kT, tj * kT + e % kT);
  };
  auto store = [&](double* P, const double (*T)[kT + 1], int ti, int tj, bool transposed) {
#pragma unroll
    for (int e = tid; e < kT * kT; e += 256) {
      const int i = e / kT, j = e % kT;
      if (ti * kT + i < n && tj * kT + j < n)
        P[static_cast<size_t>(ti * kT + i) * n + tj * kT + j] = transposed ? T[j][i] : T[i][j];
    }
  };
  // the wave's quadrant of a tile, element v
  auto qrow = [&](int v) { return 16 * (w >> 1) + (l >> 4) + 4 * v; };
  const int qcol = 16 * (w & 1) + (l & 15);
  auto put = [&](double (*T)[kT + 1], const f64x4& c) {
#pragma unroll
    for (int v = 0; v < 4; ++v) T[qrow(v)][qcol] = c[v];
  };
  // which tile: the trailing lower ones row by row, then the right-hand sides, then the
  // finished row k of Y
  const int m = nt - k - 1, n_low = k < 0 ? 1 : m * (m + 1) / 2, n_rhs = k < 0 ? 0 : m * (k + 1);
  int a, b, t = blockIdx.x;
  if (t < n_low) {
    int i = 0;
    while (t > i) t -= ++i;
    a = k + 1 + i;
    b = k + 1 + t;
  } else if (t < n_low + n_rhs) {
    a = (t - n_low) % (k + 1);
    b = k + 1 + (t - n_low) / (k + 1);
  } else if (k >= 0 && t < n_low + n_rhs + k) {
    a = t - n_low - n_rhs;
    b = k;
  } else {
    return;
  }
  const bool last = b == k;               // V_a itself is the result
  const bool diag = a == k + 1 && b == a;  // the next diagonal tile
  const f64x4 zero = {0.0, 0.0, 0.0, 0.0};
  f64x4 c = zero;
  if (!last && a != k) {
#pragma unroll
    for (int v = 0; v < 4; ++v) c[v] = mat_at(M, n, a * kT + qrow(v), b * kT + qcol);
  }
  if (k >= 0) {
    load(W, Y, k, k);
    if (a == k) load(Va, Yt, k, k);
    else load(X, M, a, k);
    if (!last && b != a) load(Z, M, b, k);
    __syncthreads();
    if (a != k) put(Va, mul_nt<false>(X, W, w, l, zero));
    if (!last && b != a) put(Vb, mul_nt<false>(Z, W, w, l, zero));
    __syncthreads();
    if (last) {
      store(Yt, Va, a, k, false);
      store(Y, Va, k, a, true);
      return;
    }
    c = mul_nt<true>(Va, b != a ? Vb : Va, w, l, c);
  }
  if (diag) {
    put(X, c);
    __syncthreads();
    if (w == 0) invert_tile(X, Z, flag);
    __syncthreads();
    store(Y, Z, a, a, false);
    store(Yt, Z, a, a, true);
    return;
  }
#pragma unroll
  for (int v = 0; v < 4; ++v) {
    const int i = a * kT + qrow(v), j = b * kT + qcol;
    if (i < n && j < n) M[static_cast<size_t>(i) * n + j] = c[v];
  }
}

// y[seg] = M_seg x[seg] for every terminal segment of a level; one wave per row.
// seg t covers scalar rows [dof_off[t], dof_off[t+1]) of the level vectors (relative
// to dof0), its n x n matrix starts at mat_off[t]; row i uses columns [0, i] (lower)
// or [i, n) (upper).
template <int NR, class TI, class TO>
__global__ __launch_bounds__(256) void dense_tri_batched_kernel(const double* __restrict__ mats,
                                                                const int64_t* __restrict__ mat_off,
                                                                const int32_t* __restrict__ dof_off, int nseg,
                                                                int dof0, int upper, const TI* __restrict__ x,
                                                                TO* __restrict__ y) {
  const int grow = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  if (grow >= dof_off[nseg]) return;
  const int t = seg_of(dof_off, nseg, grow);
  const int n = dof_off[t + 1] - dof_off[t];
  const int i = grow - dof_off[t];
  const double* Mr = mats + mat_off[t] + static_cast<int64_t>(i) * n;
  const size_t xb = static_cast<size_t>(dof0 + dof_off[t]) * NR;
  const int lo = upper ? i : 0, hi = upper ? n : i + 1;
  double s[NR];
#pragma unroll
  for (int q = 0; q < NR; ++q) s[q] = 0.0;
  for (int k = lo + lane; k < hi; k += 64) {
    const double m = Mr[k];
#pragma unroll
    for (int q = 0; q < NR; ++q) s[q] = fmadd(m, static_cast<double>(x[xb + static_cast<size_t>(k) * NR + q]), s[q]);
  }
#pragma unroll
  for (int q = 0; q < NR; ++q) s[q] = group_sum<64>(s[q]);
  if (lane < NR) {
    double v = 0.0;
#pragma unroll
    for (int q = 0; q < NR; ++q)
      if (q == lane) v = s[q];
    y[xb + static_cast<size_t>(i) * NR + lane] = static_cast<TO>(v);
  }
}

template <class TI, class TO>
__global__ void cast_vec_kernel(size_t n, const TI* __restrict__ a, TO* __restrict__ b) {
  const size_t g = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
  if (g < n) b[g] = static_cast<TO>(a[g]);
}

// ---------------------------------------------------------------------------
// Single-system CG kernels (fused path)
// ---------------------------------------------------------------------------
// S_RZ / S_RZ1 take turns: r.z of this iteration and of the one before
enum { S_RZ = 0, S_RZ1, S_RR, S_BB, S_FLAG, S_COUNT };

// The sum of n partials (fixed order) in every thread of a 256-thread workgroup.
__device__ __forceinline__ double sum_partials(const double* __restrict__ partial, int n) {
  __shared__ double lds[4];
  __shared__ double all;
  double v = 0.0;
  for (int i = threadIdx.x; i < n; i += 256) v += partial[i];
  const double s = block_sum_256(v, lds);
  if (threadIdx.x == 0) all = s;
  __syncthreads();
  return all;
}

// sc[field] = sum of n partials; the host's copies of it, of r.z and of the flag
__global__ __launch_bounds__(256) void pcg_store_kernel(const double* __restrict__ partial, int n,
                                                        double* __restrict__ sc, int field, int rz,
                                                        double* __restrict__ host) {
  const double s = sum_partials(partial, n);
  if (threadIdx.x == 0) {
    sc[field] = s;
    host[field] = s;
    host[S_RZ] = sc[rz];
    host[S_FLAG] = sc[S_FLAG];
    __threadfence_system();
  }
}

struct EpiPcgW {
  static constexpr bool kReduce = true;
  const double* p;
  double* w;
  double* partial;
  // one right-hand side, lane i < BR owns output i
  template <int BR, int NR, int G>
  __device__ __forceinline__ RowVals<double, 1> prefetch(bool active, int row) const {
    static_assert(lane_owned<BR * NR, G>(), "CG epilogue expects BR * NR <= G");
    RowVals<double, 1> pv;
    const int lane = min(static_cast<int>(threadIdx.x) % G, BR * NR - 1);
    pv.v[0] = p[static_cast<size_t>(active ? row : 0) * (BR * NR) + lane];  // unconditional, see EpiSmooth
    return pv;
  }
  template <int BR, int NR, int G>
  __device__ __forceinline__ double apply(bool active, int row, int lane, const double (&s)[BR * NR],
                                          const RowVals<double, 1>& pre) const {
    if (!active || lane >= BR * NR) return 0.0;
    const double v = pick<BR * NR>(s, lane);
    w[static_cast<size_t>(row) * (BR * NR) + lane] = v;
    return pre.v[0] * v;
  }
};

// x += alpha p, r -= alpha w, partial sums of r.r; with r32 set, also the FP32 copy of r
// that an FP32 V-cycle takes as input (rounded to nearest).  Every workgroup adds the np
// partial sums of p.w itself and forms alpha = r.z / p.w (0, and the flag set, unless
// p.w > 0): a launch for that sum alone took 4 - 5 us.
__global__ __launch_bounds__(256) void pcg_update_kernel(size_t n, const double* __restrict__ pw, int np,
                                                         double* __restrict__ sc, int rz,
                                                         const double* __restrict__ p, const double* __restrict__ w,
                                                         double* __restrict__ x, double* __restrict__ r,
                                                         double* __restrict__ partial, float* __restrict__ r32) {
  __shared__ double lds[4];
  double acc = 0.0;
  const double d = sum_partials(pw, np);
  const double a = d > 0.0 ? sc[rz] / d : 0.0;
  if (!(d > 0.0) && blockIdx.x == 0 && threadIdx.x == 0) sc[S_FLAG] = 1.0;
  for (size_t g = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; g < n;
       g += static_cast<size_t>(gridDim.x) * blockDim.x) {
    x[g] = fmadd(a, p[g], x[g]);
    const double rv = fmadd(-a, w[g], r[g]);
    r[g] = rv;
    if (r32) r32[g] = static_cast<float>(rv);
    acc = fmadd(rv, rv, acc);
  }
  const double t = block_sum_256(acc, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// partial sums of a.b; b may be the FP32 output of an FP32 V-cycle (widened exactly)
template <class TB>
__global__ __launch_bounds__(256) void dot_kernel(size_t n, const double* __restrict__ a, const TB* __restrict__ b,
                                                  double* __restrict__ partial) {
  __shared__ double lds[4];
  double acc = 0.0;
  for (size_t g = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; g < n;
       g += static_cast<size_t>(gridDim.x) * blockDim.x)
    acc = fmadd(a[g], static_cast<double>(b[g]), acc);
  const double t = block_sum_256(acc, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// p = z + beta p, beta = r.z / the previous r.z (old < 0: p = z).  Every workgroup adds the
// np partial sums of r.z itself; the first keeps it as sc[now].
template <class TZ>
__global__ __launch_bounds__(256) void pcg_p_kernel(size_t n, const double* __restrict__ rz, int np,
                                                    double* __restrict__ sc, int old, int now,
                                                    const TZ* __restrict__ z, double* __restrict__ p) {
  const double s = sum_partials(rz, np);
  const double beta = old >= 0 ? s / sc[old] : 0.0;
  if (blockIdx.x == 0 && threadIdx.x == 0) sc[now] = s;
  for (size_t g = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; g < n;
       g += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const double zv = static_cast<double>(z[g]);
    p[g] = old >= 0 ? fmadd(beta, p[g], zv) : zv;
  }
}

__global__ __launch_bounds__(256) void pcg_init_kernel(size_t n, const double* __restrict__ b, double* __restrict__ x,
                                                       double* __restrict__ r, double* __restrict__ partial) {
  __shared__ double lds[4];
  double acc = 0.0;
  for (size_t g = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x; g < n;
       g += static_cast<size_t>(gridDim.x) * blockDim.x) {
    const double v = b[g];
    r[g] = v;
    x[g] = 0.0;
    acc = fmadd(v, v, acc);
  }
  const double t = block_sum_256(acc, lds);
  if (threadIdx.x == 0) partial[blockIdx.x] = t;
}

// ---------------------------------------------------------------------------
// Batched CG: one independent recurrence per (instance, right-hand side).
// Scalars are stored [field][seg * nr + q]; a converged system gets alpha = 0 and
// keeps its x and r.
// ---------------------------------------------------------------------------
enum { B_RZ = 0, B_PW, B_ALPHA, B_RR, B_BETA, B_BB, B_DONE, B_ITS, B_FIELDS };

// Field f of system k = (segment, rhs) lives at bs[f * stride + k].
__device__ __forceinline__ double& bf(double* bs, int stride, int f, int k) { return bs[f * stride + k]; }

// bb = b.b ; start the system (done = 1 when b = 0, = 3 when maxit = 0)
struct OpBInit {
  double* bs;
  int stride, nr, maxit;
  __device__ void operator()(int s, int q, double v) const {
    const int k = s * nr + q;
    bf(bs, stride, B_BB, k) = v;
    bf(bs, stride, B_RR, k) = v;
    bf(bs, stride, B_ITS, k) = 0.0;
    bf(bs, stride, B_ALPHA, k) = 0.0;
    bf(bs, stride, B_BETA, k) = 0.0;
    bf(bs, stride, B_DONE, k) = !(v > 0.0) ? 1.0 : (maxit <= 0 ? 3.0 : 0.0);
  }
};
struct OpBRz0 {
  double* bs;
  int stride, nr;
  __device__ void operator()(int s, int q, double v) const { bf(bs, stride, B_RZ, s * nr + q) = v; }
};
// pw = p.w ; alpha = rz / pw for running systems (breakdown: done = 2)
struct OpBAlpha {
  double* bs;
  int stride, nr;
  __device__ void operator()(int s, int q, double v) const {
    const int k = s * nr + q;
    bf(bs, stride, B_PW, k) = v;
    double a = 0.0;
    if (bf(bs, stride, B_DONE, k) == 0.0) {
      if (!(v > 0.0)) bf(bs, stride, B_DONE, k) = 2.0;
      else a = bf(bs, stride, B_RZ, k) / v;
    }
    bf(bs, stride, B_ALPHA, k) = a;
  }
};
// rr = r.r ; count the update, stop at ||r|| <= rtol ||b|| (done = 1) or maxit (done = 3)
struct OpBRr {
  double* bs;
  int stride, nr, maxit;
  double rtol;
  __device__ void operator()(int s, int q, double v) const {
    const int k = s * nr + q;
    if (bf(bs, stride, B_DONE, k) != 0.0) return;
    bf(bs, stride, B_RR, k) = v;
    const double its = bf(bs, stride, B_ITS, k) + 1.0;
    bf(bs, stride, B_ITS, k) = its;
    if (sqrt(v) <= rtol * sqrt(bf(bs, stride, B_BB, k))) bf(bs, stride, B_DONE, k) = 1.0;
    else if (its >= maxit) bf(bs, stride, B_DONE, k) = 3.0;
  }
};
// rz' = r.z ; beta = rz' / rz for running systems
struct OpBBeta {
  double* bs;
  int stride, nr;
  __device__ void operator()(int s, int q, double v) const {
    const int k = s * nr + q;
    double b = 0.0;
    if (bf(bs, stride, B_DONE, k) == 0.0) {
      b = v / bf(bs, stride, B_RZ, k);
      bf(bs, stride, B_RZ, k) = v;
    }
    bf(bs, stride, B_BETA, k) = b;
  }
};

// stat[0] = systems still running, stat[1] = systems that broke down
__global__ void bpcg_status_kernel(const double* __restrict__ bs, int stride, int nsys, int32_t* __restrict__ stat) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  int run = 0, brk = 0;
  for (int k = 0; k < nsys; ++k) {
    const double d = bs[B_DONE * stride + k];
    run += d == 0.0;
    brk += d == 2.0;
  }
  stat[0] = run;
  stat[1] = brk;
}

// r = b, x = 0
__global__ void bpcg_init_kernel(size_t n, const double* __restrict__ b, double* __restrict__ x,
                                 double* __restrict__ r) {
  const size_t g = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
  if (g >= n) return;
  r[g] = b[g];
  x[g] = 0.0;
}

// The vector updates run over the chunks of the dot products, one workgroup a chunk: thread t
// keeps column t % NR, so a chunk's system is looked up once, and the update of r also gives
// the partial sums of r.r.  Ten systems of 9 - 44 elements an edge, eight right-hand sides,
// FP32 hierarchy: update 56 + 15 us for the dot -> 48, direction 41 -> 23 us; before, every
// element searched its system.  The solve 20.3 -> 19.5 ms with 20 iterations.

// x += alpha p, r -= alpha w per system (alpha = 0: frozen, untouched); with r32 set,
// also the FP32 copy of r that an FP32 V-cycle takes as input; partial sums of r.r
template <int NR>
__global__ __launch_bounds__(256) void bpcg_axpy_kernel(const int32_t* __restrict__ lo, const int32_t* __restrict__ hi,
                                                        const int32_t* __restrict__ off, int nseg,
                                                        const double* __restrict__ bs, int stride,
                                                        const double* __restrict__ p, const double* __restrict__ w,
                                                        double* __restrict__ x, double* __restrict__ r,
                                                        float* __restrict__ r32, double* __restrict__ partial) {
  static_assert(NR == 1 || NR == 8);
  __shared__ double lds[4 * NR];
  const int c = blockIdx.x, q = threadIdx.x % NR;
  const int sg = nseg > 1 ? seg_of(off, nseg, lo[c]) : 0;
  const double a = bs[B_ALPHA * stride + sg * NR + q];
  const size_t end = static_cast<size_t>(hi[c]) * NR;
  double acc = 0.0;
#pragma unroll 4
  for (size_t g = static_cast<size_t>(lo[c]) * NR + threadIdx.x; g < end; g += 256) {
    double rv = r[g];
    if (a != 0.0) {
      x[g] = fmadd(a, p[g], x[g]);
      rv = fmadd(-a, w[g], rv);
      r[g] = rv;
      if (r32) r32[g] = static_cast<float>(rv);
    }
    acc = fmadd(rv, rv, acc);
  }
#pragma unroll
  for (int d = NR; d < 64; d <<= 1) acc += __shfl_xor(acc, d, 64);
  if ((threadIdx.x & 63) < NR) lds[(threadIdx.x >> 6) * NR + q] = acc;
  __syncthreads();
  if (threadIdx.x < NR)
    partial[static_cast<size_t>(c) * NR + q] = ((lds[q] + lds[NR + q]) + lds[2 * NR + q]) + lds[3 * NR + q];
}

// p = z + beta p  (p = z on the first step or when beta = 0)
template <int NR, class TZ>
__global__ __launch_bounds__(256) void bpcg_p_kernel(const int32_t* __restrict__ lo, const int32_t* __restrict__ hi,
                                                     const int32_t* __restrict__ off, int nseg,
                                                     const double* __restrict__ bs, int stride, int use_beta,
                                                     const TZ* __restrict__ z, double* __restrict__ p) {
  const int c = blockIdx.x, q = threadIdx.x % NR;
  double b = 0.0;
  if (use_beta) {
    const int sg = nseg > 1 ? seg_of(off, nseg, lo[c]) : 0;
    b = bs[B_BETA * stride + sg * NR + q];
  }
  const size_t end = static_cast<size_t>(hi[c]) * NR;
#pragma unroll 4
  for (size_t g = static_cast<size_t>(lo[c]) * NR + threadIdx.x; g < end; g += 256) {
    const double v = static_cast<double>(z[g]);
    p[g] = b != 0.0 ? fmadd(b, p[g], v) : v;
  }
}

// ---------------------------------------------------------------------------
// Learned eigenbound support: level features, reference Lanczos with full
// reorthogonalisation (the judge), smoother growth test
// ---------------------------------------------------------------------------
constexpr int kFeatStats = 9;  // sum g, sum g^2, max g, sum h, max h, max d, min d, sum nb, max nb

__device__ __forceinline__ double wave_max(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmax(v, __shfl_xor(v, off, 64));
  return v;
}
__device__ __forceinline__ double wave_min(double v) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v = fmin(v, __shfl_xor(v, off, 64));
  return v;
}

constexpr int kFeatSplit = 8;  // workgroups per chunk of the feature statistics
constexpr int kFeatLanes = 8;  // lanes per block row

// Per slice (an eighth of a chunk) of block rows: g_i = max scalar row of
// |D_i^-1 [A_i1 .. A_in]| summed, h_i = sum_{j != i} ||D_i^-1 A_ij||_F, d_i = ||A_ii||_F,
// nb_i = blocks in the row; partial[slice][kFeatStats] holds the slice's sums / maxima /
// minimum.  Eight lanes share a row's blocks: with a thread per row a level of some
// thousand rows occupied a few workgroups, each with a chain of 27 dependent blocks.
template <int BS, class TM, class TD>
__global__ __launch_bounds__(256) void feature_stats_kernel(const int32_t* __restrict__ rp,
                                                            const int32_t* __restrict__ ci,
                                                            const TM* __restrict__ val, const TD* __restrict__ dinv,
                                                            const int32_t* __restrict__ lo,
                                                            const int32_t* __restrict__ hi,
                                                            double* __restrict__ partial) {
  __shared__ double lsum[5][4];
  __shared__ double lext[4][4];
  const int c = blockIdx.x * kFeatSplit + blockIdx.y;
  const int c0 = lo[blockIdx.x] / BS, c1 = hi[blockIdx.x] / BS;
  const int per = (c1 - c0 + kFeatSplit - 1) / kFeatSplit;
  const int r0 = c0 + static_cast<int>(blockIdx.y) * per, r1 = min(c1, r0 + per);
  const int lane = threadIdx.x % kFeatLanes;
  double sg = 0.0, sg2 = 0.0, mg = 0.0, sh = 0.0, mh = 0.0, md = 0.0, mnd = 1e300, snb = 0.0, mnb = 0.0;
  for (int r = r0 + static_cast<int>(threadIdx.x) / kFeatLanes; r < r1; r += 256 / kFeatLanes) {
    double D[BS * BS];
    for (int t = 0; t < BS * BS; ++t) D[t] = static_cast<double>(dinv[static_cast<size_t>(r) * BS * BS + t]);
    double rows[BS];
    for (int i = 0; i < BS; ++i) rows[i] = 0.0;
    double h = 0.0, d = 0.0;
    for (int k = rp[r] + lane; k < rp[r + 1]; k += kFeatLanes) {
      const TM* a = val + static_cast<size_t>(k) * BS * BS;
      double fro = 0.0;
      for (int i = 0; i < BS; ++i)
        for (int j = 0; j < BS; ++j) {
          double m = 0.0;
          for (int q = 0; q < BS; ++q) m += D[i * BS + q] * ld<double>(a + q * BS + j);
          rows[i] += fabs(m);
          fro += m * m;
        }
      if (ci[k] == r) {
        double dd = 0.0;
        for (int t = 0; t < BS * BS; ++t) dd += ld<double>(a + t) * ld<double>(a + t);
        d = sqrt(dd);
      } else {
        h += sqrt(fro);
      }
    }
#pragma unroll
    for (int i = 0; i < BS; ++i) rows[i] = group_sum<kFeatLanes>(rows[i]);
    h = group_sum<kFeatLanes>(h);
    d = group_sum<kFeatLanes>(d);  // one lane holds the diagonal block
    double g = rows[0];
    for (int i = 1; i < BS; ++i) g = fmax(g, rows[i]);
    const double nb = static_cast<double>(rp[r + 1] - rp[r]);
    if (lane == 0) {
      sg += g;
      sg2 += g * g;
      sh += h;
      snb += nb;
    }
    mg = fmax(mg, g);
    mh = fmax(mh, h);
    md = fmax(md, d);
    mnd = fmin(mnd, d);
    mnb = fmax(mnb, nb);
  }
  const double t0 = block_sum_256(sg, lsum[0]);
  const double t1 = block_sum_256(sg2, lsum[1]);
  const double t3 = block_sum_256(sh, lsum[2]);
  const double t7 = block_sum_256(snb, lsum[3]);
  const int w = threadIdx.x >> 6;
  mg = wave_max(mg);
  mh = wave_max(mh);
  md = wave_max(md);
  mnd = wave_min(mnd);
  mnb = wave_max(mnb);
  if ((threadIdx.x & 63) == 0) {
    lext[0][w] = mg;
    lext[1][w] = mh;
    lext[2][w] = md;
    lext[3][w] = mnd;
    lsum[4][w] = mnb;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    double* o = partial + static_cast<size_t>(c) * kFeatStats;
    o[0] = t0;
    o[1] = t1;
    o[2] = fmax(fmax(lext[0][0], lext[0][1]), fmax(lext[0][2], lext[0][3]));
    o[3] = t3;
    o[4] = fmax(fmax(lext[1][0], lext[1][1]), fmax(lext[1][2], lext[1][3]));
    o[5] = fmax(fmax(lext[2][0], lext[2][1]), fmax(lext[2][2], lext[2][3]));
    o[6] = fmin(fmin(lext[3][0], lext[3][1]), fmin(lext[3][2], lext[3][3]));
    o[7] = t7;
    o[8] = fmax(fmax(lsum[4][0], lsum[4][1]), fmax(lsum[4][2], lsum[4][3]));
  }
}

// Features of segment s (one wave each) from its slices: every lane takes each 64th slice,
// then a fixed tree.
__global__ __launch_bounds__(64) void feature_finish_kernel(const double* __restrict__ partial,
                                                            const int32_t* __restrict__ seg_ptr,
                                                            const int32_t* __restrict__ row_off, int bs, int level,
                                                            float* __restrict__ feat) {
  const int sg = blockIdx.x;
  double st[kFeatStats] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 1e300, 0.0, 0.0};
  for (int c = seg_ptr[sg] * kFeatSplit + threadIdx.x; c < seg_ptr[sg + 1] * kFeatSplit; c += 64) {
    const double* p = partial + static_cast<size_t>(c) * kFeatStats;
    st[0] += p[0];
    st[1] += p[1];
    st[2] = fmax(st[2], p[2]);
    st[3] += p[3];
    st[4] = fmax(st[4], p[4]);
    st[5] = fmax(st[5], p[5]);
    st[6] = fmin(st[6], p[6]);
    st[7] += p[7];
    st[8] = fmax(st[8], p[8]);
  }
  for (int t : {0, 1, 3, 7}) st[t] = group_sum<64>(st[t]);
  for (int t : {2, 4, 5, 8}) st[t] = wave_max(st[t]);
  st[6] = wave_min(st[6]);
  if (threadIdx.x != 0) return;
  const double nr = static_cast<double>(row_off[sg + 1] - row_off[sg]);
  float* f = feat + static_cast<size_t>(sg) * 12;
  const double mean_g = st[0] / nr;
  f[0] = static_cast<float>(log(st[2]));
  f[1] = static_cast<float>(log(mean_g));
  f[2] = static_cast<float>(log(sqrt(st[1] / nr)));
  f[3] = static_cast<float>(log1p(st[4]));
  f[4] = static_cast<float>(log1p(st[3] / nr));
  f[5] = static_cast<float>(log(st[5] / st[6]));
  f[6] = static_cast<float>(st[7] / nr);
  f[7] = static_cast<float>(st[8]);
  f[8] = static_cast<float>(log(nr * bs));
  f[9] = static_cast<float>(level);
  f[10] = static_cast<float>(bs / 6.0);
  f[11] = static_cast<float>(log1p(st[3] / nr) - log(mean_g));
}

// x = (f - mean) / std per feature (model statistics after the parameters)
__global__ void feature_normalize_kernel(int n, const float* __restrict__ feat, const float* __restrict__ stats,
                                         float* __restrict__ x) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= n * 12) return;
  const int j = e % 12;
  x[e] = (feat[e] - stats[j]) / stats[12 + j];
}

// network outputs -> lambda = exp(y0 sd0 + mu0), omega = y1 sd1 + mu1
__global__ void predict_finish_kernel(int n, const float* __restrict__ y, const float* __restrict__ tstats,
                                      double* __restrict__ lam, double* __restrict__ omega) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  lam[i] = exp(static_cast<double>(y[2 * i]) * tstats[2] + tstats[0]);
  omega[i] = static_cast<double>(y[2 * i + 1]) * tstats[3] + tstats[1];
}

// wy -= alpha_seg y + beta_seg y_prev (beta part only when y_prev != NULL)
template <int BS>
__global__ void judge_orth_kernel(int nbr, const int32_t* __restrict__ off, int nseg,
                                  const LevelScalars* __restrict__ sc, int step, const double* __restrict__ y,
                                  const double* __restrict__ y_prev, double* __restrict__ wy) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nbr) return;
  const LevelScalars& S = sc[seg_of(off, nseg, r)];
  const double al = S.alpha[step];
  const double be = y_prev ? S.beta[step - 1] : 0.0;
  for (int j = 0; j < BS; ++j) {
    const size_t o = static_cast<size_t>(r) * BS + j;
    double v = wy[o] - al * y[o];
    if (y_prev) v -= be * y_prev[o];
    wy[o] = v;
  }
}

// wu = Dinv wy
template <int BS, class TD>
__global__ void judge_dinv_kernel(int nbr, const TD* __restrict__ dinv, const double* __restrict__ wy,
                                  double* __restrict__ wu) {
  const int r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= nbr) return;
  const TD* D = dinv + static_cast<size_t>(r) * BS * BS;
  for (int i = 0; i < BS; ++i) {
    double z = 0.0;
    for (int j = 0; j < BS; ++j) z += static_cast<double>(D[i * BS + j]) * wy[static_cast<size_t>(r) * BS + j];
    wu[static_cast<size_t>(r) * BS + i] = z;
  }
}

// partial[c][j] = sum over chunk c of Y_j . w, j < kk (Y_j at Y + j * n)
__global__ __launch_bounds__(256) void multi_dot_kernel(const double* __restrict__ Y, size_t n, int kk,
                                                        const double* __restrict__ w, const int32_t* __restrict__ lo,
                                                        const int32_t* __restrict__ hi, double* __restrict__ partial) {
  __shared__ double lds[2][4];
  const int c = blockIdx.x;
  for (int j = 0; j < kk; ++j) {
    const double* yj = Y + static_cast<size_t>(j) * n;
    double acc = 0.0;
    for (int i = lo[c] + threadIdx.x; i < hi[c]; i += 256) acc = fmadd(yj[i], w[i], acc);
    const double s = block_sum_256(acc, lds[j & 1]);
    if (threadIdx.x == 0) partial[static_cast<size_t>(c) * kk + j] = s;
  }
}

struct OpStoreCoef {
  double* coef;  // [seg][kMaxLanczos]
  __device__ void operator()(int s, int q, double v) const { coef[s * kMaxLanczos + q] = v; }
};

// wu -= sum_j c_j U_j ; wy -= sum_j c_j Y_j (c of the element's segment; off in block rows)
__global__ void judge_reorth_kernel(size_t n, int bs, const int32_t* __restrict__ off, int nseg, int kk,
                                    const double* __restrict__ coef, const double* __restrict__ U,
                                    const double* __restrict__ Y, double* __restrict__ wu, double* __restrict__ wy) {
  const size_t i = blockIdx.x * static_cast<size_t>(blockDim.x) + threadIdx.x;
  if (i >= n) return;
  const double* c = coef + seg_of(off, nseg, static_cast<int>(i / bs)) * kMaxLanczos;
  double a = wu[i], b = wy[i];
  for (int j = 0; j < kk; ++j) {
    a -= c[j] * U[static_cast<size_t>(j) * n + i];
    b -= c[j] * Y[static_cast<size_t>(j) * n + i];
  }
  wu[i] = a;
  wy[i] = b;
}

// sc[s].tmp[which] = v
struct OpStoreTmp {
  LevelScalars* sc;
  int which;
  __device__ void operator()(int s, int, double v) const { sc[s].tmp[which] = v; }
};

}  // namespace blk
