// Generation step support for a population optimiser on top of the evaluator:
// a counter-based candidate sampler and the acceptance of partial changes.
//
// Sec. 2.2: each partial change is accepted only if it improves the solution;
// changes to FOS elements whose affected tetrahedra are disjoint (one colour
// class of single points: equal index parity on every axis) are independent, so
// all accepted changes of a class are applied together.  "Improves" is read in
// the multi-objective sense: the candidate is feasible and either Pareto-
// dominates the current solution or is not dominated by any member of the
// elitist archive.
#include <hip/hip_runtime.h>
#include <algorithm>
#include <math.h>

#include "dsm_internal.h"

namespace dsm {
namespace {

__device__ __forceinline__ unsigned long long mix64(unsigned long long z) {
  z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
  z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
  return z ^ (z >> 31);
}

// standard normal from two counter-based uniforms (Box-Muller)
__device__ __forceinline__ double normal(unsigned long long seed, unsigned long long ctr) {
  const unsigned long long a = mix64(seed + 0x9e3779b97f4a7c15ull * (2 * ctr + 1));
  const unsigned long long b = mix64(seed + 0x9e3779b97f4a7c15ull * (2 * ctr + 2));
  const double u1 = ((double)(a >> 11) + 1.0) * (1.0 / 9007199254740993.0);  // (0, 1]
  const double u2 = (double)(b >> 11) * (1.0 / 9007199254740992.0);
  return sqrt(-2.0 * log(u1)) * cos(6.283185307179586 * u2);
}

// cand [S][F][K][2][3]: current position of single point pts[f] plus
// N(0, sigma) voxels on its free axes, clamped to the image box and rounded to
// the 1/128-voxel lattice (half to even).
__global__ void k_sample(DevProblem pr, int S, const float* __restrict__ X, int F, const int* __restrict__ pts, int K,
                         float sigma, unsigned long long seed, unsigned long long counter,
                         const unsigned long long* __restrict__ counter_dev, float* __restrict__ cand) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (counter_dev) counter += *counter_dev;
  const int64_t n = (int64_t)S * F * K * 6;
  if (e >= n) return;
  const int comp = (int)(e % 6);
  const int64_t row = e / 6;
  const int f = (int)((row / K) % F);
  const int s = (int)(row / ((int64_t)F * K));
  const int g = comp / 3, a = comp % 3;
  const int p = pts[f];
  if (p < 0 || p >= pr.P) {
    cand[e] = NAN;  // flagged as non-finite by the evaluator
    return;
  }
  const float x = X[(((size_t)s * 2 + g) * pr.P + p) * 3 + a];
  const int idx = a == 0 ? p % pr.n[0] : (a == 1 ? (p / pr.n[0]) % pr.n[1] : p / (pr.n[0] * pr.n[1]));
  const bool free_axis = idx > 0 && idx < pr.n[a] - 1;
  double v = x;
  if (free_axis) {
    v += sigma * normal(seed, counter * 0x100000000ull + (unsigned long long)e);
    v = fmin(fmax(v, -0.5), pr.D[a] - 0.5);
  }
  v = rint((v + 0.5) * kLat) / kLat - 0.5;
  cand[e] = (float)v;
}

// ------------------------------------------------ estimated distributions
// RV-GOMEA, on which Sec. 2.2 builds, draws the variables of a FOS element
// from a normal distribution estimated on selected solutions of the
// population.  For a single-point element the variables are the point's 6
// coordinates (source grid x y z, target grid x y z); coordinates pinned to
// the box (border points) are not variables.

// Multi-point elements (such as the paper's per-cube tetrahedra): the
// variables of element f are the coordinates of its points
// fos_pts[fos_off[f] .. fos_off[f+1]) in order, 6 per point (source x y z,
// target x y z), at most kEstPoints points.  The distribution is estimated
// over all of them jointly (full covariance).
constexpr int kEstPoints = 4, kEstVars = 6 * kEstPoints, kEstTri = kEstVars * (kEstVars + 1) / 2;
constexpr int kEstTile = 192;  // selected solutions staged in LDS at a time

__device__ __forceinline__ double readlane64(double v, int l) {
  const long long u = __double_as_longlong(v);
  const unsigned lo = __builtin_amdgcn_readlane((unsigned)u, l), hi = __builtin_amdgcn_readlane((unsigned)(u >> 32), l);
  return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

__device__ __forceinline__ int64_t wide_block() { return blockIdx.x + (int64_t)gridDim.x * blockIdx.y; }

// Mean and Cholesky factor of the elements' distributions, for elements of up
// to NP points (NP = 1: the single points pts[f], off null; else CSR).  Per
// element f: mean [F][NV] of the variables over the solutions sel[0..n_sel)
// (indices outside [0, S) are skipped), and chol [F][NE], the lower Cholesky
// factor (row r holding columns 0..r) of their maximum-likelihood covariance
// (divisor: the number of solutions used) restricted to the free variables;
// rows and columns of pinned coordinates, and of variables beyond 6 x (number
// of points), are 0, and a pivot that is not positive (a rank-deficient
// selection) gives a zero column.  Elements with no point, more than NP
// points, an invalid point or no valid solution get zeros.  Cluster blockIdx.z
// has a selection, means and factors of its own, one after the other.
//
// One workgroup per element, one thread per covariance entry.  There are few
// elements in a call (5 to 75), so the kernel is bound by the length of its
// chain, not by the chip: the centred variables are staged once in FP64, each
// entry is one pass over them in selection order, and the factorisation keeps
// row r in the registers of lane r and subtracts column k's products as soon
// as the column is known (the order of the products of an entry is that of
// the row-by-row form).  On 64 elements of 4 points over 70 solutions: 208 us
// a call with the factorisation on one thread and two staging passes, 18.2 with
// the library's root and division in it, 16.6 now.
template <int NP>
__global__ __launch_bounds__(NP == 1 ? 64 : 320) void k_estimate(DevProblem pr, int S, const float* __restrict__ X,
                                                                 int n_sel, const int* __restrict__ sel, int F,
                                                                 const int* __restrict__ off,
                                                                 const int* __restrict__ pts,
                                                                 double* __restrict__ mean, double* __restrict__ chol) {
  constexpr int NV = 6 * NP, NE = NV * (NV + 1) / 2, WG = NP == 1 ? 64 : 320;
  static_assert(NE <= WG, "one thread per covariance entry");
  __shared__ float s_x[kEstTile][NV];
  __shared__ double s_d[kEstTile][NV];  // centred, 0 for skipped solutions and pinned variables
  __shared__ double s_mu[NV];
  __shared__ double s_C[NE];
  __shared__ bool s_ok[kEstTile], s_free[NV];
  if (wide_block() >= F) return;
  const int f = (int)wide_block(), t = threadIdx.x;
  sel += (size_t)blockIdx.z * n_sel;
  double* mu = mean + ((size_t)blockIdx.z * F + f) * NV;
  double* L = chol + ((size_t)blockIdx.z * F + f) * NE;
  const int b = off ? off[f] : f, np = off ? off[f + 1] - b : 1;
  bool ok = b >= 0 && np >= 1 && np <= NP && (!off || b + np <= off[F]);
  for (int k = 0; ok && k < np; ++k) ok = pts[b + k] >= 0 && pts[b + k] < pr.P;
  int n = 0;  // solutions used
  if (ok)
    for (int i0 = 0; i0 < n_sel; i0 += WG) {
      const int s = i0 + t < n_sel ? sel[i0 + t] : -1;
      n += __syncthreads_count(s >= 0 && s < S);
    }
  if (n == 0) {
    for (int i = t; i < NV; i += WG) mu[i] = 0.0;
    for (int i = t; i < NE; i += WG) L[i] = 0.0;
    return;
  }
  const int nv = 6 * np;
  if (t < NV) {  // variable t: point t / 6, coordinate t % 6; free unless pinned to the box
    bool fr = false;
    if (t < nv) {
      const int p = pts[b + t / 6], a = t % 3;
      const int idx = a == 0 ? p % pr.n[0] : (a == 1 ? (p / pr.n[0]) % pr.n[1] : p / (pr.n[0] * pr.n[1]));
      fr = idx > 0 && idx < pr.n[a] - 1;
    }
    s_free[t] = fr;
  }
  auto stage = [&](int i0) {
    const int rows = min(kEstTile, n_sel - i0);
    for (int q = t; q < rows * NV; q += WG) {
      const int i = q / NV, v = q % NV, s = sel[i0 + i];
      const bool use = s >= 0 && s < S;
      float x = 0.f;
      if (use && v < nv) {
        const int p = pts[b + v / 6], c = v % 6;
        x = X[(((size_t)s * 2 + c / 3) * pr.P + p) * 3 + c % 3];
      }
      s_x[i][v] = x;
      if (v == 0) s_ok[i] = use;
    }
    __syncthreads();
    return rows;
  };
  double m = 0.0;
  int rows = 0;
  for (int i0 = 0; i0 < n_sel; i0 += kEstTile) {
    rows = stage(i0);
    if (t < NV) {
#pragma unroll 8
      for (int i = 0; i < rows; ++i) m += (double)s_x[i][t];  // skipped solutions add 0
    }
    if (i0 + kEstTile < n_sel) __syncthreads();
  }
  if (t < NV) s_mu[t] = m / n;
  __syncthreads();
  int r = 0;  // entry t: row r, column c
  while (t < NE && (r + 1) * (r + 2) / 2 <= t) ++r;
  const int c = t < NE ? t - r * (r + 1) / 2 : 0;
  double acc = 0.0;
  for (int i0 = 0; i0 < n_sel; i0 += kEstTile) {
    if (n_sel > kEstTile) rows = stage(i0);  // a single tile is still there
    for (int q = t; q < rows * NV; q += WG) {
      const int i = q / NV, v = q % NV;
      s_d[i][v] = s_ok[i] && s_free[v] ? (double)s_x[i][v] - s_mu[v] : 0.0;
    }
    __syncthreads();
#pragma unroll 4
    for (int i = 0; i < rows; ++i) acc += s_d[i][r] * s_d[i][c];
    if (i0 + kEstTile < n_sel) __syncthreads();
  }
  if (t < NE) s_C[t] = s_free[r] && s_free[c] ? acc / n : 0.0;
  __syncthreads();
  if (t < 64) {
    const int row = min(t, NV - 1), base = row * (row + 1) / 2;  // lanes past the last row repeat it
    double v[NV];
#pragma unroll
    for (int k = 0; k < NV; ++k) v[k] = k <= row ? s_C[base + k] : 0.0;
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (k < nv) {
        const double pivot = readlane64(v[k], k);
        double l = 0.0;
        if (pivot > 0.0) {
          // y = 1 / sqrt(pivot) by two Newton steps, then the root and the
          // quotient each corrected by their residual (within an ulp): 11
          // dependent steps, a square root and a division took 30
          double y = __builtin_amdgcn_rsq(pivot);
          y = fma(0.5 * y, fma(-(pivot * y), y, 1.0), y);
          y = fma(0.5 * y, fma(-(pivot * y), y, 1.0), y);
          double d = pivot * y;
          d = fma(fma(-d, d, pivot), 0.5 * y, d);
          l = v[k] * y;
          l = row == k ? d : fma(fma(-l, d, v[k]), y, l);
        }
        v[k] = l;
#pragma unroll
        for (int j = k + 1; j < NV; ++j) v[j] -= l * readlane64(l, j);
      }
#pragma unroll
    for (int k = 0; k < NV; ++k)
      if (t < NV && k <= row) s_C[base + k] = v[k];
  }
  __syncthreads();
  if (t < NV) mu[t] = s_mu[t];
  if (t < NE) L[t] = s_C[t];
}

// Candidates drawn from the estimated distributions: mean + sqrt(mult) L z on
// the free variables, z ~ N(0, I) from the counter-based generator (NV draws
// per candidate, counters as in k_sample); pinned coordinates keep the
// solution's value; clamped to the image box and rounded to the 1/128-voxel
// lattice (half to even).  NP = 1: K candidates cand [S][F][K][2][3] of the
// single points pts[f] (off null); else one candidate cand [S][fos_off[F]][2][3]
// of the elements of up to NP points.  An invalid point, element or cluster
// gives NaN (flagged as non-finite by the evaluator); elements with malformed
// offsets are not written.
//
// A group of LG lanes per candidate, lane t drawing and combining variables t,
// t + LG, ... (z passed between the lanes), so that the FP64 logarithm and
// cosine of the draws, which bound the kernel, run side by side instead of NV
// times in a row, and nothing is kept in scratch memory.  Candidates are
// numbered as they are stored, so a wave reads and writes in one piece (with
// the element slowest, for one factor a wave: 5 % slower at 729,000 points, the
// same at 13,500 elements).
template <int NP, int LG>
__global__ __launch_bounds__(256) void k_sample_dist(DevProblem pr, int S, const float* __restrict__ X, int F,
                                                     const int* __restrict__ off, const int* __restrict__ pts, int K,
                                                     const double* __restrict__ mean, const double* __restrict__ chol,
                                                     const float* __restrict__ mult, int n_clusters,
                                                     const int* __restrict__ cluster, const double* __restrict__ shift,
                                                     const unsigned char* __restrict__ ams, double delta,
                                                     unsigned long long seed, unsigned long long counter,
                                                     const unsigned long long* __restrict__ counter_dev,
                                                     float* __restrict__ cand) {
  constexpr int NV = 6 * NP, NE = NV * (NV + 1) / 2, NU = (NV + LG - 1) / LG;  // variables of a lane
  static_assert(64 % LG == 0 && (NU == 1 || NP == 1), "several variables a lane for single points only");
  const int64_t g = wide_block() * (256 / LG) + threadIdx.x / LG;
  const int t = threadIdx.x % LG;
  if (counter_dev) counter += *counter_dev;
  if (g >= (int64_t)S * F * K) return;
  const int64_t sf = g / K;
  const int s = (int)(sf / F), f = (int)(sf - (int64_t)s * F);
  const int b = off ? off[f] : f, np = off ? off[f + 1] - b : 1;
  if (off && (b < 0 || np < 0 || b + np > off[F])) return;  // malformed offsets: nothing of this element to write
  float* out = off ? cand + ((size_t)s * off[F] + b) * 6 : cand + g * 6;
  const int cl = cluster ? cluster[s] : 0;
  bool ok = np >= 1 && np <= NP && cl >= 0 && cl < n_clusters;
  for (int k = 0; ok && k < np; ++k) ok = pts[b + k] >= 0 && pts[b + k] < pr.P;
  if (!ok) {
    for (int e = t; e < 6 * np; e += LG) out[e] = NAN;
    return;
  }
  const int nv = 6 * np;
  const size_t d = (size_t)cl * F + f;  // distribution of the solution's cluster
  double z[NU], w[NU];
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int v = t + LG * u;
    z[u] = v < nv ? normal(seed, counter * 0x100000000ull + (unsigned long long)(g * NV + v)) : 0.0;
    w[u] = 0.0;
  }
  for (int k0 = 0; k0 < nv; k0 += 6) {  // the factor's entries 6 at a time: one wait for memory each
#pragma unroll
    for (int u = 0; u < NU; ++u) {
      const int v = t + LG * u;
      const double* L = chol + d * NE + v * (v + 1) / 2;
      double l[6];
#pragma unroll
      for (int q = 0; q < 6; ++q) l[q] = v < nv && k0 + q <= v ? L[k0 + q] : 0.0;
#pragma unroll
      for (int q = 0; q < 6; ++q) {
        const double zk = LG == 1 ? z[q % NU] : __shfl(z[q / LG % NU], NU == 1 ? k0 + q : q % LG, LG);  // k0 = 0 if NU > 1
        if (k0 + q <= v && v < nv) w[u] += l[q] * zk;
      }
    }
  }
#pragma unroll
  for (int u = 0; u < NU; ++u) {
    const int v = t + LG * u;
    if (v >= nv) continue;
    const int p = pts[b + v / 6], c = v % 6, gr = c / 3, a = c % 3;
    const int idx = a == 0 ? p % pr.n[0] : (a == 1 ? (p / pr.n[0]) % pr.n[1] : p / (pr.n[0] * pr.n[1]));
    double x = X[(((size_t)s * 2 + gr) * pr.P + p) * 3 + a];
    if (idx > 0 && idx < pr.n[a] - 1) {
      const double sc = sqrt((double)mult[d]);
      double m = mean[d * NV + v];
      if (shift && ams[s]) m += delta * (double)mult[d] * shift[(size_t)p * 6 + c];  // anticipated mean shift
      x = fmin(fmax(m + sc * w[u], -0.5), pr.D[a] - 0.5);
    }
    out[v] = (float)(rint((x + 0.5) * kLat) / kLat - 0.5);
  }
}

// Whether a row of the archive, up to the first row of padding (first value
// +inf), dominates v: the G lanes of a group take a row each.
template <int G>
__device__ __forceinline__ bool archive_dominates(const double* __restrict__ arch, int n_arch, const double v[3], int lane) {
  bool dominated = false;
  for (int q0 = 0; q0 < n_arch && !dominated; q0 += G) {
    const int q = q0 + lane;
    const double* a = arch + (size_t)q * 3;
    bool le = true, lt = false;
    if constexpr (G == 1) {
      if (a[0] == INFINITY) break;
      for (int o = 0; o < 3; ++o) {
        le = le && a[o] <= v[o];
        lt = lt || a[o] < v[o];
      }
      dominated = le && lt;
    } else {
      bool end = q >= n_arch, dom = false;
      if (!end) {
        end = a[0] == INFINITY;
        for (int o = 0; o < 3; ++o) {
          le = le && a[o] <= v[o];
          lt = lt || a[o] < v[o];
        }
        dom = le && lt;
      }
      // the group's lanes of the wave's votes
      const int shift = threadIdx.x & 63 & ~(G - 1);
      const unsigned long long ends = __ballot(end) >> shift & (~0ull >> (64 - G));
      const unsigned long long doms = __ballot(dom) >> shift & (~0ull >> (64 - G));
      dominated = (doms & (ends ? (ends & -ends) - 1 : ~0ull)) != 0;  // of the rows ahead of the end
      if (ends) break;
    }
  }
  return dominated;
}

// Accept / apply one colour class of elements, G lanes per (solution, element)
// pair: they share the scan of the archive and the copy of the element's
// coordinates and of its points' candidate terms.  With a thread per pair, a
// pair's dependent loads (up to the whole archive, then up to 4 x 48 tetrahedra
// x 3 terms) run one after another: 75 us a class of the phantom's 6^3 grid
// (2,000 pairs).
template <int G>
__global__ __launch_bounds__(256) void k_accept(DevProblem pr, int S, float* __restrict__ X, int F,
                                                const int* __restrict__ off, const int* __restrict__ pts,
                                                const float* __restrict__ cand, const double* __restrict__ part_old,
                                                const double* __restrict__ part_new, const uint32_t* __restrict__ flags,
                                                const double* __restrict__ terms_cand, double* __restrict__ cache,
                                                const double* __restrict__ obj, int n_arch,
                                                const double* __restrict__ arch,
                                                const int* __restrict__ single_objective,
                                                unsigned char* __restrict__ accepted) {
  const int64_t e = blockIdx.x * (int64_t)(256 / G) + threadIdx.x / G;  // the same on every lane of a group
  const int lane = threadIdx.x % G;
  if (e >= (int64_t)S * F) return;
  const int s = (int)(e / F), f = (int)(e - (int64_t)s * F);
  bool acc = flags[e] == 0u;
  if (acc) {
    double d[3], nv[3];
    bool le = true, lt = false;
    for (int o = 0; o < 3; ++o) {
      d[o] = part_new[(size_t)e * 3 + o] - part_old[(size_t)e * 3 + o];
      nv[o] = obj[(size_t)s * 3 + o] + d[o];
      le = le && d[o] <= 0.0;
      lt = lt || d[o] < 0.0;
    }
    acc = le && lt;
    const int so = single_objective ? single_objective[s] : -1;
    if (so >= 0 && so < 3) {
      acc = d[so] < 0.0;  // a single-objective cluster's member: improve that objective
    } else if (!acc && n_arch > 0) {
      bool improves = false;
      for (int o = 0; o < 3; ++o) improves = improves || d[o] < 0.0;
      acc = improves && !archive_dominates<G>(arch, n_arch, nv, lane);
    }
  }
  if (accepted && lane == 0) accepted[e] = acc ? 1 : 0;
  if (!acc) return;
  // the element's points: pts[off[f] .. off[f+1]) with candidates at
  // [s][off[F]][2][3], or the single point pts[f] without off
  const int j0 = off ? off[f] : f, j1 = off ? off[f + 1] : f + 1, n = off ? off[F] : F;
  for (int j = j0; j < j1; ++j) {
    const int p = pts[j];
    if (p < 0 || p >= pr.P) continue;  // such elements are flagged by the evaluator
    for (int c = lane; c < 6; c += G)
      X[(((size_t)s * 2 + c / 3) * pr.P + p) * 3 + c % 3] = cand[((size_t)s * n + j) * 6 + c];
    const int k0 = pr.star_off[p], k1 = pr.star_off[p + 1];
    if constexpr (G == 1) {
      for (int k = k0; k < k1; ++k) {
        const size_t t = ((size_t)s * pr.T + pr.star[k]) * 3;
        for (int o = 0; o < 3; ++o) cache[t + o] = terms_cand[t + o];
      }
    } else {
      for (int i = lane; i < 3 * (k1 - k0); i += G) {
        const size_t t = ((size_t)s * pr.T + pr.star[k0 + i / 3]) * 3 + i % 3;
        cache[t] = terms_cand[t];
      }
    }
  }
}

// Sec. 2.4 grid refinement: fine point (I, J, K) of a 2n-1 grid is the mean of
// the coarse points whose indices are floor or ceil of (I/2, J/2, K/2): a
// coarse point, an edge middle, a face middle or a cube centre.  The mean of
// lattice integers (1, 2, 4 or 8 of them) is exact in FP64 and is rounded
// to the lattice half to even.  One thread per (solution, grid, fine point).
__global__ void k_refine(int nx, int ny, int nz, int S, const float* __restrict__ Xc, float* __restrict__ Xf) {
  const int fx = 2 * nx - 1, fy = 2 * ny - 1, fz = 2 * nz - 1;
  const int64_t Pc = (int64_t)nx * ny * nz, Pf = (int64_t)fx * fy * fz;
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)S * 2 * Pf) return;
  const int64_t sg = e / Pf;
  const int f = (int)(e - sg * Pf);
  const int I = f % fx, J = (f / fx) % fy, K = f / (fx * fy);
  const int i0 = I >> 1, i1 = (I + 1) >> 1, j0 = J >> 1, j1 = (J + 1) >> 1, k0 = K >> 1, k1 = (K + 1) >> 1;
  const float* base = Xc + sg * Pc * 3;
  double u[3] = {0.0, 0.0, 0.0};
  for (int c = 0; c < 8; ++c) {  // the 8 index combinations; repeated corners weigh equally
    const int i = (c & 1) ? i1 : i0, j = (c & 2) ? j1 : j0, k = (c & 4) ? k1 : k0;
    const float* x = base + ((int64_t)(k * ny + j) * nx + i) * 3;
    for (int d = 0; d < 3; ++d) u[d] += ((double)x[d] + 0.5) * kLat;
  }
  float* y = Xf + e * 3;
  for (int d = 0; d < 3; ++d) y[d] = (float)(rint(u[d] * 0.125) / kLat - 0.5);
}

// Forced improvements (RV-GOMEA): a solution s with donor[s] in [0, S) takes,
// for every listed point, the donor's current coordinates in both grids as its
// candidate (cand [S][n][2][3], the partial-evaluation layout); other
// solutions' candidates are left as they are.
__global__ void k_donor(int S, int P, const float* __restrict__ X, int n, const int* __restrict__ pts,
                        const int* __restrict__ donor, float* __restrict__ cand) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)S * n * 6) return;
  const int s = (int)(e / ((int64_t)n * 6));
  const int k = (int)((e / 6) % n), c = (int)(e % 6);
  const int d = donor[s], p = pts[k];
  if (d < 0 || d >= S || p < 0 || p >= P) return;
  cand[e] = X[(((size_t)d * 2 + c / 3) * P + p) * 3 + c % 3];
}

// Standard-deviation ratio of the improvements (AMaLGaM's adaptive variance
// scaling, used by RV-GOMEA): per (cluster j, element f) the mean of the
// accepted candidates of the cluster's solutions, compared with the
// distribution's mean variable by variable in units of the variable's standard
// deviation (sqrt of the row norm of L); the largest ratio, or -1 without an
// accepted candidate.  One workgroup per (cluster, element): its threads test
// a solution each and list the accepted ones in order, then only those are
// staged and summed (lane v variable v, in solution order): few of a cluster's
// solutions accept, and a pass over all of them took 61 us for 500 solutions,
// most of it waiting for one row after another.
constexpr int kSdrTile = 256;

__global__ __launch_bounds__(kSdrTile) void k_sdr(int S, int F, const int* __restrict__ off,
                                                  const float* __restrict__ cand,
                                                  const unsigned char* __restrict__ accepted, int n_clusters,
                                                  const int* __restrict__ cluster, const double* __restrict__ mean,
                                                  const double* __restrict__ chol, int nvar, double* __restrict__ sdr) {
  __shared__ float s_x[kSdrTile][kEstVars];
  __shared__ int s_row[kSdrTile];
  __shared__ int s_cnt[kSdrTile / 64];
  __shared__ double s_L[kEstTri];
  const int64_t e = wide_block();  // (cluster, element)
  if (e >= (int64_t)n_clusters * F) return;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  const int j = (int)(e / F), f = (int)(e - (int64_t)j * F);
  const int b = off[f], np = off[f + 1] - b, total = off[F];
  const int nv = 6 * np;
  if (b < 0 || np < 1 || nv > nvar || b + np > total) {
    if (t == 0) sdr[e] = -1.0;
    return;
  }
  const int tri = nvar * (nvar + 1) / 2;
  for (int i = t; i < tri; i += kSdrTile) s_L[i] = chol[(size_t)e * tri + i];
  double sum = 0.0;
  int n = 0;
  for (int s0 = 0; s0 < S; s0 += kSdrTile) {
    const int s = s0 + t;
    const bool use = s < S && (cluster ? cluster[s] : 0) == j && accepted[(size_t)s * F + f];
    const unsigned long long m = __ballot(use);
    if (lane == 0) s_cnt[wave] = __popcll(m);
    __syncthreads();
    int at = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u)), rows = 0;
    for (int w = 0; w < kSdrTile / 64; ++w) {
      at += w < wave ? s_cnt[w] : 0;
      rows += s_cnt[w];
    }
    if (use) s_row[at] = s;
    __syncthreads();
    for (int q = t; q < rows * nv; q += kSdrTile) {
      const int i = q / nv, v = q - i * nv;
      s_x[i][v] = cand[((size_t)s_row[i] * total + b) * 6 + v];
    }
    __syncthreads();
    if (t < nv) {
#pragma unroll 4
      for (int i = 0; i < rows; ++i) sum += (double)s_x[i][t];
    }
    n += rows;
    __syncthreads();
  }
  if (n == 0) {
    if (t == 0) sdr[e] = -1.0;
    return;
  }
  if (wave != 0) return;
  double r = 0.0;
  if (lane < nv) {
    const double* L = s_L + lane * (lane + 1) / 2;
    double s2 = 0.0;
    for (int k = 0; k <= lane; ++k) s2 += L[k] * L[k];
    if (s2 > 0.0) r = fabs(sum / n - mean[(size_t)e * nvar + lane]) / sqrt(s2);
  }
  for (int m = 32; m >= 1; m >>= 1) r = fmax(r, __shfl_xor(r, m, 64));  // the maximum does not depend on order
  if (lane == 0) sdr[e] = r;
}

// ---------------------------------------------------------------- clustering
// Balanced k-leader-means of the selected solutions in objective space (the
// clustering of MO-RV-GOMEA, on which the paper's optimiser builds, Sec. 2.2):
// normalisation over the selection, farthest-first leaders, k-means from the
// leaders, each cluster the c nearest selected solutions, every solution
// assigned to its nearest mean.  One workgroup; every floating-point step runs
// in a fixed order without contraction (sums in selection order by one thread
// per cluster and objective), so the result does not depend on the schedule.
constexpr int kClusterWG = 1024, kClusterWaves = kClusterWG / 64;

__device__ __forceinline__ double dist2(const double* a, const double* b) {
#pragma clang fp contract(off)
  const double d0 = a[0] - b[0], d1 = a[1] - b[1], d2 = a[2] - b[2];
  return d0 * d0 + d1 * d1 + d2 * d2;
}

__device__ __forceinline__ int nearest_mean(const double* y, const double (*mu)[3], int k) {
  int best = 0;
  double bd = dist2(y, mu[0]);
  for (int j = 1; j < k; ++j) {
    const double d = dist2(y, mu[j]);
    if (d < bd) {
      best = j;
      bd = d;
    }
  }
  return best;
}

// Index of the largest v[0..n) (lowest index among equals), for all threads.
__device__ int block_argmax(const double* v, int n, double* wv, int* wi, int* out) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  double bv = -INFINITY;
  int bi = 0x7fffffff;
  for (int i = tid; i < n; i += kClusterWG)
    if (v[i] > bv) {  // increasing i: an equal later value never replaces
      bv = v[i];
      bi = i;
    }
  for (int m = 32; m >= 1; m >>= 1) {
    const double ov = __shfl_xor(bv, m);
    const int oi = __shfl_xor(bi, m);
    if (ov > bv || (ov == bv && oi < bi)) {
      bv = ov;
      bi = oi;
    }
  }
  if (lane == 0) {
    wv[wave] = bv;
    wi[wave] = bi;
  }
  __syncthreads();
  if (tid == 0) {
    double b = wv[0];
    int i0 = wi[0];
    for (int w = 1; w < kClusterWaves; ++w)
      if (wv[w] > b || (wv[w] == b && wi[w] < i0)) {
        b = wv[w];
        i0 = wi[w];
      }
    *out = i0;
  }
  __syncthreads();
  return *out;
}

__global__ __launch_bounds__(kClusterWG) void k_cluster(int S, const double* __restrict__ obj, int n_sel,
                                                        const int* __restrict__ sel, int k, int cmax,
                                                        int* __restrict__ members, int* __restrict__ assign,
                                                        double* __restrict__ means_out) {
#pragma clang fp contract(off)
  __shared__ int s_idx[kClusterSelMax];
  __shared__ double s_Y[kClusterSelMax][3];
  __shared__ double s_d[kClusterSelMax];
  __shared__ int s_lab[kClusterSelMax];
  __shared__ double s_mu[kClusterMax][3];
  __shared__ int s_lead[kClusterMax];
  __shared__ double s_lo[3], s_rng[3];
  __shared__ double s_red[kClusterWaves][6];
  __shared__ int s_wcnt[kClusterWaves];
  __shared__ double s_wv[kClusterWaves];
  __shared__ int s_wi[kClusterWaves];
  __shared__ int s_n, s_arg;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  // valid selected solutions, compacted in selection order
  if (tid == 0) s_n = 0;
  __syncthreads();
  for (int base = 0; base < n_sel; base += kClusterWG) {
    const int i = base + tid;
    const int s = i < n_sel ? sel[i] : -1;
    const bool v = s >= 0 && s < S;
    const unsigned long long m = __ballot(v);
    const int pre = (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
    if (lane == 0) s_wcnt[wave] = __popcll(m);
    __syncthreads();
    int off = s_n;
    for (int w = 0; w < wave; ++w) off += s_wcnt[w];
    if (v) s_idx[off + pre] = s;
    __syncthreads();
    if (tid == 0) {
      int t = s_n;
      for (int w = 0; w < kClusterWaves; ++w) t += s_wcnt[w];
      s_n = t;
    }
    __syncthreads();
  }
  const int n = s_n;
  const int c = min(n, (2 * n + k - 1) / k);
  for (int e = tid; e < k * cmax; e += kClusterWG)
    if (n < k || e % cmax >= c) members[e] = -1;
  if (n < k) {
    for (int s = tid; s < S; s += kClusterWG) assign[s] = -1;
    if (means_out && tid < 3 * k) means_out[tid] = NAN;
    return;
  }
  // per-objective range over the selection (min and max are order-free)
  double lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (int i = tid; i < n; i += kClusterWG)
    for (int o = 0; o < 3; ++o) {
      const double x = obj[(size_t)s_idx[i] * 3 + o];
      lo[o] = fmin(lo[o], x);
      hi[o] = fmax(hi[o], x);
    }
  for (int m = 32; m >= 1; m >>= 1)
    for (int o = 0; o < 3; ++o) {
      lo[o] = fmin(lo[o], __shfl_xor(lo[o], m));
      hi[o] = fmax(hi[o], __shfl_xor(hi[o], m));
    }
  if (lane == 0)
    for (int o = 0; o < 3; ++o) {
      s_red[wave][o] = lo[o];
      s_red[wave][3 + o] = hi[o];
    }
  __syncthreads();
  if (tid < 3) {
    double a = s_red[0][tid], b = s_red[0][3 + tid];
    for (int w = 1; w < kClusterWaves; ++w) {
      a = fmin(a, s_red[w][tid]);
      b = fmax(b, s_red[w][3 + tid]);
    }
    s_lo[tid] = a;
    s_rng[tid] = b - a > 0.0 ? b - a : 1.0;
  }
  __syncthreads();
  for (int i = tid; i < n; i += kClusterWG)
    for (int o = 0; o < 3; ++o) s_Y[i][o] = (obj[(size_t)s_idx[i] * 3 + o] - s_lo[o]) / s_rng[o];
  __syncthreads();
  // farthest-first leaders
  for (int i = tid; i < n; i += kClusterWG) s_d[i] = s_Y[i][0];
  __syncthreads();
  int lead = block_argmax(s_d, n, s_wv, s_wi, &s_arg);
  if (tid == 0) s_lead[0] = lead;
  for (int i = tid; i < n; i += kClusterWG) s_d[i] = dist2(s_Y[i], s_Y[lead]);
  __syncthreads();
  for (int l = 1; l < k; ++l) {
    lead = block_argmax(s_d, n, s_wv, s_wi, &s_arg);
    if (tid == 0) s_lead[l] = lead;
    for (int i = tid; i < n; i += kClusterWG) s_d[i] = fmin(s_d[i], dist2(s_Y[i], s_Y[lead]));
    __syncthreads();
  }
  if (tid < 3 * k) s_mu[tid / 3][tid % 3] = s_Y[s_lead[tid / 3]][tid % 3];
  for (int i = tid; i < n; i += kClusterWG) s_lab[i] = -1;
  __syncthreads();
  // k-means from the leaders
  for (int it = 0; it < kClusterRounds; ++it) {
    int changed = 0;
    for (int i = tid; i < n; i += kClusterWG) {
      const int j = nearest_mean(s_Y[i], s_mu, k);
      changed |= j != s_lab[i];
      s_lab[i] = j;
    }
    if (!__syncthreads_or(changed)) break;
    if (tid < 3 * k) {
      const int j = tid / 3, o = tid % 3;
      double acc = 0.0;
      int cnt = 0;
      for (int i = 0; i < n; ++i)
        if (s_lab[i] == j) {
          acc += s_Y[i][o];
          ++cnt;
        }
      if (cnt) s_mu[j][o] = acc / cnt;
    }
    __syncthreads();
  }
  // cluster j: the c selected solutions nearest to mean j (rank by distance, then position)
  for (int j = 0; j < k; ++j) {
    for (int i = tid; i < n; i += kClusterWG) s_d[i] = dist2(s_Y[i], s_mu[j]);
    __syncthreads();
    for (int i = tid; i < n; i += kClusterWG) {
      const double di = s_d[i];
      int rank = 0;
      for (int m = 0; m < n; ++m) rank += s_d[m] < di || (s_d[m] == di && m < i);
      if (rank < c) members[(size_t)j * cmax + rank] = s_idx[i];
    }
    __syncthreads();
  }
  for (int s = tid; s < S; s += kClusterWG) {
    double y[3];
    for (int o = 0; o < 3; ++o) y[o] = (obj[(size_t)s * 3 + o] - s_lo[o]) / s_rng[o];
    assign[s] = nearest_mean(y, s_mu, k);
  }
  if (means_out && tid < 3 * k) means_out[tid] = s_mu[tid / 3][tid % 3];
}

// Lanes of a pair by the number of pairs: once there are enough to fill the
// device, more lanes only repeat the pair's own loads.  In us, with 64 / 16 / 1
// lanes, for 30 % of the pairs accepted without an archive and for all of them
// tested against 3,000 rows: 13,500 pairs 23 / 23 / 29 and 89 / 129 / 890,
// 51,200 pairs 29 / 28 / 37 and 238 / 278 / 901, 125,000 pairs 43 / 38 / 45 and 538
// / 593 / 918, 729,000 pairs 121 / 78 / 71 and 3,001 / 3,106 / 2,706 (51,200 pairs
// all rejected: 24 / 21 / 20).
void launch_accept(const DevProblem& pr, int S, float* X, int F, const int* off, const int* pts, const float* cand,
                   const double* part_old, const double* part_new, const uint32_t* flags, const double* terms_cand,
                   double* cache, const double* obj, int n_arch, const double* arch, const int* single_objective,
                   unsigned char* accepted, hipStream_t st) {
  const int64_t pairs = (int64_t)S * F;
  auto launch = [&](auto* kernel, int lanes) {
    kernel<<<(unsigned)((pairs * lanes + 255) / 256), 256, 0, st>>>(pr, S, X, F, off, pts, cand, part_old, part_new, flags,
                                                                   terms_cand, cache, obj, n_arch, arch,
                                                                   single_objective, accepted);
  };
  if (pairs <= 49152)
    launch(k_accept<64>, 64);
  else if (pairs <= 196608)
    launch(k_accept<16>, 16);
  else
    launch(k_accept<1>, 1);
}

}  // namespace
}  // namespace dsm

using namespace dsm;

extern "C" {

dsm_status dsm_sample_candidates(dsm_problem* p, int32_t S, const float* X, int32_t F, const int32_t* fos_pts, int32_t K,
                                 float sigma, uint64_t seed, uint64_t counter, const uint64_t* counter_dev, float* cand,
                                 void* stream) {
  if (!p || S < 0 || F < 0 || K < 1 || !(sigma >= 0.f)) return DSM_ERR_ARG;
  const int64_t n = (int64_t)S * F * K * 6;
  if (n == 0) return DSM_OK;  // empty buffers may be null
  if (!X || !fos_pts || !cand) return DSM_ERR_ARG;
  k_sample<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)stream>>>(p->dev, S, X, F, fos_pts, K, sigma, seed,
                                                                       counter, (const unsigned long long*)counter_dev,
                                                                       cand);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_estimate_distributions(dsm_problem* p, int32_t S, const float* X, int32_t n_sel, const int32_t* sel,
                                      int32_t F, const int32_t* fos_pts, double* mean, double* chol, void* stream) {
  if (!p || S < 0 || F < 0 || n_sel < 0) return DSM_ERR_ARG;
  if (F == 0) return DSM_OK;  // empty buffers may be null
  if (!fos_pts || !mean || !chol || (n_sel > 0 && (!X || !sel))) return DSM_ERR_ARG;
  k_estimate<1><<<wide_grid(F), 64, 0, (hipStream_t)stream>>>(p->dev, S, X, n_sel, sel, F, nullptr, fos_pts, mean, chol);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_sample_estimated(dsm_problem* p, int32_t S, const float* X, int32_t F, const int32_t* fos_pts, int32_t K,
                                const double* mean, const double* chol, const float* mult, int32_t n_clusters,
                                const int32_t* cluster, const double* shift, const uint8_t* ams, double delta,
                                uint64_t seed, uint64_t counter, const uint64_t* counter_dev, float* cand,
                                void* stream) {
  if (!p || S < 0 || F < 0 || K < 1) return DSM_ERR_ARG;
  const int64_t n = (int64_t)S * F * K;
  if (n == 0) return DSM_OK;  // empty buffers may be null
  if (!X || !fos_pts || !mean || !chol || !mult || !cand || n_clusters < 1 || (shift && !ams)) return DSM_ERR_ARG;
  auto launch = [&](auto* kernel, int lanes) {
    kernel<<<wide_grid((n * lanes + 255) / 256), 256, 0, (hipStream_t)stream>>>(
        p->dev, S, X, F, nullptr, fos_pts, K, mean, chol, mult, n_clusters, cluster, shift, ams, delta, seed, counter,
        (const unsigned long long*)counter_dev, cand);
  };
  // a lane per variable while the lanes are too few to fill the device (13,500
  // candidates: 18.8 us, a thread each 20.2); beyond, a quarter of those lanes is
  // idle and every load is repeated (54,000: 23.5 against 20.8, 729,000: 106 against 57)
  if (n <= 40960)
    launch(k_sample_dist<1, 8>, 8);
  else
    launch(k_sample_dist<1, 1>, 1);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_estimate_elements(dsm_problem* p, int32_t S, const float* X, int32_t n_sel, const int32_t* sel, int32_t F,
                                 const int32_t* fos_off, const int32_t* fos_pts, double* mean, double* chol,
                                 void* stream) {
  if (!p || S < 0 || F < 0 || n_sel < 0) return DSM_ERR_ARG;
  if (F == 0) return DSM_OK;  // empty buffers may be null
  if (!fos_off || !fos_pts || !mean || !chol || (n_sel > 0 && (!X || !sel))) return DSM_ERR_ARG;
  k_estimate<kEstPoints><<<wide_grid(F), 320, 0, (hipStream_t)stream>>>(p->dev, S, X, n_sel, sel, F, fos_off, fos_pts, mean,
                                                                      chol);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_estimate_clusters(dsm_problem* p, int32_t S, const float* X, int32_t n_clusters, int32_t n_sel,
                                 const int32_t* sel, int32_t F, const int32_t* fos_off, const int32_t* fos_pts,
                                 double* mean, double* chol, void* stream) {
  if (!p || S < 0 || F < 0 || n_sel < 0 || n_clusters < 1 || n_clusters > kClusterMax) return DSM_ERR_ARG;
  if (F == 0) return DSM_OK;  // empty buffers may be null
  if (!fos_pts || !mean || !chol || (n_sel > 0 && (!X || !sel))) return DSM_ERR_ARG;
  dim3 grid = wide_grid(F);
  grid.z = (unsigned)n_clusters;
  if (fos_off)
    k_estimate<kEstPoints><<<grid, 320, 0, (hipStream_t)stream>>>(p->dev, S, X, n_sel, sel, F, fos_off, fos_pts, mean, chol);
  else
    k_estimate<1><<<grid, 64, 0, (hipStream_t)stream>>>(p->dev, S, X, n_sel, sel, F, nullptr, fos_pts, mean, chol);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_sample_elements(dsm_problem* p, int32_t S, const float* X, int32_t F, const int32_t* fos_off,
                               const int32_t* fos_pts, const double* mean, const double* chol, const float* mult,
                               int32_t n_clusters, const int32_t* cluster, const double* shift, const uint8_t* ams,
                               double delta, uint64_t seed, uint64_t counter, const uint64_t* counter_dev, float* cand,
                               void* stream) {
  if (!p || S < 0 || F < 0) return DSM_ERR_ARG;
  const int64_t n = (int64_t)S * F;
  if (n == 0) return DSM_OK;  // empty buffers may be null
  if (!X || !fos_off || !fos_pts || !mean || !chol || !mult || !cand || n_clusters < 1 || (shift && !ams))
    return DSM_ERR_ARG;
  k_sample_dist<kEstPoints, 32><<<wide_grid((n + 7) / 8), 256, 0, (hipStream_t)stream>>>(
      p->dev, S, X, F, fos_off, fos_pts, 1, mean, chol, mult, n_clusters, cluster, shift, ams, delta, seed, counter,
      (const unsigned long long*)counter_dev, cand);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_cluster_objectives(int32_t S, const double* obj, int32_t n_sel, const int32_t* sel, int32_t k,
                                  int32_t* members, int32_t* assign, double* means, void* stream) {
  if (S < 0 || n_sel < 0 || k < 1 || k > kClusterMax) return DSM_ERR_ARG;
  if (n_sel > kClusterSelMax) return DSM_ERR_CAPACITY;
  const int cmax = std::min<int>(n_sel, (2 * n_sel + k - 1) / k);
  if ((S > 0 && (!obj || !assign)) || (n_sel > 0 && !sel) || (cmax > 0 && !members)) return DSM_ERR_ARG;
  if (S == 0 && cmax == 0 && !means) return DSM_OK;  // nothing to write
  k_cluster<<<1, kClusterWG, 0, (hipStream_t)stream>>>(S, obj, n_sel, sel, k, cmax, members, assign, means);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_refine_population(const int32_t* mesh_coarse, int32_t S, const float* Xc, float* Xf, void* stream) {
  if (!mesh_coarse || S < 0 || (S > 0 && (!Xc || !Xf))) return DSM_ERR_ARG;
  const int nx = mesh_coarse[0], ny = mesh_coarse[1], nz = mesh_coarse[2];
  if (nx < 2 || ny < 2 || nz < 2 || nx > 129 || ny > 129 || nz > 129) return DSM_ERR_DOMAIN;
  const int64_t n = (int64_t)S * 2 * (2 * nx - 1) * (2 * ny - 1) * (2 * nz - 1);
  if (n == 0) return DSM_OK;
  k_refine<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)stream>>>(nx, ny, nz, S, Xc, Xf);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_accept(dsm_problem* p, int32_t S, float* X, int32_t F, const int32_t* fos_pts, const float* cand,
                      const double* part_old, const double* part_new, const uint32_t* flags, const double* terms_cand,
                      double* terms_cache, double* obj, int32_t n_archive, const double* archive,
                      const int32_t* single_objective, uint8_t* accepted, void* stream) {
  if (!p || S < 0 || F < 0 || n_archive < 0 || (n_archive > 0 && !archive) || S > p->max_S) return DSM_ERR_ARG;
  if (S == 0) return DSM_OK;  // empty buffers may be null
  if (!X || !terms_cache || !obj || (F > 0 && (!fos_pts || !cand || !part_old || !part_new || !flags || !terms_cand)))
    return DSM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (F > 0)
    launch_accept(p->dev, S, X, F, nullptr, fos_pts, cand, part_old, part_new, flags, terms_cand, terms_cache, obj, n_archive,
                  archive, single_objective, accepted, st);
  if (hipGetLastError() != hipSuccess) return DSM_ERR_DEVICE;
  return launch_full_reduce(p->dev, S, terms_cache, obj, st) == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_improvement_ratio(int32_t S, int32_t F, const int32_t* fos_off, const float* cand,
                                 const uint8_t* accepted, int32_t n_clusters, const int32_t* cluster,
                                 const double* mean, const double* chol, int32_t n_vars, double* sdr, void* stream) {
  if (S < 0 || F < 0 || n_clusters < 1 || (n_vars != 6 && n_vars != kEstVars)) return DSM_ERR_ARG;
  const int64_t n = (int64_t)n_clusters * F;
  if (n == 0) return DSM_OK;
  if (!fos_off || !mean || !chol || !sdr || (S > 0 && (!cand || !accepted))) return DSM_ERR_ARG;
  k_sdr<<<wide_grid(n), kSdrTile, 0, (hipStream_t)stream>>>(S, F, fos_off, cand, accepted, n_clusters, cluster, mean, chol,
                                                    n_vars, sdr);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_copy_from_donor(dsm_problem* p, int32_t S, const float* X, int32_t n_pts, const int32_t* fos_pts,
                               const int32_t* donor, float* cand, void* stream) {
  if (!p || S < 0 || n_pts < 0) return DSM_ERR_ARG;
  const int64_t n = (int64_t)S * n_pts * 6;
  if (n == 0) return DSM_OK;  // empty buffers may be null
  if (!X || !fos_pts || !donor || !cand) return DSM_ERR_ARG;
  k_donor<<<(unsigned)((n + 255) / 256), 256, 0, (hipStream_t)stream>>>(S, p->dev.P, X, n_pts, fos_pts, donor, cand);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_accept_elements(dsm_problem* p, int32_t S, float* X, int32_t F, const int32_t* fos_off,
                               const int32_t* fos_pts, const float* cand, const double* part_old,
                               const double* part_new, const uint32_t* flags, const double* terms_cand,
                               double* terms_cache, double* obj, int32_t n_archive, const double* archive,
                               const int32_t* single_objective, uint8_t* accepted, void* stream) {
  if (!p || S < 0 || F < 0 || n_archive < 0 || (n_archive > 0 && !archive) || S > p->max_S) return DSM_ERR_ARG;
  if (S == 0) return DSM_OK;  // empty buffers may be null
  if (!X || !terms_cache || !obj ||
      (F > 0 && (!fos_off || !fos_pts || !cand || !part_old || !part_new || !flags || !terms_cand)))
    return DSM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  if (F > 0)
    launch_accept(p->dev, S, X, F, fos_off, fos_pts, cand, part_old, part_new, flags, terms_cand, terms_cache, obj, n_archive,
                  archive, single_objective, accepted, st);
  if (hipGetLastError() != hipSuccess) return DSM_ERR_DEVICE;
  return launch_full_reduce(p->dev, S, terms_cache, obj, st) == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

}  // extern "C"
