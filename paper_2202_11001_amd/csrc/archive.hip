// Generation bookkeeping of the multi-objective optimiser on the device: the
// elitist archive (the approximation set of Sec. 2.4), the selection the
// distributions are estimated on, the adaptive multiplier step and the
// forced-improvement replacement (both from RV-GOMEA, which Sec. 2.2 builds
// on).  Every entry point only enqueues kernels: sizes that live on the device
// (the archive's row count) are read by the kernels, never by the host.
#include <hip/hip_runtime.h>
#include <math.h>

#include <algorithm>

#include "dsm_internal.h"

namespace dsm {
namespace {

constexpr int kMergeWG = 256, kMergeWaves = kMergeWG / 64;

// The three comparisons are written without short-circuits: in a loop over
// many vectors, branches around each coordinate's load cost more than the load.
__device__ __forceinline__ bool dominates3(const double* a, const double* b) {
  const double a0 = a[0], a1 = a[1], a2 = a[2], b0 = b[0], b1 = b[1], b2 = b[2];
  return (a0 <= b0) & (a1 <= b1) & (a2 <= b2) & ((a0 < b0) | (a1 < b1) | (a2 < b2));
}
__device__ __forceinline__ bool equal3(const double* a, const double* b) {
  return (a[0] == b[0]) & (a[1] == b[1]) & (a[2] == b[2]);
}
// a before b in lexicographic order
__device__ __forceinline__ bool lex_less(const double* a, const double* b) {
  const double a0 = a[0], a1 = a[1], a2 = a[2], b0 = b[0], b1 = b[1], b2 = b[2];
  return (a0 < b0) | ((a0 == b0) & ((a1 < b1) | ((a1 == b1) & (a2 < b2))));
}

// Workspace of one merge (byte offsets, 256-aligned regions).
struct MergeWork {
  size_t alive, keep_n, src, vec, rows, hdr, total;
};
__host__ __device__ inline size_t al256(size_t x) { return (x + 255) & ~size_t(255); }
__host__ __device__ inline MergeWork merge_work(int cap, int m, int row_floats) {
  MergeWork w;
  size_t o = 0;
  w.alive = o;  // uint64 [ceil(cap / 64)]: bit per archive row kept
  o = al256(o + sizeof(unsigned long long) * (((size_t)cap + 63) / 64));
  w.keep_n = o;  // int [m]: new point kept
  o = al256(o + sizeof(int) * (size_t)m);
  w.src = o;  // int [cap]: source of every merged row: an archive row, cap + a new point, or -1
  o = al256(o + sizeof(int) * (size_t)cap);
  w.vec = o;  // double [cap][3]: merged vectors
  o = al256(o + sizeof(double) * 3 * (size_t)cap);
  w.rows = o;  // float [cap][row_floats]: the archive rows that move
  o = al256(o + sizeof(float) * (size_t)cap * row_floats);
  w.hdr = o;  // int [2]: merged count, overflow
  o = al256(o + sizeof(int) * 2);
  w.total = o;
  return w;
}

// A merge is four kernels: what is kept, where it goes, the archive rows that
// move copied out, and everything written to its place.  With payload rows the
// copies bound it (a row that moves is read and written twice, a new one
// once, one that keeps its place not at all); the tests against m points are
// split over a workgroup's waves so that they are short.  The merges of eight
// generations of 500 points with 32 KB rows took 414 us each as seven kernels
// (one thread walking all points for each archive row: 116 and 88 us; every
// element of the whole capacity divided into row and column: 110 and 76 us;
// a prefix sum over the capacity by one workgroup: 25 us).

__device__ __forceinline__ int64_t wide_block() { return blockIdx.x + (int64_t)gridDim.x * blockIdx.y; }

constexpr int kMergeTile = 512;  // new points staged in LDS at a time

// Workgroups [0, ceil(cap / 64)): the 64 archive rows of a word, each wave
// testing them against a quarter of the new points; row i (of n) is kept iff
// no new point dominates it (the archive's own rows are mutually
// non-dominated and distinct).  Then one workgroup per new point: kept iff no
// archive row dominates or equals it, no new point dominates it and no earlier
// new point equals it.
__global__ __launch_bounds__(kMergeWG) void k_merge_mark(const double* __restrict__ arch,
                                                       const int* __restrict__ n_arch, int cap, int m,
                                                       const double* __restrict__ pts,
                                                       unsigned long long* __restrict__ alive,
                                                       int* __restrict__ keep_n, int* __restrict__ src) {
  __shared__ double s_p[kMergeTile][3];
  __shared__ unsigned long long s_dead[kMergeWaves];
  __shared__ int drop;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, words = (cap + 63) / 64;
  const int n = min(*n_arch, cap);
  const int64_t wg = wide_block();
  if (wg < words) {
    const int word = (int)wg;
    const int64_t i = (int64_t)word * 64 + lane;
    if (t < 64 && i < cap) src[i] = -1;  // NaN vectors have no place in the order and may leave positions free
    if ((int64_t)word * 64 >= n) {
      if (t == 0) alive[word] = 0;
      return;
    }
    double a[3] = {0.0, 0.0, 0.0};
    if (i < n)
      for (int c = 0; c < 3; ++c) a[c] = arch[3 * (size_t)i + c];
    bool dead = i >= n;
    for (int j0 = 0; j0 < m; j0 += kMergeTile) {
      const int mt = min(kMergeTile, m - j0);
      for (int e = t; e < 3 * mt; e += kMergeWG) s_p[e / 3][e % 3] = pts[3 * (size_t)j0 + e];
      __syncthreads();
#pragma unroll 4
      for (int j = wave; j < mt; j += kMergeWaves) dead |= dominates3(s_p[j], a);
      __syncthreads();
    }
    const unsigned long long d = __ballot(dead);
    if (lane == 0) s_dead[wave] = d;
    __syncthreads();
    if (t == 0) {
      unsigned long long all = 0;
      for (int w = 0; w < kMergeWaves; ++w) all |= s_dead[w];
      alive[word] = ~all;
    }
    return;
  }
  if (wg - words >= m) return;
  const int j = (int)(wg - words);
  if (t == 0) drop = 0;
  __syncthreads();
  const double* p = pts + 3 * (size_t)j;
  int d = 0;
  for (int i = t; i < n && !d; i += kMergeWG) {
    const double* a = arch + 3 * (size_t)i;
    d = dominates3(a, p) || equal3(a, p);
  }
  for (int k = t; k < m && !d; k += kMergeWG) {
    const double* q = pts + 3 * (size_t)k;
    d = dominates3(q, p) || (k < j && equal3(q, p));
  }
  if (d) atomicOr(&drop, 1);
  __syncthreads();
  if (t == 0) keep_n[j] = drop ? 0 : 1;
}

__device__ __forceinline__ int wave_add(int v) {
  for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
  return v;
}

// Archive rows kept in words [0, w), counted by the 64 lanes of a wave.
__device__ __forceinline__ int kept_before(const unsigned long long* __restrict__ alive, int w, int lane) {
  int c = 0;
  for (int k = lane; k < w; k += 64) c += __popcll(alive[k]);
  return wave_add(c);
}

// Output positions: kept archive rows keep their order (they are sorted) and
// make room for the kept new points lexicographically below them; a kept new
// point goes after the kept archive rows and kept new points below it (the
// sorted archive is searched 64 rows at a time).  Kept vectors are distinct,
// so the positions are a permutation of [0, k); src[position] is written.
// Workgroups [0, words) take the rows of a word, their waves a quarter of the
// points each; the next ones a new point per wave; the last one the header.
__global__ __launch_bounds__(kMergeWG) void k_merge_positions(const double* __restrict__ arch,
                                                            const int* __restrict__ n_arch, int cap, int m,
                                                            const double* __restrict__ pts,
                                                            const unsigned long long* __restrict__ alive,
                                                            const int* __restrict__ keep_n, int* __restrict__ src,
                                                            int* __restrict__ hdr) {
  __shared__ double s_p[kMergeTile][3];
  __shared__ int s_keep[kMergeTile];
  __shared__ int s_cnt[kMergeWaves][64];
  __shared__ int s_pre;
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6, words = (cap + 63) / 64;
  const int n = min(*n_arch, cap);
  const int64_t wg = wide_block();
  if (wg < words) {
    const int word = (int)wg;
    const unsigned long long mine = alive[word];
    if (!mine) return;
    const int i = word * 64 + lane;
    const bool kept = (mine >> lane) & 1;
    if (wave == 0) {
      const int pre = kept_before(alive, word, lane);
      if (lane == 0) s_pre = pre;
    }
    double a[3] = {0.0, 0.0, 0.0};
    if (kept)
      for (int c = 0; c < 3; ++c) a[c] = arch[3 * (size_t)i + c];
    int below = 0;
    for (int j0 = 0; j0 < m; j0 += kMergeTile) {
      const int mt = min(kMergeTile, m - j0);
      for (int e = t; e < 3 * mt; e += kMergeWG) s_p[e / 3][e % 3] = pts[3 * (size_t)j0 + e];
      for (int e = t; e < mt; e += kMergeWG) s_keep[e] = keep_n[j0 + e];
      __syncthreads();
#pragma unroll 4
      for (int j = wave; j < mt; j += kMergeWaves) below += s_keep[j] & (int)lex_less(s_p[j], a);
      __syncthreads();
    }
    s_cnt[wave][lane] = below;
    __syncthreads();
    if (wave == 0 && kept) {
      int pos = s_pre + __popcll(mine & ((1ull << lane) - 1));
      for (int w = 0; w < kMergeWaves; ++w) pos += s_cnt[w][lane];
      if (pos < cap) src[pos] = i;  // beyond it only where the merge overflows
    }
    return;
  }
  const int64_t j = (wg - words) * kMergeWaves + wave;  // the same on every lane of a wave
  if (j < m) {
    if (!keep_n[j]) return;
    const double p[3] = {pts[3 * (size_t)j], pts[3 * (size_t)j + 1], pts[3 * (size_t)j + 2]};
    int lo = 0, hi = n;  // the first archive row not below p lies in [lo, hi]
    while (lo < hi) {
      const int step = (hi - lo + 63) / 64, q = lo + lane * step;
      const int c = __popcll(__ballot(q < hi && lex_less(arch + 3 * (size_t)min(q, n - 1), p)));
      hi = min(hi, lo + c * step);
      lo = c ? lo + (c - 1) * step + 1 : lo;
    }
    int pos = kept_before(alive, lo >> 6, lane);
    if (lo & 63) pos += __popcll(alive[lo >> 6] & ((1ull << (lo & 63)) - 1));
    int below = 0;
    for (int k = lane; k < m; k += 64) below += keep_n[k] & (int)lex_less(pts + 3 * (size_t)k, p);
    pos += wave_add(below);
    if (lane == 0 && pos < cap) src[pos] = cap + (int)j;
  } else if (wg == words + m / kMergeWaves && wave == kMergeWaves - 1) {
    int k = kept_before(alive, words, lane), kn = 0;
    for (int q = lane; q < m; q += 64) kn += keep_n[q];
    k += wave_add(kn);
    if (lane == 0) {
      hdr[0] = k;
      hdr[1] = k > cap ? 1 : 0;
    }
  }
}

// The copy of a payload row by the gridDim.y workgroups of its column of the
// grid, in pairs of floats where every row starts at a multiple of 8 bytes
// (pairs).
__device__ __forceinline__ void copy_row(float* __restrict__ dst, const float* __restrict__ src, int n, bool pairs) {
  const int first = blockIdx.y * kMergeWG + threadIdx.x, step = gridDim.y * kMergeWG;
  if (pairs) {
    float2* d = reinterpret_cast<float2*>(dst);
    const float2* s = reinterpret_cast<const float2*>(src);
#pragma unroll 4
    for (int i = first; i < n / 2; i += step) d[i] = s[i];
  } else {
#pragma unroll 4
    for (int i = first; i < n; i += step) dst[i] = src[i];
  }
}

// Floats of a row per workgroup: longer rows are split.  One workgroup copies
// some 25 GB/s, so with one to a row an archive of few, long rows (solutions on a
// fine mesh) left the device idle: 4 points merged into 8 rows of 6.4 MB took 542
// us, 16 into 32 of them 720, in parts 39 and 115 (4,096 or 16,384 floats a part:
// the same within 3 %).
constexpr int kMergePart = 8192;

// The merged vectors, and the payload of every archive row that moves, copied
// to the workspace at their new positions; with `staged` the new rows too, for
// points whose rows lie in the archive's own buffer (its free rows, say), which
// k_merge_in writes.
__global__ __launch_bounds__(kMergeWG) void k_merge_out(const double* __restrict__ arch,
                                                      const float* __restrict__ arch_rows, int cap,
                                                      const double* __restrict__ pts,
                                                      const float* __restrict__ pt_rows, int row_floats, bool pairs,
                                                      bool staged, const int* __restrict__ src,
                                                      const int* __restrict__ hdr, double* __restrict__ vec,
                                                      float* __restrict__ rows) {
  if (hdr[1]) return;  // overflow: the archive stays as it was
  const int k = hdr[0];
  const int64_t wg = blockIdx.x + (int64_t)gridDim.x * blockIdx.y, step = (int64_t)gridDim.x * gridDim.y * kMergeWG;
  for (int64_t e = wg * kMergeWG + threadIdx.x; e < 3 * (int64_t)k; e += step) {
    const int r = (int)(e / 3), c = (int)(e - 3 * (int64_t)r), from = src[r];
    vec[e] = from < 0 ? INFINITY : (from < cap ? arch[3 * (size_t)from + c] : pts[3 * (size_t)(from - cap) + c]);
  }
  if (!row_floats) return;
  for (int r = blockIdx.x; r < k; r += gridDim.x) {
    const int from = src[r];
    if (from >= 0 && from != r && (from < cap || staged))
      copy_row(rows + (size_t)r * row_floats,
               from < cap ? arch_rows + (size_t)from * row_floats : pt_rows + (size_t)(from - cap) * row_floats, row_floats,
               pairs);
  }
}

// Writes the archive: vectors and moved rows from the workspace, new rows from
// the points (the workspace with `staged`), +inf after the count; the count and
// the overflow flag.
__global__ __launch_bounds__(kMergeWG) void k_merge_in(double* __restrict__ arch, float* __restrict__ arch_rows, int cap,
                                                     const float* __restrict__ pt_rows, int row_floats, bool pairs,
                                                     bool staged, const int* __restrict__ src,
                                                     const int* __restrict__ hdr, const double* __restrict__ vec,
                                                     const float* __restrict__ rows,
                                                     int* __restrict__ n_arch, int* __restrict__ overflow) {
  const int k = hdr[0];
  const bool over = hdr[1] != 0;
  const int64_t wg = blockIdx.x + (int64_t)gridDim.x * blockIdx.y, step = (int64_t)gridDim.x * gridDim.y * kMergeWG;
  if (wg == 0 && threadIdx.x == 0) {
    if (overflow) *overflow = over ? 1 : 0;
    if (!over) *n_arch = k;
  }
  if (over) return;
  for (int64_t e = wg * kMergeWG + threadIdx.x; e < 3 * (int64_t)cap; e += step)
    arch[e] = e < 3 * (int64_t)k ? vec[e] : INFINITY;
  if (!row_floats) return;
  for (int r = blockIdx.x; r < k; r += gridDim.x) {
    const int from = src[r];
    if (from >= 0 && from != r)
      copy_row(arch_rows + (size_t)r * row_floats,
               from < cap || staged ? rows + (size_t)r * row_floats : pt_rows + (size_t)(from - cap) * row_floats, row_floats,
               pairs);
  }
}

// Selection: one workgroup.  Range of every objective, dominated-by counts,
// keys count * 4 + normalised sum (the sum is below 4, so counts decide
// first), ranks by counting (ties by index), scatter of the first n_sel.
constexpr int kSelWG = 1024;
__global__ __launch_bounds__(kSelWG) void k_select(int S, const double* __restrict__ obj, int n_sel,
                                                   int* __restrict__ sel, int* __restrict__ dominated_by) {
  extern __shared__ double s_key[];  // [S]
  __shared__ double s_red[kSelWG / 64][6];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  double v[6] = {INFINITY, INFINITY, INFINITY, -INFINITY, -INFINITY, -INFINITY};  // lo xyz, hi xyz
  for (int i = t; i < S; i += kSelWG)
    for (int c = 0; c < 3; ++c) {
      v[c] = fmin(v[c], obj[3 * (size_t)i + c]);
      v[3 + c] = fmax(v[3 + c], obj[3 * (size_t)i + c]);
    }
  for (int off = 32; off >= 1; off >>= 1)
    for (int c = 0; c < 3; ++c) {
      v[c] = fmin(v[c], __shfl_xor(v[c], off, 64));
      v[3 + c] = fmax(v[3 + c], __shfl_xor(v[3 + c], off, 64));
    }
  if (lane == 0)
    for (int c = 0; c < 6; ++c) s_red[wave][c] = v[c];
  __syncthreads();
  double rl[3], range[3];
  for (int c = 0; c < 3; ++c) {
    double lo = s_red[0][c], hi = s_red[0][3 + c];
    for (int w = 1; w < kSelWG / 64; ++w) {
      lo = fmin(lo, s_red[w][c]);
      hi = fmax(hi, s_red[w][3 + c]);
    }
    rl[c] = lo;
    range[c] = fmax(hi - lo, 1e-300);
  }
  for (int i = t; i < S; i += kSelWG) {
    const double* o = obj + 3 * (size_t)i;
    int cnt = 0;
    for (int j = 0; j < S; ++j) cnt += dominates3(obj + 3 * (size_t)j, o);
    double nrm = 0.0;
    for (int c = 0; c < 3; ++c) nrm = nrm + (o[c] - rl[c]) / range[c];
    s_key[i] = (double)cnt * 4.0 + nrm;
    if (dominated_by) dominated_by[i] = cnt;
  }
  __syncthreads();
  for (int i = t; i < S; i += kSelWG) {
    const double k = s_key[i];
    int rank = 0;
    for (int j = 0; j < S; ++j) rank += s_key[j] < k || (s_key[j] == k && j < i);
    if (rank < n_sel) sel[rank] = i;
  }
}

// RV-GOMEA's anticipated mean shift: the change of the selection's point means
// since the previous generation; prev keeps the current means.
__global__ void k_ams_shift(int n, const double* __restrict__ mean, double* __restrict__ prev, double* __restrict__ shift,
                            int has_prev) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const double m = mean[i];
    if (has_prev) shift[i] = m - prev[i];
    prev[i] = m;
  }
}

// MO-RV-GOMEA's single-objective clusters: objective o = 0, 1, 2 (while o < k)
// takes, of the clusters not yet taken, the one with the lowest mean in o (the
// lowest index among equal means); every solution gets its cluster's objective.
// Each workgroup derives the (at most kClusterMax) assignments itself.
__global__ void k_so_clusters(int k, const double* __restrict__ means, int S, const int* __restrict__ assign,
                              int* __restrict__ so) {
  __shared__ int of_cluster[kClusterMax];
  if (threadIdx.x == 0) {
    for (int j = 0; j < k; ++j) of_cluster[j] = -1;
    for (int o = 0; o < 3 && o < k; ++o) {
      int best = -1;
      double bv = 0.0;
      for (int j = 0; j < k; ++j)
        if (of_cluster[j] < 0 && (best < 0 || means[3 * j + o] < bv)) {
          best = j;
          bv = means[3 * j + o];
        }
      of_cluster[best] = o;  // o < k clusters are taken, so one is free
    }
  }
  __syncthreads();
  for (int s = blockIdx.x * blockDim.x + threadIdx.x; s < S; s += gridDim.x * blockDim.x) {
    const int a = assign[s];
    so[s] = a >= 0 && a < k ? of_cluster[a] : -1;
  }
}

// RV-GOMEA's forced-improvement donors, one workgroup: the solutions no member
// dominates, in ascending order (block-wide prefix), and every solution whose
// no-improvement stretch exceeds nis_max takes the list's entry at
// min(floor(u[s] n), n - 1).
__global__ __launch_bounds__(1024) void k_draw_donors(int S, const int* __restrict__ nis, int nis_max,
                                                      const int* __restrict__ dominated_by, const float* __restrict__ u,
                                                      int* __restrict__ donor, int* __restrict__ n_forced) {
  extern __shared__ int s_nd[];  // [S]
  __shared__ int part[1024];
  __shared__ int s_forced;
  const int t = threadIdx.x;
  const int per = (S + 1023) / 1024;
  const int b = min(S, t * per), e = min(S, b + per);
  int c = 0;
  for (int i = b; i < e; ++i) c += dominated_by[i] == 0;
  part[t] = c;
  if (t == 0) s_forced = 0;
  __syncthreads();
  for (int off = 1; off < 1024; off <<= 1) {
    const int v = t >= off ? part[t - off] : 0;
    __syncthreads();
    part[t] += v;
    __syncthreads();
  }
  int run = part[t] - c;
  for (int i = b; i < e; ++i)
    if (dominated_by[i] == 0) s_nd[run++] = i;
  const int n = part[1023];
  __syncthreads();
  int forced = 0;
  for (int s = t; s < S; s += 1024) {
    int d = -1;
    if (nis[s] > nis_max && n > 0) {
      d = s_nd[min(max((int)(u[s] * (float)n), 0), n - 1)];
      ++forced;
    }
    donor[s] = d;
  }
  if (forced) atomicAdd(&s_forced, forced);
  __syncthreads();
  if (t == 0 && n_forced) n_forced[0] += s_forced;
}

// AMaLGaM's adaptive variance scaling, one thread per distribution (float32).
__global__ void k_avs(int n, float* __restrict__ mult, int* __restrict__ nis, const double* __restrict__ sdr,
                      int nis_max, float eta, float lo, float hi) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const float c = mult[i];
  const double r = sdr[i];
  float c1;
  int n1;
  if (r >= 0.0) {
    c1 = c < 1.f ? 1.f : c;
    if (r > 1.0) c1 = c1 / eta;
    n1 = 0;
  } else {
    n1 = c <= 1.f ? nis[i] + 1 : nis[i];
    c1 = c;
    if (c > 1.f || n1 >= nis_max) c1 = c * eta;
    if (c1 < 1.f && n1 < nis_max) c1 = 1.f;
  }
  mult[i] = fminf(fmaxf(c1, lo), hi);
  nis[i] = n1;
}

// The simple multiplier schedule: per (cluster j, element f), one thread
// scanning the solutions: a hit if a solution of cluster j (every solution
// without clusters) had element f accepted; the multiplier is divided by eta
// after a hit, else multiplied by it, within [lo, hi].
__global__ void k_multiplier_step(int k, int F, int S, const unsigned char* __restrict__ acc,
                                  const int* __restrict__ cluster, float* __restrict__ mult, float eta, float lo,
                                  float hi) {
  const int e = blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= k * F) return;
  const int j = e / F, f = e - j * F;
  bool hit = false;
  for (int s = 0; s < S && !hit; ++s) hit = acc[(size_t)s * F + f] != 0 && (!cluster || cluster[s] == j);
  const float c = mult[e];
  mult[e] = hit ? fminf(c / eta, hi) : fmaxf(c * eta, lo);
}

// improved[s] |= some element of solution s was accepted.
__global__ void k_mark_improved(int S, int F, const unsigned char* __restrict__ acc, unsigned char* __restrict__ improved) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s >= S) return;
  unsigned char any = 0;
  for (int f = 0; f < F; ++f) any |= acc[(size_t)s * F + f];
  if (any) improved[s] = 1;
}

// Forced-improvement replacement, first pass: the donors' rows (coordinates,
// objectives, term cache) of the solutions to replace are staged, so that a
// donor replaced in the same step still gives its values from before it.
__global__ void k_forced_stage(int S, int row_x, int row_c, const float* __restrict__ X, const double* __restrict__ obj,
                               const double* __restrict__ cache, const int* __restrict__ donor,
                               const unsigned char* __restrict__ improved, float* __restrict__ wx,
                               double* __restrict__ wobj, double* __restrict__ wcache) {
  const int s = blockIdx.y;
  const int d = donor[s];
  if (d < 0 || d >= S || improved[s]) return;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < row_x + 3 + row_c; k += gridDim.x * blockDim.x) {
    if (k < row_x)
      wx[(size_t)s * row_x + k] = X[(size_t)d * row_x + k];
    else if (k < row_x + 3)
      wobj[3 * (size_t)s + (k - row_x)] = obj[3 * (size_t)d + (k - row_x)];
    else
      wcache[(size_t)s * row_c + (k - row_x - 3)] = cache[(size_t)d * row_c + (k - row_x - 3)];
  }
}

// Second pass: the staged rows are written; the stretches are updated.
__global__ void k_forced_apply(int S, int row_x, int row_c, float* __restrict__ X, double* __restrict__ obj,
                               double* __restrict__ cache, const int* __restrict__ donor,
                               const unsigned char* __restrict__ improved, const float* __restrict__ wx,
                               const double* __restrict__ wobj, const double* __restrict__ wcache,
                               int* __restrict__ nis, int* __restrict__ n_replaced) {
  const int s = blockIdx.y;
  const int d = donor[s];
  const bool replace = d >= 0 && d < S && !improved[s];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    nis[s] = (improved[s] || d >= 0) ? 0 : nis[s] + 1;
    if (replace && n_replaced) atomicAdd(n_replaced, 1);
  }
  if (!replace) return;
  for (int k = blockIdx.x * blockDim.x + threadIdx.x; k < row_x + 3 + row_c; k += gridDim.x * blockDim.x) {
    if (k < row_x)
      X[(size_t)s * row_x + k] = wx[(size_t)s * row_x + k];
    else if (k < row_x + 3)
      obj[3 * (size_t)s + (k - row_x)] = wobj[3 * (size_t)s + (k - row_x)];
    else
      cache[(size_t)s * row_c + (k - row_x - 3)] = wcache[(size_t)s * row_c + (k - row_x - 3)];
  }
}

}  // namespace
}  // namespace dsm

using namespace dsm;

extern "C" {

size_t dsm_archive_work_bytes(int32_t capacity, int32_t m, int32_t row_floats) {
  if (capacity < 1 || m < 0 || row_floats < 0) return 0;
  return merge_work(capacity, m, row_floats).total;
}

dsm_status dsm_archive_merge(int32_t capacity, double* archive, int32_t* n_archive, int32_t m, const double* points,
                             int32_t row_floats, float* archive_rows, const float* point_rows, void* work,
                             int32_t* overflow, void* stream) {
  if (capacity < 1 || m < 0 || row_floats < 0) return DSM_ERR_ARG;
  if (!archive || !n_archive || !work || (m > 0 && !points)) return DSM_ERR_ARG;
  if (row_floats > 0 && (!archive_rows || (m > 0 && !point_rows))) return DSM_ERR_ARG;
  hipStream_t st = (hipStream_t)stream;
  const MergeWork w = merge_work(capacity, m, row_floats);
  unsigned char* base = (unsigned char*)work;
  unsigned long long* alive = (unsigned long long*)(base + w.alive);
  int* keep_n = (int*)(base + w.keep_n);
  int* src = (int*)(base + w.src);
  double* vec = (double*)(base + w.vec);
  float* rows = (float*)(base + w.rows);
  int* hdr = (int*)(base + w.hdr);
  const int words = (capacity + 63) / 64;
  k_merge_mark<<<wide_grid((int64_t)words + m), kMergeWG, 0, st>>>(archive, n_archive, capacity, m, points, alive, keep_n, src);
  // m / waves + 1 workgroups after the words: the last one's last wave has no point and writes the header
  k_merge_positions<<<wide_grid((int64_t)words + m / kMergeWaves + 1), kMergeWG, 0, st>>>(archive, n_archive, capacity, m, points, alive,
                                                                     keep_n, src, hdr);
  const bool pairs = row_floats % 2 == 0 && (((uintptr_t)archive_rows | (uintptr_t)point_rows | (uintptr_t)rows) & 7) == 0;
  // a workgroup per row (or part of one) with payload; the vectors alone (3 values a row) take few
  const unsigned most = row_floats ? std::min(capacity, 16384) : std::min((3 * (capacity / kMergeWG) + 3), 1024);
  const dim3 wgs(most, std::max(1u, std::min(((unsigned)row_floats + kMergePart - 1) / kMergePart, 16384u / most)));
  const uintptr_t a0 = (uintptr_t)archive_rows, p0 = (uintptr_t)point_rows;
  const bool staged = row_floats && p0 < a0 + sizeof(float) * (size_t)capacity * row_floats &&
                      a0 < p0 + sizeof(float) * (size_t)m * row_floats;
  k_merge_out<<<wgs, kMergeWG, 0, st>>>(archive, archive_rows, capacity, points, point_rows, row_floats, pairs, staged, src,
                                       hdr, vec, rows);
  k_merge_in<<<wgs, kMergeWG, 0, st>>>(archive, archive_rows, capacity, point_rows, row_floats, pairs, staged, src, hdr, vec,
                                      rows, n_archive, overflow);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_select(int32_t S, const double* obj, int32_t n_sel, int32_t* sel, int32_t* dominated_by, void* stream) {
  if (S < 0 || n_sel < 0 || n_sel > S) return DSM_ERR_ARG;
  if (S > 8192) return DSM_ERR_CAPACITY;
  if (S == 0) return DSM_OK;
  if (!obj || (n_sel > 0 && !sel)) return DSM_ERR_ARG;
  k_select<<<1, kSelWG, sizeof(double) * S, (hipStream_t)stream>>>(S, obj, n_sel, sel, dominated_by);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_avs_update(int32_t n, float* mult, int32_t* nis, const double* sdr, int32_t nis_max, float eta, float lo,
                          float hi, void* stream) {
  if (n < 0 || !(eta > 0.f && eta < 1.f) || !(lo > 0.f && lo <= hi)) return DSM_ERR_ARG;
  if (n == 0) return DSM_OK;
  if (!mult || !nis || !sdr) return DSM_ERR_ARG;
  k_avs<<<(n + 255) / 256, 256, 0, (hipStream_t)stream>>>(n, mult, nis, sdr, nis_max, eta, lo, hi);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_multiplier_step(int32_t k, int32_t F, int32_t S, const uint8_t* accepted, const int32_t* cluster,
                               float* mult, float eta, float lo, float hi, void* stream) {
  if (k < 1 || F < 0 || S < 0 || !(eta > 0.f && eta < 1.f) || !(lo > 0.f && lo <= hi)) return DSM_ERR_ARG;
  if (F == 0) return DSM_OK;
  if (!mult || (S > 0 && !accepted) || (k > 1 && !cluster)) return DSM_ERR_ARG;
  k_multiplier_step<<<(k * F + 255) / 256, 256, 0, (hipStream_t)stream>>>(k, F, S, accepted, k > 1 ? cluster : nullptr,
                                                                        mult, eta, lo, hi);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_mark_improved(int32_t S, int32_t F, const uint8_t* accepted, uint8_t* improved, void* stream) {
  if (S < 0 || F < 0) return DSM_ERR_ARG;
  if (S == 0 || F == 0) return DSM_OK;
  if (!accepted || !improved) return DSM_ERR_ARG;
  k_mark_improved<<<(S + 255) / 256, 256, 0, (hipStream_t)stream>>>(S, F, accepted, improved);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_ams_shift(int32_t n, const double* mean, double* prev, double* shift, int32_t has_prev, void* stream) {
  if (n < 0) return DSM_ERR_ARG;
  if (n == 0) return DSM_OK;
  if (!mean || !prev || (has_prev && !shift)) return DSM_ERR_ARG;
  k_ams_shift<<<std::min(1024, (n + 255) / 256), 256, 0, (hipStream_t)stream>>>(n, mean, prev, shift, has_prev ? 1 : 0);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_single_objective_clusters(int32_t k, const double* means, int32_t S, const int32_t* assign, int32_t* so,
                                         void* stream) {
  if (k < 1 || k > kClusterMax || S < 0) return DSM_ERR_ARG;
  if (S == 0) return DSM_OK;
  if (!means || !assign || !so) return DSM_ERR_ARG;
  k_so_clusters<<<std::min(64, (S + 255) / 256), 256, 0, (hipStream_t)stream>>>(k, means, S, assign, so);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

dsm_status dsm_draw_donors(int32_t S, const int32_t* nis, int32_t nis_max, const int32_t* dominated_by, const float* u,
                           int32_t* donor, int32_t* n_forced, void* stream) {
  if (S < 0) return DSM_ERR_ARG;
  if (S > 8192) return DSM_ERR_CAPACITY;
  if (S == 0) return DSM_OK;
  if (!nis || !dominated_by || !u || !donor) return DSM_ERR_ARG;
  k_draw_donors<<<1, 1024, sizeof(int) * S, (hipStream_t)stream>>>(S, nis, nis_max, dominated_by, u, donor, n_forced);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

size_t dsm_forced_work_bytes(const dsm_problem* p, int32_t S) {
  if (!p || S < 0) return 0;
  return (size_t)S * (sizeof(float) * 6 * p->topo.P + sizeof(double) * 3 + sizeof(double) * 3 * p->topo.T);
}

dsm_status dsm_forced_replace(dsm_problem* p, int32_t S, float* X, double* obj, double* cache, const int32_t* donor,
                              const uint8_t* improved, int32_t* nis, void* work, int32_t* n_replaced, void* stream) {
  if (!p || S < 0) return DSM_ERR_ARG;
  if (S == 0) return DSM_OK;
  if (!X || !obj || !cache || !donor || !improved || !nis || !work) return DSM_ERR_ARG;
  const int row_x = 6 * p->topo.P, row_c = 3 * p->topo.T;
  float* wx = (float*)work;
  double* wobj = (double*)(wx + (size_t)S * row_x);  // row_x = 6 P floats: 8-byte aligned
  double* wcache = wobj + 3 * (size_t)S;
  hipStream_t st = (hipStream_t)stream;
  const dim3 grid((unsigned)std::min(64, (row_x + 3 + row_c + 255) / 256), (unsigned)S);
  k_forced_stage<<<grid, 256, 0, st>>>(S, row_x, row_c, X, obj, cache, donor, improved, wx, wobj, wcache);
  k_forced_apply<<<grid, 256, 0, st>>>(S, row_x, row_c, X, obj, cache, donor, improved, wx, wobj, wcache, nis,
                                       n_replaced);
  return hipGetLastError() == hipSuccess ? DSM_OK : DSM_ERR_DEVICE;
}

}  // extern "C"
