// gfx950 kernels of the dual simplex-mesh objective evaluator.
//
// Work decomposition (Sec. 2.2: the affected tetrahedra of a partial change
// are re-evaluated; Sec. 2.3: every objective is a sum of per-cell terms):
//   one workgroup per (FOS element, chunk of its affected tetrahedra,
//   solution) in partial evaluation, or per (chunk of tetrahedra, solution) in
//   full evaluation.  Its work units are (version, direction, tetrahedron,
//   batch of 64 voxel rows); each of the 4 waves takes a contiguous range of
//   units.  A wave computes the exact x-span of 64 rows (one row per lane),
//   prefix-sums the span lengths, and then sweeps the voxels of those rows 64
//   at a time, adjacent lanes on adjacent voxels, so that both the streamed
//   own-image reads and the trilinear gathers from the other image are
//   coalesced.
//
// Exactness: coordinates are lattice integers (1/128 voxel, |u| <= 2^16), so
// every orientation value and every face function evaluated at a voxel centre
// is an integer below 2^53 and FP64 arithmetic on it is exact; the voxel set of
// a tetrahedron is therefore decided bit-exactly.  Sampling and the
// dissimilarity sum are FP32 (per-lane compensated sums, FP64 across lanes).
#include <hip/hip_runtime.h>

#include "dsm_internal.h"

namespace dsm {

namespace {

__device__ __forceinline__ double dot3(const double a[3], const double b[3]) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

// Lattice value of one coordinate and its constraint bits.
__device__ __forceinline__ unsigned lattice_of(float x, int D, double& u) {
  if (!isfinite(x)) {
    u = 0.0;
    return DSM_FLAG_NONFINITE;
  }
  const double v = ((double)x + 0.5) * kLat;
  u = v;
  if (v != floor(v)) return DSM_FLAG_LATTICE;
  if (v < 0.0 || v > kLat * D) return DSM_FLAG_DOMAIN;
  return 0u;
}

// The constraint bits of lattice_of for coordinate x, in FP32: scaling by 128
// is exact, and (x + 0.5) 128 is a lattice integer in [0, 128 D] iff 128 x is
// one in [-64, 128 D - 64].  Coordinates that vanish next to 0.5 in FP64, whose
// spacing is 2^-53 above and 2^-54 below it (a tie at either end rounds to 0.5),
// count as 0, as they do there; x is set to 0 then.
__device__ __forceinline__ unsigned lattice_bits(float& x, int D) {
  if (x <= 0x1p-54f && x >= -0x1p-55f) x = 0.f;
  const float t = x * 128.f;
  if (!isfinite(x)) return DSM_FLAG_NONFINITE;
  if (t != floorf(t)) return DSM_FLAG_LATTICE;
  return t < -64.f || t > (float)(128 * D - 64) ? DSM_FLAG_DOMAIN : 0u;
}

// 6 x signed volume of (a, b, c, d); exact for lattice integers.
__device__ __forceinline__ double orient(const double a[3], const double b[3], const double c[3], const double d[3]) {
  const double u[3] = {b[0] - a[0], b[1] - a[1], b[2] - a[2]};
  const double v[3] = {c[0] - a[0], c[1] - a[1], c[2] - a[2]};
  const double w[3] = {d[0] - a[0], d[1] - a[1], d[2] - a[2]};
  const double cx = v[1] * w[2] - v[2] * w[1];
  const double cy = v[2] * w[0] - v[0] * w[2];
  const double cz = v[0] * w[1] - v[1] * w[0];
  return u[0] * cx + u[1] * cy + u[2] * cz;
}

// Blockid -> logical index so that each of the 8 XCDs (which receive
// workgroups round robin) processes one contiguous range of logical indices;
// consecutive logical indices share a FOS element and hence an image region.
// Index k on XCD x of n; -1 beyond the XCD's range.
__device__ __forceinline__ int xcd_logical(int x, int k, int n) {
  const int q = n >> 3, r = n & 7;
  return k < q + (x < r ? 1 : 0) ? x * q + min(x, r) + k : -1;
}

// Element order of a partial launch without a slot table (more than kOrderMax
// elements, or no room for one): every eighth element,
// starting from 0, then from 1, and so on.  The logical workgroup space is
// element-major and each XCD takes a contiguous range of it, so in mesh order
// the XCDs holding the border layers (whose points have smaller stars) would
// finish early; interleaved, every XCD takes elements from the whole mesh.
// Returns the element at position gp of that order, for G elements.
__device__ __forceinline__ int interleaved_group(int gp, int G) {
  int r = 0, base = 0;
  for (; r < 7; ++r) {
    const int cnt = (G - r + 7) >> 3;  // elements g < G with g % 8 == r
    if (gp < base + cnt) break;
    base += cnt;
  }
  return ((gp - base) << 3) + r;
}

// Makes LDS writes of some lanes visible to the other lanes of the same wave
// (and keeps the compiler from moving LDS accesses across this point).
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int kCtrl>
__device__ __forceinline__ double dpp64(double v) {
  const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), kCtrl, 0xF, 0xF, true);
  const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), kCtrl, 0xF, 0xF, true);
  return __hiloint2double(hi, lo);
}

__device__ __forceinline__ double lane_value(double v, int l) {
  return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), l), __builtin_amdgcn_readlane(__double2loint(v), l));
}

// Sum over the 64 lanes of a wave, all lanes active, in a fixed order: within
// each row of 16 lanes by DPP permutations, then over the four rows.
__device__ __forceinline__ double wave_sum(double v) {
  v += dpp64<0xB1>(v);   // quad_perm [1,0,3,2]
  v += dpp64<0x4E>(v);   // quad_perm [2,3,0,1]
  v += dpp64<0x141>(v);  // row_half_mirror: the other quad of 8 lanes
  v += dpp64<0x140>(v);  // row_mirror: the other 8 lanes of the row
  return (lane_value(v, 0) + lane_value(v, 16)) + (lane_value(v, 32) + lane_value(v, 48));
}

// Sum over the kFinishLanes lanes of a lane group, in a fixed butterfly order
// (every lane of the group ends with the same sum).
__device__ __forceinline__ double group_sum(double v) {
  for (int off = kFinishLanes / 2; off >= 1; off >>= 1) v += __shfl_xor(v, off, kFinishLanes);
  return v;
}

// Inclusive prefix sum over the 64 lanes of a wave, all lanes active: DPP
// shifts within rows of 16 lanes, then the row totals carried by the
// broadcasts of lanes 15 and 31.
__device__ __forceinline__ int wave_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);   // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);   // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);   // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);   // row_shr:8
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);  // row_bcast:15 into rows 1, 3
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);  // row_bcast:31 into rows 2, 3
  return v;
}

// Inclusive prefix maximum over the 64 lanes of a wave of values >= 0, all lanes active.
__device__ __forceinline__ int wave_incl_max(int v) {
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false));
  return v;
}

// Inclusive prefix sum within each row of 16 lanes (the lanes of a row active).
__device__ __forceinline__ int row16_incl_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);  // row_shr:1
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);  // row_shr:2
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);  // row_shr:4
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);  // row_shr:8
  return v;
}

// Parameters of one (tetrahedron, direction) for rasterising the own grid's
// voxels and mapping them into the other grid.  Lives in LDS, where it decides
// how many workgroups of the sweep a CU holds: 496 instead of 560 bytes here,
// voxel markers of a byte and no partial sums beside the coordinates let 6
// instead of 5 stay that sweep both versions of 8 tetrahedra (64^3, current
// terms recomputed: 1375 -> 1280 us).
constexpr int kMaxSlices = 64;  // slice-table capacity; taller tetrahedra enumerate bounding-box rows

struct RasterTet {
  // o_i(x,y,z) - thr_i = A x + C0 + CY y + CZ z at voxel (x,y,z): F[i] = (C0, CY, CZ, -1 / A or 0)
  double F[4][4];
  double M[3][4];  // own voxel coords -> other grid voxel coords: p' = M[.][3] + M[.][0..2] v
  int nrows;                       // candidate rows
  unsigned short zlo, nz, ylo, ny; // bounding box (slices, rows)
  unsigned char sliced;  // 1: candidate rows from the slice table, 0: every bounding-box row
  unsigned char pairs;   // slice table: 0 one row group per slice, 1 one per pair of slices
  unsigned short y0[kMaxSlices];      // first candidate row (its y) of each row group
  unsigned short rs[kMaxSlices + 1];  // exclusive prefix of candidate rows per row group (<= 64 * 512)
};
static_assert(sizeof(RasterTet) == 496, "LDS budget of the sweep");

// The x coefficient of a face, 128 times an integer below 2^34: exact from the
// rounding of its reciprocal.  And thr_i (setup_face).
__device__ __forceinline__ double face_A(const double F[4]) {
  return F[3] != 0.0 ? kLat * rint(-1.0 / (F[3] * kLat)) : 0.0;
}
__device__ __forceinline__ double face_thr(const double F[4]) {
  const bool pos = F[3] != 0.0 ? F[3] < 0.0 : (F[1] != 0.0 ? F[1] > 0.0 : F[2] > 0.0);
  return pos ? 0.0 : 1.0;
}

// The row of the lane's voxel, with m the lanes of a chunk where a row starts
// (mk: 1 on those) and `before` rows that start ahead of the chunk.
__device__ __forceinline__ int row_at(unsigned long long m, int mk, int before) {
  return (int)__builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32),
                                        __builtin_amdgcn_mbcnt_lo((unsigned)m, (unsigned)(before - 1))) + mk;
}

// Conservative row range [ya, yb] of the cross-section of the tetrahedron
// (own-grid lattice vertices L, integers below 2^17 and hence exact in FP32)
// with voxel slice z: the rows whose centres lie in the y-extent of the
// section polygon (every voxel of the closed tetrahedron in that slice does),
// whose vertices are the edge / plane intersections.  They are computed in
// FP32 with an approximate reciprocal, with an error of a few 1e-3 lattice
// units at most; the extent is widened by 1/2 lattice unit against it.  The
// exact spans decide the voxels.
__device__ __forceinline__ void slice_rows(const float L[4][3], int z, int Dy, int& ya, int& yb) {
  const float Uz = 128.f * z + 64.f;
  float lo = INFINITY, hi = -INFINITY;
  for (int a = 0; a < 4; ++a) {
    if (L[a][2] == Uz) {
      lo = fminf(lo, L[a][1]);
      hi = fmaxf(hi, L[a][1]);
    }
    for (int b = a + 1; b < 4; ++b) {
      const float za = L[a][2], zb = L[b][2];
      if ((za < Uz && zb > Uz) || (za > Uz && zb < Uz)) {
        const float y = fmaf((Uz - za) * __builtin_amdgcn_rcpf(zb - za), L[b][1] - L[a][1], L[a][1]);
        lo = fminf(lo, y);
        hi = fmaxf(hi, y);
      }
    }
  }
  if (lo > hi) {
    ya = 0;
    yb = -1;
    return;
  }
  ya = max(0, (int)ceilf((lo - 64.5f) * (1.f / 128.f)));
  yb = min(Dy - 1, (int)floorf((hi - 63.5f) * (1.f / 128.f)));
}

// Rasterisation parameters of the tetrahedron with own-grid vertices xo[4][3]
// and other-grid vertices xt[4][3] (voxel units, already validated on the
// lattice), in parts that run on different threads: the face function opposite
// each vertex, the three columns of the affine map's matrix, and the bounding
// box.  setup_slices (or setup_slices16) then runs on one wave, after these
// writes are visible to it, and fills the slice table and the map's offset.
// Differences of lattice coordinates are exact in FP32; every FP64 product and
// sum below is an exact integer.

// Face opposite vertex i: o_i(U) = G . U + K is the orientation with vertex i
// replaced by U (zero on the face, 6 x volume at vertex i), taken positive at
// vertex i.  U lies in the tetrahedron iff o_i(U) >= thr_i for all i, where
// thr_i = 0 if the first non-zero component of G_i (x, then y, then z) is
// positive and 1 otherwise: the top-left rule of Sec. 2.3.1 extended to 3-D by
// perturbing U by (+e, +e^2, +e^3).  Returns (L_i - L_j) . G before the sign is
// taken: for i = 0 this is minus 6 x the signed volume.
__device__ __forceinline__ double setup_face(const float* xo, int i, RasterTet& rt) {
  const int j = i == 0 ? 1 : 0, k = i <= 1 ? 2 : 1, l = i <= 2 ? 3 : 2;
  double Lj[3], a[3], b[3], d[3];
  for (int c = 0; c < 3; ++c) {
    const float xj = xo[3 * j + c];
    Lj[c] = (double)fmaf(xj, 128.f, 64.f);
    a[c] = (double)((xo[3 * k + c] - xj) * 128.f);
    b[c] = (double)((xo[3 * l + c] - xj) * 128.f);
    d[c] = (double)((xo[3 * i + c] - xj) * 128.f);
  }
  double g[3] = {a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]};
  const double s = dot3(g, d);
  if (s < 0.0)
    for (int c = 0; c < 3; ++c) g[c] = -g[c];
  const double K = -dot3(g, Lj);
  rt.F[i][1] = kLat * g[1];
  rt.F[i][2] = kLat * g[2];
  const bool pos = g[0] != 0.0 ? g[0] > 0.0 : (g[1] != 0.0 ? g[1] > 0.0 : g[2] > 0.0);
  rt.F[i][0] = 64.0 * (g[0] + g[1] + g[2]) + K - (pos ? 0.0 : 1.0);
  rt.F[i][3] = g[0] != 0.0 ? -1.0 / (kLat * g[0]) : 0.0;
  return s;
}

// Column c of M: M[r][c] = sum_k Oedge[r][k] * 128 adj(E)[k][c] / vol, E = own
// edge matrix (lattice), E[r][k] component r of edge k.
__device__ __forceinline__ void setup_column(const float* xo, const float* xt, int c, RasterTet& rt) {
  const int c1 = c == 2 ? 0 : c + 1, c2 = c == 0 ? 2 : c - 1;
  double m0[3], m1[3], m2[3];  // rows c, c + 1, c + 2 of E
  for (int k = 0; k < 3; ++k) {
    m0[k] = (double)((xo[3 * (k + 1) + c] - xo[c]) * 128.f);
    m1[k] = (double)((xo[3 * (k + 1) + c1] - xo[c1]) * 128.f);
    m2[k] = (double)((xo[3 * (k + 1) + c2] - xo[c2]) * 128.f);
  }
  // column c of adj(E): cofactors of row c of E
  const double adj[3] = {m1[1] * m2[2] - m1[2] * m2[1], m1[2] * m2[0] - m1[0] * m2[2], m1[0] * m2[1] - m1[1] * m2[0]};
  const double vol = dot3(m0, adj);
  for (int r = 0; r < 3; ++r) {
    double acc = 0.0;
    for (int k = 0; k < 3; ++k) acc += (double)(xt[3 * (k + 1) + r] - xt[r]) * adj[k];
    rt.M[r][c] = vol > 0.0 ? acc * kLat / vol : 0.0;
  }
}

__device__ __forceinline__ void setup_box(const float* xo, const int D[3], RasterTet& rt) {
  int lo[3], hi[3];
  for (int c = 1; c < 3; ++c) {
    const float a = fminf(fminf(xo[c], xo[3 + c]), fminf(xo[6 + c], xo[9 + c]));
    const float b = fmaxf(fmaxf(xo[c], xo[3 + c]), fmaxf(xo[6 + c], xo[9 + c]));
    // voxel i (centred at lattice 128 i + 64) lies in the extent iff a <= i <= b
    lo[c] = max(0, (int)ceilf(a));
    hi[c] = min(D[c] - 1, (int)floorf(b));
  }
  rt.zlo = (unsigned short)lo[2];
  rt.nz = (unsigned short)max(0, hi[2] - lo[2] + 1);
  rt.ylo = (unsigned short)lo[1];
  rt.ny = (unsigned short)max(0, hi[1] - lo[1] + 1);
}

// Candidate rows of the row group that starts at slice k: slice k alone
// (pairs = 0), or slices k and k + 1 for even k (pairs = 1), whose candidate
// rows alternate between the two slices over the union of their row ranges.
// [ya, yb] is slice k's row range; with pairs, lane ^ 1 holds slice k + 1's
// (called on both lanes).  Returns the group's first y in gya and its number of
// candidate rows in cnt (0 on lanes that start no group).
template <int kPairs>
__device__ __forceinline__ void group_rows(int ya, int yb, int k, int nz, int& gya, int& cnt) {
  int lo = ya, hi = yb, m = 1;
  if (kPairs) {
    const int oya = __shfl_xor(ya, 1, 64), oyb = __shfl_xor(yb, 1, 64);
    if (k + 1 < nz) {
      m = 2;
      if (oyb >= oya) {
        lo = yb >= ya ? min(ya, oya) : oya;
        hi = yb >= ya ? max(yb, oyb) : oyb;
      }
    }
  }
  gya = hi >= lo ? lo : 0;
  cnt = (k & kPairs) || k >= nz ? 0 : m * max(0, hi - lo + 1);
}

__device__ void setup_slices(const float* xo, const float* xt, const int D[3], int lane, RasterTet& rt) {
  const int nz = rt.nz;
  if (nz <= kMaxSlices) {
    // candidate rows of slice zlo + lane, prefix-summed over the slices
    int cnt = 0, ya = 0;
    if (lane < nz) {
      float L[4][3];
      for (int q = 0; q < 4; ++q)
        for (int c = 0; c < 3; ++c) L[q][c] = (xo[3 * q + c] + 0.5f) * 128.f;
      int yb;
      slice_rows(L, rt.zlo + lane, D[1], ya, yb);
      cnt = max(0, yb - ya + 1);
    }
    const int incl = wave_incl_scan(cnt);
    if (lane < nz) {
      rt.rs[lane] = (unsigned short)(incl - cnt);
      rt.y0[lane] = (unsigned short)ya;
    }
    if (lane == 63) {
      rt.rs[min(nz, kMaxSlices)] = (unsigned short)incl;
      rt.nrows = incl;
      rt.sliced = 1;
      rt.pairs = 0;
    }
  } else if (lane == 0) {
    rt.nrows = nz * rt.ny;
    rt.sliced = 0;
    rt.pairs = 0;
  }
  if (lane < 3) {
    const int r = lane;
    rt.M[r][3] = (double)xt[r] - (rt.M[r][0] * (double)xo[0] + rt.M[r][1] * (double)xo[1] + rt.M[r][2] * (double)xo[2]);
  }
  wave_sync();
}

// setup_slices on a group of 16 lanes (one DPP row, `sub` = lane within the
// group; all 16 lanes call it) for tetrahedra of few slices: slices in rounds of
// 16, the candidate-row prefix carried from round to round.  Returns the number
// of rows (on every lane of the group).  kPairs: row groups of slice pairs
// (group_rows).
template <int kPairs>
__device__ int setup_slices16(const float* xo, const float* xt, const int D[3], int lane, int sub, RasterTet& rt) {
  constexpr int pairs = kPairs;
  const int nz = rt.nz;
  int nrows;
  if (nz <= kMaxSlices) {
    float L[4][3];
    for (int q = 0; q < 4; ++q)
      for (int c = 0; c < 3; ++c) L[q][c] = (xo[3 * q + c] + 0.5f) * 128.f;
    int carry = 0;
    for (int base = 0; base < nz; base += 16) {
      const int k = base + sub;
      int ya = 0, yb = -1;
      if (k < nz) slice_rows(L, rt.zlo + k, D[1], ya, yb);
      int gya, cnt;
      group_rows<kPairs>(ya, yb, k, nz, gya, cnt);
      const int incl = row16_incl_scan(cnt);
      if (k < nz && !(k & pairs)) {
        rt.rs[k >> pairs] = (unsigned short)(carry + incl - cnt);
        rt.y0[k >> pairs] = (unsigned short)gya;
      }
      carry += __shfl(incl, lane | 15, 64);
    }
    nrows = carry;
    if (sub == 0) {
      rt.rs[(nz + pairs) >> pairs] = (unsigned short)carry;
      rt.nrows = carry;
      rt.sliced = 1;
      rt.pairs = pairs;
    }
  } else {
    nrows = nz * rt.ny;
    if (sub == 0) {
      rt.nrows = nrows;
      rt.sliced = 0;
      rt.pairs = 0;
    }
  }
  if (sub < 3) {
    const int r = sub;
    rt.M[r][3] = (double)xt[r] - (rt.M[r][0] * (double)xo[0] + rt.M[r][1] * (double)xo[1] + rt.M[r][2] * (double)xo[2]);
  }
  return nrows;
}

// Everything on one wave.
__device__ void setup_raster(const float* xo, const float* xt, const int D[3], int lane, RasterTet& rt) {
  if (lane < 4)
    setup_face(xo, lane, rt);
  else if (lane < 7)
    setup_column(xo, xt, lane - 4, rt);
  else if (lane == 7)
    setup_box(xo, D, rt);
  wave_sync();
  setup_slices(xo, xt, D, lane, rt);
}

// Exact x-span [x0, x1] (inclusive; empty if x0 > x1) of voxel row (y, z):
// every face's bound rounded by the reciprocal and corrected by evaluating the
// (integer) face function next to it.
__device__ __forceinline__ void row_span_exact(const RasterTet& rt, double y, double z, int Dx, int& x0, int& x1) {
  int lo = 0, hi = Dx - 1;
#pragma unroll 1
  for (int i = 0; i < 4; ++i) {
    const double A = face_A(rt.F[i]);
    const double h = rt.F[i][0] + rt.F[i][1] * y + rt.F[i][2] * z;  // need A x + h >= 0
    const double q = fmin(fmax(h * rt.F[i][3], -2.0), (double)Dx + 1.0);
    if (A > 0.0) {
      int x = (int)ceil(q);
      if (A * (x - 1) + h >= 0.0)
        x -= 1;
      else if (A * x + h < 0.0)
        x += 1;
      lo = max(lo, x);
    } else if (A < 0.0) {
      int x = (int)floor(q);
      if (A * (x + 1) + h >= 0.0)
        x += 1;
      else if (A * x + h < 0.0)
        x -= 1;
      hi = min(hi, x);
    } else if (h < 0.0) {
      lo = Dx;
      hi = -1;
    }
  }
  x0 = lo;
  x1 = hi;
}

// The same span for the 64 rows of a wave (used lanes: `used`).  The largest
// lower and the smallest upper bound over the faces, each a real number within
// 1e-12 of its exact value, decide the span by one rounding unless one of them
// lies within 1e-9 of an integer; only then (faces through voxel centres) the
// wave takes the exact form.  4 instead of about 28 instructions per face and
// row: the row spans are half of the sweep's instructions on tetrahedra of
// tens to hundreds of voxels.
__device__ __forceinline__ void row_span(const RasterTet& rt, bool used, int y, int z, int Dx, int& x0, int& x1) {
  const double yd = (double)y, zd = (double)z;
  double f[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int k = 0; k < 4; ++k) f[i][k] = rt.F[i][k];
  double lo = -0.5, hi = (double)Dx - 0.5;  // no integer: the image's own ends are certain
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const double h = f[i][0] + f[i][1] * yd + f[i][2] * zd;
    const int side = __builtin_amdgcn_readfirstlane(__double2hiint(f[i][3]));  // a branch of the whole wave
    if (side < 0)  // A > 0
      lo = fmax(lo, h * f[i][3]);
    else if (side > 0)
      hi = fmin(hi, h * f[i][3]);
    else if (h < 0.0)
      lo = (double)Dx + 0.5;
  }
  lo = fmin(lo, (double)Dx + 0.5);
  hi = fmax(hi, -1.5);
  const double fl = __builtin_amdgcn_fract(lo), fh = __builtin_amdgcn_fract(hi);
  if (__ballot(used && (fabs(fl - 0.5) > 0.5 - 1e-9 || fabs(fh - 0.5) > 0.5 - 1e-9))) {
    row_span_exact(rt, yd, zd, Dx, x0, x1);
  } else {
    x0 = (int)ceil(lo);
    x1 = (int)floor(hi);
  }
}

// One compacted (non-empty) row: both fields are read from one LDS address.
struct RowRec {
  // x: own-image linear index minus start (as int bits); yzw: mapped position
  // of the span's first voxel (sweep), or its x minus start, y, z (as int bits)
  float4 rec;
  int start;   // exclusive prefix of span lengths
  int pad[3];
};

struct WaveRows {
  RowRec row[64];
  // per voxel slot of the current 128-voxel chunk pair: 1 where a row starts (in build_rows the row's group)
  unsigned char marker[128];
};

// A unit's rows find their row groups by a walk over the groups that start
// inside the unit (no LDS round trip) for up to this many, else by marks in LDS
// and a prefix maximum, whose cost does not grow with them.
constexpr int kWalkGroups = 3;

// Computes the spans of rows [64 b, 64 b + 64) of rt, stores the non-empty
// ones compacted (in row order) in wr, and returns the number of voxels.  With
// a slice table, row r is y-major within its row group: y = y0 + (r - rs) of
// the group's slice, or, for a pair of slices, rows alternate between them,
// (y0, z), (y0, z + 1), (y0 + 1, z), ...; every bounding-box row otherwise,
// y = ylo + r % ny.  The linear index of a span's first voxel (x0, y, z) is
// lin = base + z sz + y sy + x0; wr stores lin minus the row's start, or with
// kOwnBytes the byte offset of its value in the bordered z-pair image minus 8
// times the start (the second row of a pair reads the second value of the
// element that holds the first row's voxel, so the two rows share the own
// image's cache lines) and the mapped position of the first voxel,
// M (x0, y, z, 1) + shift.  *my_start receives the first voxel index of this
// lane's row, or a large negative value if it is empty.  kPairs must equal
// rt.pairs (a compile-time copy, so that the slice-by-slice order pays
// nothing for the other).
template <bool kOwnBytes, int kPairs>
__device__ __forceinline__ int build_rows(const RasterTet& rt, int b, int lane, const int D[3], int sy, int sz,
                                          int base, float shift, WaveRows& wr, int* my_start) {
  const int r0 = b * 64, r = r0 + lane;
  int len = 0, lin = 0;
  float bx = 0.f, by = 0.f, bz = 0.f;
  int y, z, h = 0;
  if (rt.sliced) {
    // lane k holds row group k's first candidate row and first y; row r lies
    // in the last group that starts at or before r: the group of the unit's
    // first row, advanced over the groups that start inside the unit (in order)
    const int nz = rt.nz, ng = (nz + kPairs) >> kPairs;
    const int rsk = lane < ng ? (int)rt.rs[lane] : 0x7fffffff;
    const int y0k = lane < ng ? (int)rt.y0[lane] : 0;
    // row r of group k, which starts at row s with y = ys
    auto place = [&](int k, int s, int ys) {
      const int rr = r - s;
      if (kPairs) {
        const int two = 2 * k + 1 < nz ? 1 : 0;  // the group is a pair of slices
        h = rr & two;
        y = ys + (rr >> two);
        z = rt.zlo + 2 * k + h;
      } else {
        y = ys + rr;
        z = rt.zlo + k;
      }
    };
    const int jb = __popcll(__ballot(rsk <= r0)) - 1;  // rs[0] = 0
    unsigned long long inside = __ballot(rsk > r0 && rsk < r0 + 64);
    if (__popcll(inside) <= kWalkGroups) {
      place(jb, __builtin_amdgcn_readlane(rsk, jb), __builtin_amdgcn_readlane(y0k, jb));
      while (inside) {
        const int k = __builtin_ctzll(inside);
        inside &= inside - 1;
        const int s = __builtin_amdgcn_readlane(rsk, k);
        if (r >= s) place(k, s, __builtin_amdgcn_readlane(y0k, k));
      }
    } else {
      // every group with rows marks its first one; a row's group is the
      // largest mark at or before it
      wr.marker[lane] = 0;
      wave_sync();
      const int at = rsk - r0;
      if (lane < ng && at > 0 && at < 64 && rt.rs[lane + 1] > rsk) wr.marker[at] = (unsigned char)lane;
      wave_sync();
      const int k = wave_incl_max(lane == 0 ? jb : (int)wr.marker[lane]);
      place(k, (int)rt.rs[k], (int)rt.y0[k]);
    }
  } else {
    y = rt.ylo + r % rt.ny;
    z = rt.zlo + r / rt.ny;
  }
  int x0, x1;
  row_span(rt, r < rt.nrows, y, z, D[0], x0, x1);
  if (r < rt.nrows) {
    if (x1 >= x0) {
      len = x1 - x0 + 1;
      lin = base + z * sz + y * sy + x0;
      if (kOwnBytes) lin = (lin - h * sz) * 8 + 4 * h;
      if (kOwnBytes) {
        const double v[3] = {(double)x0, (double)y, (double)z};
        bx = (float)(rt.M[0][3] + rt.M[0][0] * v[0] + rt.M[0][1] * v[1] + rt.M[0][2] * v[2] + shift);
        by = (float)(rt.M[1][3] + rt.M[1][0] * v[0] + rt.M[1][1] * v[1] + rt.M[1][2] * v[2] + shift);
        bz = (float)(rt.M[2][3] + rt.M[2][0] * v[0] + rt.M[2][1] * v[1] + rt.M[2][2] * v[2] + shift);
      }
    }
  }
  const int incl = wave_incl_scan(len);
  const int start = incl - len;
  const unsigned long long ne = __ballot(len > 0);
  const int slot = __builtin_amdgcn_mbcnt_hi((unsigned)(ne >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)ne, 0u));
  wave_sync();
  if (len > 0) {
    wr.row[slot].start = start;
    if (!kOwnBytes) {
      bx = __int_as_float(x0 - start);
      by = __int_as_float(y);
      bz = __int_as_float(z);
    }
    wr.row[slot].rec = make_float4(__int_as_float(kOwnBytes ? lin - 8 * start : lin - start), bx, by, bz);
  }
  wave_sync();
  *my_start = len > 0 ? start : -(1 << 30);
  return __builtin_amdgcn_readlane(incl, 63);
}

__device__ __forceinline__ __amdgpu_buffer_rsrc_t image_rsrc(const float* p, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)p, (short)0, bytes, 0x00020000);
}

typedef float float4v __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float4v load4(__amdgpu_buffer_rsrc_t r, int voff, int soff) {
  return __builtin_bit_cast(float4v, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

__device__ __forceinline__ float load1(__amdgpu_buffer_rsrc_t r, int voff) {
  return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(r, voff, 0, 0));
}

// Per-wave constants of the sampled (other) image.  Images use the bordered
// z-pair layout: element (x', y', z') holds the values at (x'-1, y'-1, z'-1)
// and (x'-1, y'-1, z'), border-replicated, so one 16-byte load at element
// (ix, iy, iz) returns the taps (x, z), (x, z+1), (x+1, z), (x+1, z+1) of the
// cell of shifted position q = p + 1 with ix = floor(q_x) etc.
struct SampleCtx {
  __amdgpu_buffer_rsrc_t own, oth;  // bordered image buffers
  int sx8, sxy8;                    // byte strides of y and z
  float tau;
};

// The 8 trilinear taps of the sampled image around shifted position
// (px, py, pz) = p + 1, p in [-0.5, D-0.5] up to rounding: truncation is floor,
// and the replicated border stands in for clamping p to [0, D-1].
struct Taps {
  float4v ty0, ty1;  // (x,z) (x,z+1) (x+1,z) (x+1,z+1) at y and at y+1
  float fx, fy, fz;
};

__device__ __forceinline__ Taps load_taps(const SampleCtx& c, float px, float py, float pz) {
  Taps t;
  const int ix = (int)px, iy = (int)py, iz = (int)pz;
  t.fx = __builtin_amdgcn_fractf(px);
  t.fy = __builtin_amdgcn_fractf(py);
  t.fz = __builtin_amdgcn_fractf(pz);
  const int voff = (int)(__umul24((unsigned)iy, (unsigned)c.sx8) + (__umul24((unsigned)iz, (unsigned)c.sxy8) + ((unsigned)ix << 3)));
  t.ty0 = load4(c.oth, voff, 0);
  t.ty1 = load4(c.oth, voff, c.sx8);
  return t;
}

// Sec. 2.3.1 contribution of a voxel pair: squared intensity difference, and
// the maximal difference 1 where an empty voxel meets a non-empty one; the
// empty indicator of the sampled position is interpolated like the intensity.
__device__ __forceinline__ float contrib_of(const SampleCtx& c, float a, const Taps& tp) {
  const float4v ty0 = tp.ty0, ty1 = tp.ty1;
  const float fx = tp.fx, fy = tp.fy, fz = tp.fz;
  struct {
    float x, y;
  } t00{ty0.x, ty0.z}, t10{ty1.x, ty1.z}, t01{ty0.y, ty0.w}, t11{ty1.y, ty1.w};
  const float tau = c.tau;
  const float i00 = fmaf(fx, t00.y - t00.x, t00.x), i10 = fmaf(fx, t10.y - t10.x, t10.x);
  const float i01 = fmaf(fx, t01.y - t01.x, t01.x), i11 = fmaf(fx, t11.y - t11.x, t11.x);
  const float i0 = fmaf(fy, i10 - i00, i00), i1 = fmaf(fy, i11 - i01, i01);
  const float b = fmaf(fz, i1 - i0, i0);
  // empty indicators of the 8 taps as wave masks (combined in scalar registers)
  constexpr int kOLE = 5;  // ordered less-or-equal
  const unsigned long long m000 = __builtin_amdgcn_fcmpf(t00.x, tau, kOLE), m100 = __builtin_amdgcn_fcmpf(t00.y, tau, kOLE);
  const unsigned long long m010 = __builtin_amdgcn_fcmpf(t10.x, tau, kOLE), m110 = __builtin_amdgcn_fcmpf(t10.y, tau, kOLE);
  const unsigned long long m001 = __builtin_amdgcn_fcmpf(t01.x, tau, kOLE), m101 = __builtin_amdgcn_fcmpf(t01.y, tau, kOLE);
  const unsigned long long m011 = __builtin_amdgcn_fcmpf(t11.x, tau, kOLE), m111 = __builtin_amdgcn_fcmpf(t11.y, tau, kOLE);
  const unsigned long long all = m000 & m100 & m010 & m110 & m001 & m101 & m011 & m111;
  const unsigned long long any = m000 | m100 | m010 | m110 | m001 | m101 | m011 | m111;
  const bool ea = a <= tau;
  const float d = a - b;
  // where the 8 taps of every lane agree, the interpolated indicator is the
  // first tap's: m is 0 or 1 and the contribution is d^2 or 1 (the values of
  // the general formula below)
  float res = ea != (t00.x <= tau) ? 1.f : d * d;
  if (any & ~all) {  // some lane has taps on both sides of tau: interpolate its indicator
    const float e000 = t00.x <= tau ? 1.f : 0.f, e100 = t00.y <= tau ? 1.f : 0.f;
    const float e010 = t10.x <= tau ? 1.f : 0.f, e110 = t10.y <= tau ? 1.f : 0.f;
    const float e001 = t01.x <= tau ? 1.f : 0.f, e101 = t01.y <= tau ? 1.f : 0.f;
    const float e011 = t11.x <= tau ? 1.f : 0.f, e111 = t11.y <= tau ? 1.f : 0.f;
    const float m00 = fmaf(fx, e100 - e000, e000), m10 = fmaf(fx, e110 - e010, e010);
    const float m01 = fmaf(fx, e101 - e001, e001), m11 = fmaf(fx, e111 - e011, e011);
    const float m0 = fmaf(fy, m10 - m00, m00), m1 = fmaf(fy, m11 - m01, m01);
    const float eb = fmaf(fz, m1 - m0, m0);
    const float m = fabsf((ea ? 1.f : 0.f) - eb);
    res = fmaf(1.f - m, d * d, m);
  }
  return res;
}

// Samples voxels q0 + lane (row r0) and q0 + 64 + lane (row r1) of the
// compacted rows and adds their contributions to the lane's compensated sum.
// Both samples' loads are issued before either is used.  With TAIL, slots
// past the last voxel repeat the last voxel (same row) and are weighted 0.
template <bool TAIL>
__device__ __forceinline__ void sweep_pair(const WaveRows& wr, const SampleCtx& sc, int q0, int nvox, int lane, int r0,
                                           int r1, float jx, float jy, float jz, float& sum, float& comp) {
  const int qa = q0 + lane, qb = qa + 64;
  const int ea = TAIL ? min(qa, nvox - 1) : qa, eb = TAIL ? min(qb, nvox - 1) : qb;
  const RowRec ra = wr.row[r0], rb = wr.row[r1];
  const float foa = (float)(ea - ra.start), fob = (float)(eb - rb.start);
  const float ava = load1(sc.own, __float_as_int(ra.rec.x) + (ea << 3));
  const Taps ta = load_taps(sc, fmaf(jx, foa, ra.rec.y), fmaf(jy, foa, ra.rec.z), fmaf(jz, foa, ra.rec.w));
  const float avb = load1(sc.own, __float_as_int(rb.rec.x) + (eb << 3));
  const Taps tb = load_taps(sc, fmaf(jx, fob, rb.rec.y), fmaf(jy, fob, rb.rec.z), fmaf(jz, fob, rb.rec.w));
  const float ca = contrib_of(sc, ava, ta);
  const float cb = contrib_of(sc, avb, tb);
  const float c = TAIL ? (qa < nvox ? ca : 0.f) + (qb < nvox ? cb : 0.f) : ca + cb;
  const float y = c - comp;
  const float t = sum + y;
  comp = (t - sum) - y;
  sum = t;
}

// The last chunk of a row batch when at most 64 voxels are left: voxel
// q0 + lane only, slots past the last voxel repeat it and are weighted 0.
__device__ __forceinline__ void sweep_one(const WaveRows& wr, const SampleCtx& sc, int q0, int nvox, int lane, int r0,
                                          float jx, float jy, float jz, float& sum, float& comp) {
  const int qa = q0 + lane;
  const int ea = min(qa, nvox - 1);
  const RowRec ra = wr.row[r0];
  const float foa = (float)(ea - ra.start);
  const float ava = load1(sc.own, __float_as_int(ra.rec.x) + (ea << 3));
  const Taps ta = load_taps(sc, fmaf(jx, foa, ra.rec.y), fmaf(jy, foa, ra.rec.z), fmaf(jz, foa, ra.rec.w));
  const float ca = contrib_of(sc, ava, ta);
  const float c = qa < nvox ? ca : 0.f;
  const float y = c - comp;
  const float t = sum + y;
  comp = (t - sum) - y;
  sum = t;
}

// Length in mm of the vector d (voxel units).
__device__ __forceinline__ double len_mm(const double sp[3], double d0, double d1, double d2) {
  const double dx = d0 * sp[0], dy = d1 * sp[1], dz = d2 * sp[2];
  return sqrt(dx * dx + dy * dy + dz * dz);
}

// x / 3 for sums x of three lattice coordinates (multiples of 1/128 below
// 1536): a product and one correction, equal to the division for each of them,
// at a quarter of its instructions.
__device__ __forceinline__ double third(double x) {
  const double q = x * (1.0 / 3.0);
  return fma(fma(-3.0, q, x), 1.0 / 3.0, q);
}

// Sec. 2.3.2: the deformation term of one tetrahedron sums over its 6 edges
// (weighted 1/k_e) and its 4 spokes (from each vertex to the centroid of the
// opposite face) the squared length difference in mm between the two grids.
// Length of edge k < 6 or spoke k - 6 of vertices V[4][3]; differences and sums
// of three lattice coordinates are exact in FP32.
constexpr int kLengths = 10;
__device__ __forceinline__ double length_of(const double sp[3], const float* V, int k) {
  double d[3];
  if (k < 6) {
    const int i = (0x211000 >> (4 * k)) & 15, j = (0x332321 >> (4 * k)) & 15;  // 01 02 03 12 13 23
    for (int c = 0; c < 3; ++c) d[c] = (double)(V[3 * i + c] - V[3 * j + c]);
  } else {
    const int q = k - 6, i = q == 0 ? 1 : 0, j = q <= 1 ? 2 : 1, l = q <= 2 ? 3 : 2;
    for (int c = 0; c < 3; ++c) d[c] = (double)V[3 * q + c] - third((double)(V[3 * i + c] + V[3 * j + c] + V[3 * l + c]));
  }
  return len_mm(sp, d[0], d[1], d[2]);
}

// Sec. 2.3.3: guidance point i of image g, if it lies inside a tetrahedron
// (own vertices Vo, set up in rt), is mapped into the other image (vertices Vt)
// and contributes the squared mm distance to the nearest point of the same
// correspondence there (0 if it lies outside).
__device__ __forceinline__ double guidance_point(const DevProblem& pr, int g, int i, int match, const float* Vt,
                                                 const RasterTet& rt) {
  const double* U = pr.gpt[g] + 3 * i;
  const double p[3] = {U[0] * (1.0 / kLat) - 0.5, U[1] * (1.0 / kLat) - 0.5, U[2] * (1.0 / kLat) - 0.5};
  // two passes over the faces, one at a time: few points come here, and the
  // registers of this function decide how many waves of the sweep a SIMD holds
  double vol = 0.0;  // exact: the o_i at any point sum to 6 x the volume
  bool in = true;
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    const double over = rt.F[q][0] + face_A(rt.F[q]) * p[0] + rt.F[q][1] * p[1] + rt.F[q][2] * p[2];
    in = in && over >= 0.0;
    vol += over + face_thr(rt.F[q]);
  }
  if (!in) return 0.0;
  double x[3] = {0, 0, 0};
#pragma unroll 1
  for (int q = 0; q < 4; ++q) {
    const double over = rt.F[q][0] + face_A(rt.F[q]) * p[0] + rt.F[q][1] * p[1] + rt.F[q][2] * p[2];
    const double lam = (over + face_thr(rt.F[q])) / vol;
    for (int c = 0; c < 3; ++c) x[c] += lam * (double)Vt[3 * q + c];
  }
  double best = INFINITY;
  const int corr = pr.gcorr[g][i];
  const int j0 = match < 0 ? 0 : match, j1 = match < 0 ? pr.ng[1 - g] : match + 1;
#pragma unroll 1
  for (int j = j0; j < j1; ++j) {
    if (pr.gcorr[1 - g][j] != corr) continue;
    const double* r = pr.gpt[1 - g] + 3 * j;
    best = fmin(best, len_mm(pr.sp, x[0] - (r[0] * (1.0 / kLat) - 0.5), x[1] - (r[1] * (1.0 / kLat) - 0.5),
                             x[2] - (r[2] * (1.0 / kLat) - 0.5)));
  }
  return best < INFINITY ? best * best : 0.0;
}

// ------------------------------------------------------------ LDS layout

struct EvalLayout {
  size_t tet, xyz, units, part, waves, rts, total;
};

__host__ __device__ inline size_t align16(size_t x) { return (x + 15) & ~size_t(15); }

__host__ __device__ inline EvalLayout eval_layout(int maxA, int nver) {
  static_assert(sizeof(double) * kWaves * 2 <= sizeof(float) * 24, "part lies over xyz");
  EvalLayout L;
  size_t o = 0;
  L.tet = o;
  o = align16(o + sizeof(int) * maxA);
  L.xyz = o;  // [nver][maxA][2][4][3] float; in the sweep [nver*2*maxA][kWaves] double (part)
  L.part = o;
  o = align16(o + sizeof(float) * 24 * (size_t)nver * maxA);
  L.units = o;  // [nver*2*maxA + 1] int (unit counts, then exclusive prefix)
  o = align16(o + sizeof(int) * (2 * (size_t)nver * maxA + 1));
  L.waves = o;  // [kWaves] WaveRows
  o = align16(o + sizeof(WaveRows) * kWaves);
  L.rts = o;  // [nver*2*maxA] RasterTet, one per (version, direction, tetrahedron)
  o = align16(o + sizeof(RasterTet) * 2 * (size_t)nver * maxA);
  L.total = o;
  return L;
}

// exclusive scan of n ints in LDS by wave 0 (n entries, writes n+1 with total)
__device__ void lds_exclusive_scan(int* v, int n, int tid) {
  if (tid < 64) {
    int carry = 0;
    for (int base = 0; base < n; base += 64) {
      const int x = base + tid < n ? v[base + tid] : 0;
      const int incl = wave_incl_scan(x);
      if (base + tid < n) v[base + tid] = carry + incl - x;
      carry += __builtin_amdgcn_readlane(incl, 63);
    }
    if (tid == 0) v[n] = carry;
  }
}

__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }
__device__ __forceinline__ float uniformf(float v) {
  return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}

// Source of vertex vid's coordinates in grid gr for version v (0 = candidate,
// 1 = current) of solution s, group g.
__device__ __forceinline__ const float* vertex_src(const EvalArgs& a, int s, int g, int v, int vid, int gr) {
  const float* src = a.X + (((size_t)s * 2 + gr) * a.pr.P + vid) * 3;
  if (v == 0 && a.partial) {
    const int pb = a.fos_off[g], pe = a.fos_off[g + 1], ncand = a.fos_off[a.G];
    for (int k = pb; k < pe; ++k)
      if (a.fos_pts[k] == vid) src = a.cand + (((size_t)s * ncand + k) * 2 + gr) * 3;
  }
  return src;
}

__device__ __forceinline__ int group_tet(const EvalArgs& a, int g, int i) {
  return a.partial ? a.aff[(size_t)g * a.maxA + i] : g * kFullChunk + i;
}

// ------------------------------------------------------------ voxel sweep kernel

// All objective terms of every (version, tetrahedron) of one chunk of at most
// a.pchunk affected tetrahedra (partial evaluation) or of one group of
// kFullChunk tetrahedra (full evaluation) of one solution.  Writes the terms of
// the evaluated version to a.terms_out (where given) and, in partial mode, the
// chunk's sums per version to sums[((s*G + g)*nchunk + c)*nver + v][3], its
// constraint flags and its candidate voxel count to cflags / ccount
// [S][G][nchunk]; k_finish combines them.  In full mode the constraint bits of
// the group go to the solution's flags: the fold check's own two kernels over
// points and tetrahedra took 12 of 680 us for 48 solutions of 187x203x77.
// The deformation and guidance terms are evaluated here, where the chunk's
// coordinates and face functions are in LDS: in a kernel of their own they
// waited for the coordinates 77 % of the time (99 us of the 191 us of a 32^3
// partial evaluation, 420 of 4,750 us of a class of the 50^3 phantom).
// Workgroups are numbered (group, chunk, solution) with the solution fastest,
// so the workgroups resident on an XCD sweep the same few tetrahedra of many
// solutions and share their image region in L2; partial launches number the
// chunks that exist by the slot table (k_slots).
// ROWS: the row order, 0 slice by slice, 1 in slice pairs (both fixed
// at compile time), 2 a.row_pairs read at run time (a batch of problems with
// both orders).
template <int PARTIAL, int ROWS>
__device__ __forceinline__ void sweep_body(const EvalArgs& a, int logical, unsigned char* smem) {
  const DevProblem& pr = a.pr;
  const int tid = threadIdx.x, lane = tid & 63, wave = uniform(tid >> 6);
  const int nchunk = PARTIAL ? a.nchunk : 1;
  // g and the counts below are the same on every lane; saying so keeps the
  // values derived from them (the direction of an entry, hence the image
  // buffer a load reads) in scalar registers
  int g, c, s;
  if (PARTIAL && a.slots) {
    const int slot = logical / a.S;
    const int2 gc = a.slots[1 + slot];
    g = uniform(gc.x);
    c = uniform(gc.y);
    s = logical - slot * a.S;
  } else {
    const int gl = logical / (a.S * nchunk), rem = logical - gl * (a.S * nchunk);
    g = uniform(PARTIAL ? interleaved_group(gl, a.G) : gl);
    c = rem / a.S;
    s = rem - c * a.S;
  }
  const int nver = a.nver;
  const EvalLayout Lay = eval_layout(kMaxChunk, nver);
  int* s_tet = (int*)(smem + Lay.tet);
  float* s_xyz = (float*)(smem + Lay.xyz);
  int* s_units = (int*)(smem + Lay.units);
  double* s_part = (double*)(smem + Lay.part);
  WaveRows* s_rows = (WaveRows*)(smem + Lay.waves);
  RasterTet* s_rts = (RasterTet*)(smem + Lay.rts);
  __shared__ unsigned s_flags;
  __shared__ unsigned s_count[kWaves];
  __shared__ unsigned s_bad[2 * kMaxChunk];   // per (version, tetrahedron): bit gr set if grid gr has a coordinate off the lattice
  __shared__ double s_dg[2 * kMaxChunk][2];   // per (version, tetrahedron): deformation and guidance term
  // before the sweep, in the space of its rows
  double* s_len = (double*)s_rows;                   // [nver*na][kLengths] length differences
  constexpr int kGuidSums = kWG / (2 * kMaxChunk);   // partial sums of a guidance term and grid, whatever nver
  double* s_guid = s_len + 2 * kMaxChunk * kLengths;  // [nver na][2][kGuidSums] partial guidance terms
  double* s_w = s_guid + 2 * kWG;                    // [na][6] edge weights
  int* s_in = (int*)(s_w + 6 * kMaxChunk);           // [2 nver na] 1 if the entry is set up
  static_assert(sizeof(WaveRows) * kWaves >= sizeof(double) * (2 * kMaxChunk * kLengths + 2 * kWG + 6 * kMaxChunk) + sizeof(int) * 4 * kMaxChunk,
                "set-up space");

  // this chunk's tetrahedra: slots [i0, i0 + na) of the group
  const int na_all = uniform(PARTIAL ? a.aff_cnt[g] : min(kFullChunk, pr.T - g * kFullChunk));
  const int i0 = c * (PARTIAL ? a.pchunk : kFullChunk);
  if (na_all <= i0) return;  // malformed element (count -1) or no tetrahedra in this chunk: k_finish sets the flags
  if (PARTIAL && a.mask && a.mask[(size_t)s * a.G + g] == 0) return;  // not requested
  const int na = min(PARTIAL ? a.pchunk : kFullChunk, na_all - i0);
  if (tid == 0) s_flags = 0u;
  if (tid < kWaves) s_count[tid] = 0u;
  if (tid < 2 * kMaxChunk) s_bad[tid] = 0u;
  for (int i = tid; i < na; i += kWG) s_tet[i] = group_tet(a, g, i0 + i);
  __syncthreads();

  // vertex coordinates of every (version, tetrahedron, grid, vertex), one
  // thread per component, and their constraint bits (lattice, box, border pins)
  const int nvt = nver * na;
  for (int e = tid; e < nvt * 24; e += kWG) {
    const int vt = e / 24, r = e - vt * 24, gr = r / 12, q = (r - gr * 12) / 3, ax = r % 3;
    const int v = vt >= na ? 1 : 0, i = vt - v * na;
    const int vid = ((const int*)&pr.tets[s_tet[i]])[q];
    const unsigned pin = pr.pin[vid];
    float x = vertex_src(a, s, g, v, vid, gr)[ax];
    unsigned fl = lattice_bits(x, ax == 0 ? pr.D[0] : (ax == 1 ? pr.D[1] : pr.D[2]));
    s_xyz[e] = x;
    if (fl)
      atomicOr(&s_bad[vt], 1u << gr);
    else if (((pin >> ax) & 1 && x != -0.5f) || ((pin >> (3 + ax)) & 1 && x != (float)(ax == 0 ? pr.D[0] : (ax == 1 ? pr.D[1] : pr.D[2])) - 0.5f))
      fl = DSM_FLAG_BORDER;
    if (v == 0 && fl) atomicOr(&s_flags, fl);
  }
  if (wave == kWaves - 1 && lane < 6 * na) s_w[lane] = pr.tet_w[6 * (size_t)s_tet[lane / 6] + lane % 6];
  __syncthreads();

  // set-up of every (version, direction, tetrahedron) entry and the lengths of
  // the deformation term.  Direction 0 = target voxels mapped into the source
  // (forward), 1 = source voxels into the target.  Entry e's own-grid vertices
  // are at entry_xyz(e) + 12 own, the other grid's at + 12 (1 - own).  The
  // tasks are grouped by kind, 64 to a wave, so that no wave runs two kinds
  // side by side: matrix columns, faces, lengths, boxes.
  const int nent = 2 * nvt;
  auto entry_vt = [&](int e, int& own) {  // entries are ordered (version, direction, tetrahedron)
    const int v = e >= 2 * na ? 1 : 0, r = e - v * 2 * na, dir = r >= na ? 1 : 0;
    own = 1 - dir;
    return v * na + (r - dir * na);
  };
  auto entry_xyz = [&](int e, int& own) { return s_xyz + (size_t)entry_vt(e, own) * 24; };
  {
    const int nj = (3 * nent + 63) >> 6, nf = (4 * nent + 63) >> 6, nl = (kLengths * nvt + 63) >> 6, nb = (nent + 63) >> 6;
    for (int job = wave; job < nj + nf + nl + nb; job += kWaves) {
      if (job < nj) {
        const int t = job * 64 + lane, e = t / 3;
        int own;
        if (e < nent && s_bad[entry_vt(e, own)] == 0u) {
          const float* xyz = entry_xyz(e, own);
          setup_column(xyz + own * 12, xyz + (1 - own) * 12, t - 3 * e, s_rts[e]);
        }
      } else if (job < nj + nf) {
        const int t = (job - nj) * 64 + lane, e = t >> 2;
        int own;
        if (e < nent) {
          const int vt = entry_vt(e, own);
          const unsigned bad = s_bad[vt];
          int ok = 0;
          if (!((bad >> own) & 1)) {
            const bool pos = setup_face(s_xyz + (size_t)vt * 24 + own * 12, t & 3, s_rts[e]) < 0.0;  // read for face 0
            ok = pos && bad == 0u ? 1 : 0;
            if (!pos && (t & 3) == 0 && e < 2 * na)  // evaluated version only
              atomicOr(&s_flags, own == 0 ? DSM_FLAG_INV_MOVING : DSM_FLAG_INV_FIXED);
          }
          if ((t & 3) == 0) s_in[e] = ok;
        }
      } else if (job < nj + nf + nl) {
        const int t = (job - nj - nf) * 64 + lane, vt = t / kLengths, k = t - vt * kLengths;
        if (vt < nvt) {
          const float* xyz = s_xyz + (size_t)vt * 24;
          s_len[t] = length_of(pr.sp, xyz, k) - length_of(pr.sp, xyz + 12, k);
        }
      } else {
        const int e = (job - nj - nf - nl) * 64 + lane;
        int own;
        if (e < nent && s_bad[entry_vt(e, own)] == 0u) setup_box(entry_xyz(e, own) + own * 12, pr.D, s_rts[e]);
      }
    }
  }
  __syncthreads();
  // guidance points, kWG / (2 nver kMaxChunk) lanes per (version, tetrahedron,
  // grid) sharing its image's points: each is first tested against the
  // tetrahedron's bounding box (exactly, on the lattice), which holds few.
  // Point i goes into partial sum i % kGuidSums, two to a lane where two
  // versions are swept, so a tetrahedron's term has the same bits either way
  // (no barrier parts this from the slice tables: what the waves read here, they
  // do not write there)
  const int gper = kWG / (2 * kMaxChunk * nver);
  const bool guided = pr.ng[0] + pr.ng[1] > 0;
  if (guided) {
    const int tg = tid / gper, vt = tg >> 1, gr = tg & 1, first = tid - tg * gper;
    const int e = vt < nvt ? (vt >= na ? na : 0) + vt + (1 - gr) * na : 0;  // the entry of grid gr's own voxels
    double* sums = s_guid + tg * kGuidSums;
    for (int q = first; q < kGuidSums; q += gper) sums[q] = 0.0;
    if (vt < nvt && s_in[e]) {
      const float *Vo = s_xyz + (size_t)vt * 24 + gr * 12, *Vt = s_xyz + (size_t)vt * 24 + (1 - gr) * 12;
      float lo[3], hi[3];
      for (int k = 0; k < 3; ++k) {
        lo[k] = fmaf(fminf(fminf(Vo[k], Vo[3 + k]), fminf(Vo[6 + k], Vo[9 + k])), 128.f, 64.f);
        hi[k] = fmaf(fmaxf(fmaxf(Vo[k], Vo[3 + k]), fmaxf(Vo[6 + k], Vo[9 + k])), 128.f, 64.f);
      }
      for (int i = first; i < pr.ng[gr]; i += gper) {
        const float4 u = pr.gbox[gr][i];
        if ((u.x >= lo[0]) & (u.x <= hi[0]) & (u.y >= lo[1]) & (u.y <= hi[1]) & (u.z >= lo[2]) & (u.z <= hi[2]))
          sums[i % kGuidSums] += guidance_point(pr, gr, i, __float_as_int(u.w), Vt, s_rts[e]);
      }
    }
  }
  if (wave == kWaves - 1 && lane < nvt) {  // deformation: edges weighted 1/k_e, then spokes
    const double *len = s_len + kLengths * lane, *w = s_w + 6 * (lane >= na ? lane - na : lane);
    double def = 0.0;
    for (int k = 0; k < 6; ++k) def += w[k] * len[k] * len[k];
    for (int k = 6; k < kLengths; ++k) def += len[k] * len[k];
    s_dg[lane][0] = def;
  }
  // slice tables, 16 lanes per entry, and the units
  for (int e0 = wave * 4; e0 < nent; e0 += kWaves * 4) {
    const int e = e0 + (lane >> 4), sub = lane & 15;
    int nunits = 0;
    if (e < nent && s_in[e]) {
      int own;
      const float* xyz = entry_xyz(e, own);
      const float *xo = xyz + own * 12, *xt = xyz + (1 - own) * 12;
      const int nrows = ROWS == 2 ? (a.row_pairs ? setup_slices16<1>(xo, xt, pr.D, lane, sub, s_rts[e])
                                                 : setup_slices16<0>(xo, xt, pr.D, lane, sub, s_rts[e]))
                                  : setup_slices16<ROWS>(xo, xt, pr.D, lane, sub, s_rts[e]);
      nunits = (nrows + 63) >> 6;
    }
    if (e < nent && sub == 0) s_units[e] = nunits;
  }
  __syncthreads();
  for (int e = tid; e < nent * kWaves; e += kWG) s_part[e] = 0.0;
  lds_exclusive_scan(s_units, nent, tid);
  if (wave == kWaves - 1 && lane < nvt) {
    double guid = 0.0;
    if (guided)
      for (int k = 0; k < 2 * kGuidSums; ++k) guid += s_guid[2 * kGuidSums * lane + k];
    s_dg[lane][1] = guid;
  }
  __syncthreads();
  const int total_units = uniform(s_units[nent]);

  // ---- voxel sweep
  SampleCtx sc;
  sc.sx8 = 8 * pr.ex;
  sc.sxy8 = 8 * pr.exy;
  sc.tau = pr.tau;
  const int own_base = pr.exy + pr.ex + 1;  // element of voxel (0, 0, 0)
  const __amdgpu_buffer_rsrc_t rs[2] = {image_rsrc(pr.img[0], pr.img_bytes), image_rsrc(pr.img[1], pr.img_bytes)};
  WaveRows& wr = s_rows[wave];
  const RasterTet* rtp = s_rts;
  int cur = -1;
  float jx = 0.f, jy = 0.f, jz = 0.f;
  unsigned counted = 0u;
  float sum = 0.f, comp = 0.f;  // compensated per-lane sum of the current (version, direction, tetrahedron)
  // each wave takes one contiguous range of units, so it sets up few tetrahedra
  const int u_begin = (wave * total_units) / kWaves, u_end = ((wave + 1) * total_units) / kWaves;
  for (int u = u_begin; u < u_end; ++u) {
    int e = cur < 0 ? 0 : cur;
    while (uniform(s_units[e + 1]) <= u) ++e;
    e = uniform(e);
    if (e != cur) {
      if (cur >= 0) {
        const double tot = wave_sum((double)sum - (double)comp);
        if (lane == 0) s_part[(size_t)cur * kWaves + wave] = tot;  // a wave's units of an entry are consecutive
        sum = comp = 0.f;
      }
      cur = e;
      const int r = e - (e / (2 * na)) * 2 * na, dir = r / na;
      const int own = 1 - dir;
      rtp = s_rts + e;
      jx = uniformf((float)rtp->M[0][0]);
      jy = uniformf((float)rtp->M[1][0]);
      jz = uniformf((float)rtp->M[2][0]);
      sc.own = own ? rs[1] : rs[0];
      sc.oth = own ? rs[0] : rs[1];
    }
    const int b = u - uniform(s_units[cur]);
    int my_start;
    const int nvox = uniform(ROWS == 2 ? (rtp->pairs ? build_rows<true, 1>(*rtp, b, lane, pr.D, pr.ex, pr.exy, own_base, 1.0f, wr, &my_start)
                                                     : build_rows<true, 0>(*rtp, b, lane, pr.D, pr.ex, pr.exy, own_base, 1.0f, wr, &my_start))
                                        : build_rows<true, ROWS>(*rtp, b, lane, pr.D, pr.ex, pr.exy, own_base, 1.0f, wr, &my_start));
    int carry = 0;  // non-empty rows that start before the current chunk
    for (int q0 = 0; q0 < nvox; q0 += 128) {
      // voxels q0 + lane and q0 + 64 + lane: rows starting in this pair of
      // chunks are marked, then counted below each slot with a ballot
      ((unsigned short*)wr.marker)[lane] = 0;
      wave_sync();
      const unsigned pos = (unsigned)(my_start - q0);
      if (pos < 128u) wr.marker[pos] = 1;
      wave_sync();
      const int mk0 = wr.marker[lane], mk1 = wr.marker[64 + lane];
      const unsigned long long M0 = __ballot(mk0 != 0), M1 = __ballot(mk1 != 0);
      const int before = carry + __popcll(M0);
      const int r0 = row_at(M0, mk0, carry), r1 = row_at(M1, mk1, before);
      carry = before + __popcll(M1);
      if (q0 + 128 <= nvox)
        sweep_pair<false>(wr, sc, q0, nvox, lane, r0, r1, jx, jy, jz, sum, comp);
      else if (q0 + 64 >= nvox)
        sweep_one(wr, sc, q0, nvox, lane, r0, jx, jy, jz, sum, comp);
      else
        sweep_pair<true>(wr, sc, q0, nvox, lane, r0, r1, jx, jy, jz, sum, comp);
    }
    if (cur < 2 * na) counted += (unsigned)nvox;  // version 0 (candidate) voxels
  }
  if (cur >= 0) {
    const double tot = wave_sum((double)sum - (double)comp);
    if (lane == 0) s_part[(size_t)cur * kWaves + wave] = tot;
  }
  if (lane == 0) s_count[wave] = counted;
  __syncthreads();

  // terms, kMaxChunk lanes of wave 0 per version (zero where the tetrahedron
  // has a coordinate off the lattice), and their sums over the chunk in a fixed
  // butterfly order
  if (wave == 0 && lane < nver * kMaxChunk) {
    const int v = lane / kMaxChunk, i = lane - v * kMaxChunk, vt = v * na + i;
    double term[3] = {0.0, 0.0, 0.0};
    if (i < na && s_bad[vt] == 0u) {
      for (int dir = 0; dir < 2; ++dir)
        for (int w = 0; w < kWaves; ++w) term[0] += s_part[((size_t)(v * 2 + dir) * na + i) * kWaves + w];
      term[1] = s_dg[vt][0];
      term[2] = s_dg[vt][1];
    }
    if (v == 0 && i < na && a.terms_out) {
      double* o = a.terms_out + ((size_t)s * pr.T + s_tet[i]) * 3;
      for (int k = 0; k < 3; ++k) o[k] = term[k];
    }
    if (PARTIAL) {
      for (int k = 0; k < 3; ++k) term[k] = group_sum(term[k]);
      const size_t ci = ((size_t)s * a.G + g) * nchunk + c;
      if (i < 3) a.sums[(ci * nver + v) * 3 + i] = i == 0 ? term[0] : (i == 1 ? term[1] : term[2]);
    }
  }
  if (!PARTIAL && tid == 0 && s_flags) atomicOr(&a.flags[s], s_flags);
  if (PARTIAL && tid == 0) {
    const size_t ci = ((size_t)s * a.G + g) * nchunk + c;
    a.cflags[ci] = s_flags;
    unsigned tot = 0u;
    for (int w = 0; w < kWaves; ++w) tot += s_count[w];
    a.ccount[ci] = tot;
  }
}

// EU: the waves per SIMD that the instructions are ordered for.  Both orders
// take 58 to 60 registers, which leaves room for 8; but where LDS holds fewer
// workgroups (two versions) or the launch has fewer, the order for 8, which
// brings a wave's loads and their uses closer together, is the slower one: 64^3
// recomputed 1305 against 1280 us, 32^3 with 16 solutions 64.8 against 62.3, but
// a class of the phantom 3,150 against 3,225 us and 512x512x100 164.6 against
// 165.4 ms (7 waves, from 70 registers: 62.5, 3,420 and 168.5).
template <int PARTIAL, int ROWS, int EU>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(EU, 8))) void k_sweep(EvalArgs a, int first) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int n = PARTIAL && a.slots ? a.S * a.slots[0].x : a.S * a.G * (PARTIAL ? a.nchunk : 1);
  const int logical = xcd_logical(blockIdx.x & 7, (first + (int)blockIdx.x) >> 3, n);
  if (logical >= 0) sweep_body<PARTIAL, ROWS>(a, logical, smem);
}

// Several problems in one launch.  Each job's workgroup range is split into 8
// equal contiguous parts, part x running on XCD x (hardware workgroup ids go
// round-robin over the XCDs): xcd_off[j] is the first per-XCD slot of job j,
// and a job of at most n workgroups takes ceil(n / 8) slots on every XCD, the
// surplus slots exiting at once.  So every XCD gets an eighth of every job
// (jobs of very different tetrahedron sizes would otherwise load the XCDs
// unevenly), and within a part the workgroups of one element's solutions stay
// together.
// Ordered for 8 waves per SIMD (7: 5,760 us for four uneven problems at half
// resolution, 8: 5,650).  ROWS as for sweep_body.
template <int ROWS>
__global__ __launch_bounds__(kWG) __attribute__((amdgpu_waves_per_eu(8, 8))) void k_sweep_batch(
    const EvalArgs* __restrict__ jobs, const int* __restrict__ xcd_off, int n_jobs, int first) {
  extern __shared__ __align__(16) unsigned char smem[];
  const int x = blockIdx.x & 7, k = (first + (int)blockIdx.x) >> 3;
  int j = 0;
  while (j + 1 < n_jobs && xcd_off[j + 1] <= k) ++j;
  j = uniform(j);
  const EvalArgs& a = jobs[j];
  const int n = uniform(a.slots ? a.S * a.slots[0].x : a.S * a.G * a.nchunk);
  const int logical = xcd_logical(x, k - uniform(xcd_off[j]), n);
  if (logical >= 0) sweep_body<1, ROWS>(a, logical, smem);
}

// ------------------------------------------------------------ finishing kernel

// The normalised sums, flags and voxel count of a (group, solution) pair of a
// partial evaluation from those of its chunks, in chunk order, and the sums of
// the current terms: the chunks' second version, or the cached terms of the
// affected tetrahedra, added chunk by chunk in the sweep's order: equal terms
// give equal sums, so a change that moves nothing has a delta of exactly 0 in
// deformation and guidance.  One group of kFinishLanes lanes per pair.
constexpr int kFinishRounds = 4;
__device__ __forceinline__ void finish_body(const EvalArgs& a, int logical, int lane) {
  const DevProblem& pr = a.pr;
  const int g = logical / a.S, s = logical - g * a.S;
  const int na = a.aff_cnt[g];
  const size_t oi = (size_t)s * a.G + g;
  if (na < 0 || (a.mask && a.mask[oi] == 0)) {
    if (lane < 3) {
      a.part_new[oi * 3 + lane] = 0.0;
      a.part_old[oi * 3 + lane] = 0.0;
    }
    if (lane == 0) {
      a.flags[oi] = na < 0 ? DSM_FLAG_BAD_FOS : DSM_FLAG_SKIPPED;
      if (a.vcount) a.vcount[oi] = 0u;
    }
    return;
  }
  // lanes 0..2 the evaluated version, 3..5 the current one where it was swept;
  // lane 6 the flags, lane 7 the counts
  const size_t c0 = oi * a.nchunk;
  const int nc = (na + a.pchunk - 1) / a.pchunk, nval = 3 * a.nver;
  double acc = 0.0;
  unsigned bits = 0u;
  if (lane < nval) {
#pragma unroll 4
    for (int c = 0; c < nc; ++c) acc += a.sums[(c0 + c) * nval + lane];
  } else if (lane == 6) {
    for (int c = 0; c < nc; ++c) bits |= a.cflags[c0 + c];
    a.flags[oi] = bits;
  } else if (lane == 7 && a.vcount) {
    for (int c = 0; c < nc; ++c) bits += a.ccount[c0 + c];
    a.vcount[oi] = bits;
  }
  if (a.nver == 1) {
    // kFinishRounds chunks' loads at a time: the loads that depend on one
    // another, not their number, are the time
    double old[3] = {0.0, 0.0, 0.0};
    for (int c = 0; c < nc; c += kFinishRounds) {
      int id[kFinishRounds];
      double t[kFinishRounds][3];
#pragma unroll
      for (int u = 0; u < kFinishRounds; ++u) {
        const int i = (c + u) * a.pchunk + lane;
        id[u] = lane < a.pchunk && i < na ? a.aff[(size_t)g * a.maxA + i] : -1;
      }
#pragma unroll
      for (int u = 0; u < kFinishRounds; ++u)
        for (int k = 0; k < 3; ++k) t[u][k] = id[u] >= 0 ? a.terms_in[((size_t)s * pr.T + id[u]) * 3 + k] : 0.0;
#pragma unroll
      for (int u = 0; u < kFinishRounds; ++u)
        if (c + u < nc)
          for (int k = 0; k < 3; ++k) old[k] += group_sum(t[u][k]);
    }
    if (lane >= 3 && lane < 6) acc = lane == 3 ? old[0] : (lane == 4 ? old[1] : old[2]);
  }
  if (lane < 3)
    a.part_new[oi * 3 + lane] = acc * pr.norm[lane];
  else if (lane < 6)
    a.part_old[oi * 3 + lane - 3] = acc * pr.norm[lane - 3];
}
static_assert(kFinishLanes == 8, "lanes of a pair by value");

// Each workgroup of 64 lanes takes kFinishPairs consecutive pairs.
__global__ __launch_bounds__(64) void k_finish(EvalArgs a, int n_pairs) {
  const int pair = blockIdx.x * kFinishPairs + (threadIdx.x / kFinishLanes);
  if (pair < n_pairs) finish_body(a, pair, threadIdx.x % kFinishLanes);
}

// Several problems: wg_off [n_jobs + 1] are the jobs' first workgroups, a job
// of n pairs taking ceil(n / kFinishPairs) of them.
__global__ __launch_bounds__(64) void k_finish_batch(const EvalArgs* __restrict__ jobs, const int* __restrict__ wg_off,
                                                     int n_jobs) {
  int j = 0;
  while (j + 1 < n_jobs && wg_off[j + 1] <= (int)blockIdx.x) ++j;
  const EvalArgs& a = jobs[j];
  const int pair = ((int)blockIdx.x - wg_off[j]) * kFinishPairs + (int)(threadIdx.x / kFinishLanes);
  if (pair < a.S * a.G) finish_body(a, pair, threadIdx.x % kFinishLanes);
}

// ------------------------------------------------------------ small kernels

__global__ void k_fill_u32(uint32_t* p, int64_t n, uint32_t v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

// Sec. 2.3.4 per point: lattice, box and border pins, both grids.
__global__ void k_fold_points(DevProblem pr, int S, const float* __restrict__ X, uint32_t* flags) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)S * pr.P) return;
  const int s = (int)(e / pr.P), p = (int)(e - (int64_t)s * pr.P);
  const int idx[3] = {p % pr.n[0], (p / pr.n[0]) % pr.n[1], p / (pr.n[0] * pr.n[1])};
  unsigned fl = 0u;
  for (int gr = 0; gr < 2; ++gr)
    for (int c = 0; c < 3; ++c) {
      double u;
      const unsigned fc = lattice_of(X[(((size_t)s * 2 + gr) * pr.P + p) * 3 + c], pr.D[c], u);
      fl |= fc;
      if (!fc && ((idx[c] == 0 && u != 0.0) || (idx[c] == pr.n[c] - 1 && u != kLat * pr.D[c]))) fl |= DSM_FLAG_BORDER;
    }
  if (fl) atomicOr(&flags[s], fl);
}

// Sec. 2.3.4 per tetrahedron: exact orientation in both grids.
__global__ void k_fold_tets(DevProblem pr, int S, const float* __restrict__ X, uint32_t* flags, int* first_bad) {
  const int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x;
  if (e >= (int64_t)S * pr.T) return;
  const int s = (int)(e / pr.T), t = (int)(e - (int64_t)s * pr.T);
  const int4 tv = pr.tets[t];
  const int vid[4] = {tv.x, tv.y, tv.z, tv.w};
  unsigned fl = 0u;
  for (int gr = 0; gr < 2; ++gr) {
    double L[4][3];
    unsigned bad = 0u;
    for (int q = 0; q < 4; ++q)
      for (int c = 0; c < 3; ++c) bad |= lattice_of(X[(((size_t)s * 2 + gr) * pr.P + vid[q]) * 3 + c], pr.D[c], L[q][c]);
    if (bad) continue;
    if (!(orient(L[0], L[1], L[2], L[3]) > 0.0)) fl |= gr == 0 ? DSM_FLAG_INV_MOVING : DSM_FLAG_INV_FIXED;
  }
  if (fl) {
    atomicOr(&flags[s], fl);
    if (first_bad) atomicMin(&first_bad[s], t);
  }
}

__global__ void k_first_bad_fix(int S, int* first_bad) {
  const int s = blockIdx.x * blockDim.x + threadIdx.x;
  if (s < S && first_bad[s] == 0x7fffffff) first_bad[s] = -1;
}

// Affected tetrahedra of element f with points fos_pts[b .. e): the sorted
// union of the points' stars, written to out (at most maxA); the count, or -1
// if it would exceed maxA.  One thread, insertion into the sorted prefix: the
// path for elements whose stars hold more than kAffCap entries.
__device__ int affected_serial(const DevProblem& pr, int b, int e, const int* __restrict__ fos_pts, int maxA,
                               int* out) {
  int n = 0;
  for (int k = b; k < e; ++k) {
    const int p = fos_pts[k];
    for (int j = pr.star_off[p]; j < pr.star_off[p + 1]; ++j) {
      const int t = pr.star[j];
      int pos = n;
      while (pos > 0 && out[pos - 1] > t) --pos;
      if (pos > 0 && out[pos - 1] == t) continue;
      if (n >= maxA) return -1;
      for (int m = n; m > pos; --m) out[m] = out[m - 1];
      out[pos] = t;
      ++n;
    }
  }
  return n;
}

constexpr int kAffCap = 1024;  // words of an element's bitmap, or its star entries sorted, in LDS

// Affected sets of the FOS elements (Sec. 2.2: the tetrahedra to re-evaluate
// when the element's points move): the distinct ids of its points' stars in
// ascending order; aff_cnt[f] = their number, or -1 for a malformed element or
// one whose set would exceed maxA.  One wave per element.  On meshes of up to
// 32 kAffCap tetrahedra the wave marks the ids in a bitmap in LDS and lists the
// marked ones; on larger ones it sorts the star entries (bitonic) and keeps the
// first of every run of equal ids.  The length of the chain bounds it: with the
// points read one after the other and the sort, a call took 12.6 us for
// 4-point elements, with a lane to a point and the bitmap 4.6.
__global__ __launch_bounds__(64) void k_affected(DevProblem pr, int F, const int* __restrict__ fos_off,
                                                 const int* __restrict__ fos_pts, int max_pts, int maxA, int* aff,
                                                 int* aff_cnt) {
  __shared__ int s_c[kAffCap];
  const int f = blockIdx.x, lane = threadIdx.x;
  const int b = fos_off[f], e = fos_off[f + 1];
  int* out = aff + (size_t)f * maxA;
  const bool marks = pr.T <= 32 * kAffCap;
  const int words = marks ? (pr.T + 2047) / 2048 : 0;  // of a lane
  for (int w = 0; w < words; ++w) s_c[64 * w + lane] = 0;
  bool bad = b < 0 || e < b || e - b > max_pts;
  int total = 0;
  for (int k0 = b; !bad && k0 < e; k0 += 64) {  // 64 points at a time, a lane each
    const int p = k0 + lane < e ? fos_pts[k0 + lane] : 0;
    bad = __any(p < 0 || p >= pr.P);
    if (bad) break;
    const int so = pr.star_off[p], n = k0 + lane < e ? pr.star_off[p + 1] - so : 0;
    const int incl = wave_incl_scan(n), all = __builtin_amdgcn_readlane(incl, 63);
    for (int i = lane; i < all; i += 64) {  // an entry's point is the last one whose entries start at or before it
      int at = 0;
      for (int k = 0; k < min(64, e - k0); ++k) {
        const int first = __builtin_amdgcn_readlane(incl - n, k);
        if (i >= first) at = __builtin_amdgcn_readlane(so, k) + i - first;
      }
      const int t = pr.star[at];
      if (marks)
        atomicOr((unsigned*)&s_c[t >> 5], 1u << (t & 31));
      else if (total + i < kAffCap)
        s_c[total + i] = t;
    }
    total += all;
  }
  if (bad) {
    if (lane == 0) aff_cnt[f] = -1;
    return;
  }
  if (!marks && total > kAffCap) {
    if (lane == 0) aff_cnt[f] = affected_serial(pr, b, e, fos_pts, maxA, out);
    return;
  }
  __syncthreads();
  if (marks) {
    int cnt = 0;
    for (int w = 0; w < words; ++w) cnt += __popc((unsigned)s_c[words * lane + w]);
    const int incl = wave_incl_scan(cnt), n_marked = __builtin_amdgcn_readlane(incl, 63);
    if (lane == 0) aff_cnt[f] = n_marked > maxA ? -1 : n_marked;
    if (n_marked > maxA) return;
    int pos = incl - cnt;
    for (int w = words * lane; w < words * (lane + 1); ++w)
      for (unsigned m = (unsigned)s_c[w]; m; m &= m - 1) out[pos++] = 32 * w + __builtin_ctz(m);
    return;
  }
  int n2 = 1;
  while (n2 < total) n2 <<= 1;
  for (int i = total + lane; i < n2; i += 64) s_c[i] = 0x7fffffff;
  __syncthreads();
  for (int k = 2; k <= n2; k <<= 1)
    for (int j = k >> 1; j > 0; j >>= 1) {
      for (int i = lane; i < n2; i += 64) {
        const int ixj = i ^ j;
        if (ixj > i) {
          const int a = s_c[i], c = s_c[ixj];
          if ((i & k) == 0 ? a > c : a < c) {
            s_c[i] = c;
            s_c[ixj] = a;
          }
        }
      }
      __syncthreads();
    }
  // lane l keeps the run starts among entries [l * chunk, (l + 1) * chunk)
  const int chunk = (total + 63) / 64;
  const int lo = min(lane * chunk, total), hi = min(lo + chunk, total);
  int cnt = 0;
  for (int i = lo; i < hi; ++i) cnt += i == 0 || s_c[i] != s_c[i - 1];
  const int incl = wave_incl_scan(cnt);
  const int n_unique = __builtin_amdgcn_readlane(incl, 63);
  if (n_unique > maxA) {
    if (lane == 0) aff_cnt[f] = -1;
    return;
  }
  int pos = incl - cnt;
  for (int i = lo; i < hi; ++i)
    if (i == 0 || s_c[i] != s_c[i - 1]) out[pos++] = s_c[i];
  if (lane == 0) aff_cnt[f] = n_unique;
}

// Full evaluation: fixed-order sum of the per-tetrahedron terms of each solution.
__global__ __launch_bounds__(kWG) void k_full_reduce(DevProblem pr, const double* __restrict__ terms, double* obj) {
  __shared__ double red[3][kWG];
  const int s = blockIdx.x, tid = threadIdx.x;
  double acc[3] = {0, 0, 0};
  for (int t = tid; t < pr.T; t += kWG)
    for (int c = 0; c < 3; ++c) acc[c] += terms[((size_t)s * pr.T + t) * 3 + c];
  for (int c = 0; c < 3; ++c) red[c][tid] = acc[c];
  __syncthreads();
  for (int w = kWG / 2; w >= 1; w >>= 1) {
    if (tid < w)
      for (int c = 0; c < 3; ++c) red[c][tid] += red[c][tid + w];
    __syncthreads();
  }
  if (tid < 3) obj[(size_t)s * 3 + tid] = red[tid][0] * pr.norm[tid];
}

// Owner map of one grid (test hook): every voxel of every tetrahedron's exact
// voxel set claims its owner entry.
__global__ __launch_bounds__(kWG) void k_owner(DevProblem pr, const float* __restrict__ Xg, int* owner, int* overlap) {
  __shared__ WaveRows rows[kWaves];
  __shared__ RasterTet rts[kWaves];
  __shared__ float xo[12];
  const int t = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int4 tv = pr.tets[t];
  const int vid[4] = {tv.x, tv.y, tv.z, tv.w};
  double L[4][3];
  unsigned bad = 0u;
  for (int q = 0; q < 4; ++q)
    for (int c = 0; c < 3; ++c) bad |= lattice_of(Xg[(size_t)vid[q] * 3 + c], pr.D[c], L[q][c]);
  if (bad || !(orient(L[0], L[1], L[2], L[3]) > 0.0)) return;
  if (threadIdx.x < 12) xo[threadIdx.x] = Xg[(size_t)vid[threadIdx.x / 3] * 3 + threadIdx.x % 3];
  __syncthreads();
  RasterTet& rt = rts[wave];
  setup_raster(xo, xo, pr.D, lane, rt);
  const int nb = (rt.nrows + 63) >> 6;
  for (int b = wave; b < nb; b += kWaves) {
    WaveRows& wr = rows[wave];
    int my_start;
    const int nvox = build_rows<false, 0>(rt, b, lane, pr.D, pr.D[0], pr.DxDy, 0, 0.0f, wr, &my_start);
    int carry = 0;
    for (int q0 = 0; q0 < nvox; q0 += 64) {
      wr.marker[lane] = 0;
      wave_sync();
      const unsigned pos = (unsigned)(my_start - q0);
      if (pos < 64u) wr.marker[pos] = 1;
      wave_sync();
      const int mk = wr.marker[lane];
      const unsigned long long M = __ballot(mk != 0);
      const int r = row_at(M, mk, carry);
      carry += __popcll(M);
      const int q = q0 + lane;
      if (q < nvox) {
        const int idx = __float_as_int(wr.row[r].rec.x) + q;
        const int prev = atomicCAS(&owner[idx], -1, t);
        if (prev != -1) atomicAdd(overlap, 1);
      }
    }
  }
}

// FP64 trilinear sample of a bordered image at voxel (i, j, k) plus d voxels,
// clamped to [0, D-1] per axis (the resampling of the objectives, Sec. 2.3.1):
// the element of cell (i, j, k) is (i + 1, j + 1, k + 1) and holds the values
// at k and k + 1, its right neighbour those at i + 1.  cell64 turns d into the
// fractions and returns the byte offset of the element.
__device__ __forceinline__ int cell64(const DevProblem& pr, const int v[3], double d[3]) {
  int i0[3];
  for (int a = 0; a < 3; ++a) {
    i0[a] = min(max(v[a] + (int)floor(d[a]), 0), pr.D[a] - 2);
    d[a] = fmin(fmax(d[a] - (double)(i0[a] - v[a]), 0.0), 1.0);
  }
  return (int)(__umul24((unsigned)(i0[1] + 1), 8u * (unsigned)pr.ex) + (unsigned)(i0[2] + 1) * (8u * (unsigned)pr.exy) +
               ((unsigned)(i0[0] + 1) << 3));
}
// p, q: the elements (x, z) (x, z+1) (x+1, z) (x+1, z+1) at y and y + 1.
__device__ __forceinline__ double trilinear64(const double f[3], float4v p, float4v q) {
  auto mix = [](double t, double u, double v) { return fma(t, v, (1.0 - t) * u); };
  const double c0 = mix(f[1], mix(f[0], p[0], p[2]), mix(f[0], q[0], q[2]));
  const double c1 = mix(f[1], mix(f[0], p[1], p[3]), mix(f[0], q[1], q[3]));
  return mix(f[2], c0, c1);
}

// Clears the outputs of dsm_transform to NaN, for the voxels that no usable
// tetrahedron covers.  With `check` only where there may be some: if every
// coordinate lies on the lattice, grid `own` keeps its border points on the
// box and none of its tetrahedra is inverted, those tile the box and every
// voxel is written.  Each workgroup looks at the whole grid by itself: no flag
// to clear, no second launch, and no memory that two calls could share.
__global__ __launch_bounds__(1024) void k_transform_clear(DevProblem pr, int own, const float* __restrict__ X2, int check,
                                                          uint32_t* dvf, int64_t nd, uint32_t* warped, int64_t nw) {
  if (check) {
    bool bad = false;
    for (int e = threadIdx.x; e < 2 * pr.P; e += blockDim.x) {
      const int gr = e >= pr.P, v = e - gr * pr.P;
      const unsigned pin = pr.pin[v];
      for (int c = 0; c < 3; ++c) {
        float x = X2[3 * (size_t)e + c];
        bad |= lattice_bits(x, pr.D[c]) != 0u;
        bad |= gr == own && ((pin >> c & 1 && x != -0.5f) || (pin >> (3 + c) & 1 && x != (float)pr.D[c] - 0.5f));
      }
    }
    const float* Xo = X2 + (size_t)own * 3 * pr.P;
    for (int t = threadIdx.x; t < pr.T; t += blockDim.x) {
      const int4 tv = pr.tets[t];
      const int vid[4] = {tv.x, tv.y, tv.z, tv.w};
      double L[4][3];
      for (int q = 0; q < 4; ++q)
        for (int c = 0; c < 3; ++c) L[q][c] = ((double)Xo[3 * (size_t)vid[q] + c] + 0.5) * kLat;
      bad |= !(orient(L[0], L[1], L[2], L[3]) > 0.0);
    }
    if (!__syncthreads_or(bad)) return;
  }
  const int64_t step = (int64_t)gridDim.x * blockDim.x;
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < nd + nw; i += step)
    (i < nd ? dvf + i : warped + (i - nd))[0] = 0x7fc00000u;
}

// The piecewise-affine map of one solution (Sec. 2.1) at every voxel of image
// `own`: each tetrahedron of grid `own` rasterises its exact voxel set (the
// same spans as the objectives) and maps every voxel centre, in FP64, onto the
// same tetrahedron of the other grid.  Writes the displacement (voxel units)
// and the other image sampled there.  `parts` workgroups per tetrahedron share
// its units of 64 rows.  The barycentric coordinates of a row's first voxel
// come from the face functions that its span came from, exact integers over
// the volume; along the row the displacement is linear, 3 multiply-adds per
// voxel.  As four determinants of every voxel (about 250 FP64 instructions)
// they made the kernel take 428 us at 512x512x100; 285 us now, for 206 MB read
// and 419 MB written.  Memory bounds it there: with only the displacements
// written it takes 75 us, with only the image 155 us, and with every load in
// one 16 KB piece 180 us.  Longer batches of loads, stores held back to the
// end of a unit, a pass for each output and an order by slices were all
// slower or no faster, at 200^3 (64 us, all of it in the last-level cache) too.
struct MapRow {
  double d[3];  // displacement of the row's first voxel
  int lin, x0;  // linear index and x of the row's first voxel, both minus start
  int y, z;
  int start;    // exclusive prefix of span lengths
  int pad;
};
__global__ __launch_bounds__(kWG) void k_transform(DevProblem pr, int own, const float* __restrict__ X2, int parts,
                                                   float* dvf, float* warped) {
  __shared__ WaveRows rows[kWaves];
  __shared__ MapRow maps[kWaves][64];
  __shared__ RasterTet rt;
  __shared__ double s_vol;
  __shared__ float xs[2][12];
  const int logical = xcd_logical(blockIdx.x & 7, blockIdx.x >> 3, pr.T * parts);
  if (logical < 0) return;
  const int t = logical / parts, part = logical - t * parts;
  const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
  const int4 tv = pr.tets[t];
  const int vid[4] = {tv.x, tv.y, tv.z, tv.w};
  bool bad = false;
  if (threadIdx.x < 24) {
    const int g = threadIdx.x / 12, e = threadIdx.x % 12, c = e % 3;
    float x = X2[((size_t)(g == 0 ? own : 1 - own) * pr.P + vid[e / 3]) * 3 + c];
    bad = lattice_bits(x, c == 0 ? pr.D[0] : (c == 1 ? pr.D[1] : pr.D[2])) != 0u;
    xs[g][e] = x;
  }
  if (__syncthreads_or(bad)) return;
  if (wave == 0) {
    double vol = 0.0;
    if (lane == 0) s_vol = vol = -setup_face(xs[0], 0, rt);
    if (lane_value(vol, 0) > 0.0) setup_raster(xs[0], xs[1], pr.D, lane, rt);
  }
  __syncthreads();
  const double vol = lane_value(s_vol, 0);
  if (!(vol > 0.0)) return;
  // position = X3 + sum over f < 3 of o_f(voxel) (X_f - X3) / vol, o_f = C[f][0] + C[f][1] i + C[f][2] j + C[f][3] k
  double C[3][4], E[3][3], X3[3], step[3] = {-1.0, 0.0, 0.0};
  const double rvol = 1.0 / vol;
  for (int a = 0; a < 3; ++a) X3[a] = lane_value((double)xs[1][9 + a], 0);
  for (int f = 0; f < 3; ++f) {
    C[f][0] = lane_value(rt.F[f][0] + face_thr(rt.F[f]), 0);
    C[f][1] = lane_value(face_A(rt.F[f]), 0);
    C[f][2] = lane_value(rt.F[f][1], 0);
    C[f][3] = lane_value(rt.F[f][2], 0);
    for (int a = 0; a < 3; ++a) {
      E[f][a] = lane_value((double)(xs[1][3 * f + a] - xs[1][9 + a]) * rvol, 0);
      step[a] = lane_value(step[a] + C[f][1] * E[f][a], 0);
    }
  }
  const __amdgpu_buffer_rsrc_t other = image_rsrc(own ? pr.img[0] : pr.img[1], pr.img_bytes);
  const int sy = 8 * pr.ex;
  const int nb = (rt.nrows + 63) >> 6;
  WaveRows& wr = rows[wave];
  MapRow* map = maps[wave];
  for (int b = part * kWaves + wave; b < nb; b += kWaves * parts) {
    int my_start;
    const int nvox = build_rows<false, 0>(rt, b, lane, pr.D, pr.D[0], pr.DxDy, 0, 0.0f, wr, &my_start);
    if (lane < __popcll(__ballot(my_start >= 0))) {
      MapRow m;
      const float4 rec = wr.row[lane].rec;
      m.start = wr.row[lane].start;
      m.lin = __float_as_int(rec.x);
      m.x0 = __float_as_int(rec.y);
      m.y = __float_as_int(rec.z);
      m.z = __float_as_int(rec.w);
      const double i = m.x0 + m.start, j = m.y, k = m.z;
      double x[3] = {X3[0], X3[1], X3[2]};
      for (int f = 0; f < 3; ++f) {
        const double o = C[f][0] + C[f][1] * i + C[f][2] * j + C[f][3] * k;
        for (int a = 0; a < 3; ++a) x[a] += o * E[f][a];
      }
      m.d[0] = x[0] - i;
      m.d[1] = x[1] - j;
      m.d[2] = x[2] - k;
      map[lane] = m;
    }
    int carry = 0;
    for (int q0 = 0; q0 < nvox; q0 += 64) {
      wr.marker[lane] = 0;
      wave_sync();
      const unsigned pos = (unsigned)(my_start - q0);
      if (pos < 64u) wr.marker[pos] = 1;
      wave_sync();
      const int mk = wr.marker[lane];
      const unsigned long long m = __ballot(mk != 0);
      const int r = row_at(m, mk, carry);
      carry += __popcll(m);
      const int q = q0 + lane;
      if (q >= nvox) break;
      const MapRow row = map[r];
      const int idx = row.lin + q;
      const double n = q - row.start;
      double d[3];
      for (int a = 0; a < 3; ++a) d[a] = row.d[a] + n * step[a];
      if (dvf) reinterpret_cast<float3*>(dvf)[idx] = make_float3((float)d[0], (float)d[1], (float)d[2]);
      if (warped) {
        const int v[3] = {row.x0 + q, row.y, row.z};
        const int at = cell64(pr, v, d);
        const float4v p = load4(other, at, 0), u = load4(other, at, sy);
        warped[idx] = (float)trilinear64(d, p, u);
      }
    }
  }
}

// Bordered z-pair layout from an image [Dz][Dy][Dx]: element (x', y', z')
// = (I[c(z'-1)][c(y'-1)][c(x'-1)], I[c(z')][c(y'-1)][c(x'-1)]); elements of a
// row past x' = Dx + 1 (pitch padding) repeat the last voxel.
__global__ void k_pack_bordered(const float* __restrict__ raw, float* __restrict__ out, int Dx, int Dy, int Dz,
                                BorderedLayout bl) {
  const int64_t n = bl.elements();
  for (int64_t e = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    const int x = (int)(e % bl.px);
    const int64_t r = e / bl.px;
    const int y = (int)(r % bl.py), z = (int)(r / bl.py);
    const int cx = min(max(x - 1, 0), Dx - 1), cy = min(max(y - 1, 0), Dy - 1);
    const int z0 = min(max(z - 1, 0), Dz - 1), z1 = min(z, Dz - 1);
    const size_t row = (size_t)cy * Dx + cx, plane = (size_t)Dx * Dy;
    float2 v;
    v.x = raw[(size_t)z0 * plane + row];
    v.y = raw[(size_t)z1 * plane + row];
    reinterpret_cast<float2*>(out)[e] = v;
  }
}

__global__ void k_fill_i32(int* p, int64_t n, int v) {
  for (int64_t i = blockIdx.x * (int64_t)blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) p[i] = v;
}

}  // namespace

// ------------------------------------------------------------ launchers

size_t eval_lds_bytes(int maxA, int nver) { return eval_layout(maxA, nver).total; }

hipError_t launch_fill_u32(uint32_t* p, int64_t n, uint32_t v, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 4096);
  k_fill_u32<<<blocks, 256, 0, stream>>>(p, n, v);
  return hipGetLastError();
}

hipError_t launch_fold(const DevProblem& pr, int S, const float* X, uint32_t* flags, int32_t* first_bad,
                       hipStream_t stream) {
  hipError_t e = launch_fill_u32(flags, S, 0u, stream);
  if (e != hipSuccess) return e;
  if (first_bad) {
    k_fill_i32<<<(S + 255) / 256, 256, 0, stream>>>(first_bad, S, 0x7fffffff);
    if ((e = hipGetLastError()) != hipSuccess) return e;
  }
  const int64_t np = (int64_t)S * pr.P, nt = (int64_t)S * pr.T;
  k_fold_points<<<(unsigned)((np + 255) / 256), 256, 0, stream>>>(pr, S, X, flags);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_fold_tets<<<(unsigned)((nt + 255) / 256), 256, 0, stream>>>(pr, S, X, flags, first_bad);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  if (first_bad) {
    k_first_bad_fix<<<(S + 255) / 256, 256, 0, stream>>>(S, first_bad);
    e = hipGetLastError();
  }
  return e;
}

// Slot table of a partial launch (G <= kOrderMax): the elements sorted by
// their number of affected tetrahedra, descending (ties by index), are dealt
// to the 8 XCDs in rounds of 8 in alternating direction (0..7, 7..0, ...); the
// order lists XCD 0's elements, then XCD 1's, and so on, so that each XCD's
// contiguous range of the workgroup space holds elements of similar total
// cost.  The table then numbers the chunks of every element in that order:
// slots[0].x = their number, slots[1 + i] = (element, chunk).  A launch has
// room for the largest possible element everywhere (its chunk count is only
// known on the device); by the table the workgroups that exist come first on
// every XCD and the others exit on one scalar load.  Without it every second
// or third workgroup looked up its element to find it had no such chunk: 520
// of 3,600 us on a class of the phantom's tetrahedra, 770 of 6,000 us on the
// uneven half-resolution batch.  One workgroup orders (cost, index) keys in
// LDS: by the number of smaller keys for up to kRankMax elements, where that is
// shorter than the steps of a sort, by a bitonic sort beyond.
constexpr int kRankMax = 256;
__global__ __launch_bounds__(1024) void k_slots(int G, const int* __restrict__ aff_cnt, int pchunk,
                                                int2* __restrict__ slots) {
  __shared__ unsigned long long key[kOrderMax];
  __shared__ int s_order[kOrderMax];
  __shared__ int s_wave[16];
  const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
  auto key_of = [&](int i) {
    return ((unsigned long long)(0xffffffffu - (unsigned)max(aff_cnt[i], 0)) << 32) | (unsigned)i;
  };
  const int nb = G >> 4, rem = G & 15;
  auto deal = [&](int i, int g) {  // element g is i-th by cost
    const int r = i & 15, x = r < 8 ? r : 15 - r;
    int start = 0;  // elements dealt to the XCDs before x
    for (int y = 0; y < x; ++y) start += 2 * nb + (y < rem ? 1 : 0) + (15 - y < rem ? 1 : 0);
    s_order[start + (i >> 4) * 2 + (r >= 8 ? 1 : 0)] = g;
  };
  if (G <= kRankMax) {
    if (t < kRankMax) key[t] = t < G ? key_of(t) : ~0ull;
    __syncthreads();
    if (t < G) {
      const unsigned long long mine = key[t];
      int rank = 0;
#pragma unroll 4
      for (int j = 0; j < G; ++j) rank += key[j] < mine;
      deal(rank, t);
    }
  } else {
    int n = 1;
    while (n < G) n <<= 1;
    for (int i = t; i < n; i += 1024) key[i] = i < G ? key_of(i) : ~0ull;
    __syncthreads();
    for (int k = 2; k <= n; k <<= 1)
      for (int j = k >> 1; j > 0; j >>= 1) {
        for (int i = t; i < n; i += 1024) {
          const int l = i ^ j;
          if (l > i) {
            const unsigned long long u = key[i], v = key[l];
            if ((u > v) == ((i & k) == 0)) {
              key[i] = v;
              key[l] = u;
            }
          }
        }
        __syncthreads();
      }
    for (int i = t; i < G; i += 1024) deal(i, (int)(unsigned)(key[i] & 0xffffffffull));
  }
  __syncthreads();
  int base = 1;
  for (int i0 = 0; i0 < G; i0 += 1024) {  // 1024 elements at a time: prefix of their chunks
    const int i = i0 + t, g = i < G ? s_order[i] : 0;
    const int nc = i < G ? (max(aff_cnt[g], 0) + pchunk - 1) / pchunk : 0;
    const int incl = wave_incl_scan(nc);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    int at = base + incl - nc, all = 0;
    for (int w = 0; w < 16; ++w) {
      at += w < wave ? s_wave[w] : 0;
      all += s_wave[w];
    }
    for (int c = 0; c < nc; ++c) slots[at + c] = make_int2(g, c);
    base += all;
    __syncthreads();
  }
  if (t == 0) slots[0] = make_int2(base - 1, 0);
}

hipError_t launch_slots(int G, const int* aff_cnt, int pchunk, int2* slots, hipStream_t stream) {
  if (G <= 0 || G > kOrderMax) return hipSuccess;
  k_slots<<<1, 1024, 0, stream>>>(G, aff_cnt, pchunk, slots);
  return hipGetLastError();
}

hipError_t launch_affected(const DevProblem& pr, int F, const int* fos_off, const int* fos_pts, int max_pts,
                           int maxA, int* aff, int* aff_cnt, hipStream_t stream) {
  if (F <= 0) return hipSuccess;
  k_affected<<<F, 64, 0, stream>>>(pr, F, fos_off, fos_pts, max_pts, maxA, aff, aff_cnt);
  return hipGetLastError();
}

// Workgroups from which a sweep keeps every SIMD at 8 waves.  2,048 do, but the
// launch has room for the largest element everywhere and two to four times the
// workgroups that exist.  The number of workgroups does not tell everything:
// with few, large tetrahedra (150^3, a 4^3 mesh, chunk 6) 8 waves take 5.93 ms
// and 7 took 5.68.
constexpr int64_t kSweepMany = 4 * 8 * 256;

// Launches a sweep of n workgroups in slices of kGridMax (a multiple of 8, so a
// slice goes on where the last one left the XCDs).  Slices and not a second
// dimension, whose numbers every workgroup would read: 5,832 elements for 8
// solutions, all masked, without a slot table 998 us so and 1,026 with it.
template <class Launch>
void sweep_slices(int64_t n, Launch launch) {
  for (int64_t first = 0; first < n; first += kGridMax) launch((unsigned)std::min(kGridMax, n - first), (int)first);
}

hipError_t launch_eval(const EvalArgs& a, hipEvent_t ev_begin, hipEvent_t ev_end, hipStream_t stream) {
  const int64_t nwg = (int64_t)a.S * a.G;
  if (nwg <= 0) return hipSuccess;
  // XCD x gets the workgroups x, x + 8, ...: as many as xcd_logical gives it, whatever the slot table leaves of them
  const int64_t most = nwg * (a.partial ? a.nchunk : 1);
  const size_t lds = eval_lds_bytes(kMaxChunk, a.nver);
  if (ev_begin) (void)hipEventRecord(ev_begin, stream);
  const bool many = a.nver == 1 && most > kSweepMany;
  auto launch = [&](auto* dense, auto* sparse) {
    sweep_slices(most, [&](unsigned wgs, int first) { (many ? dense : sparse)<<<wgs, kWG, lds, stream>>>(a, first); });
  };
  if (a.partial && a.row_pairs)
    launch(k_sweep<1, 1, 8>, k_sweep<1, 1, 6>);
  else if (a.partial)
    launch(k_sweep<1, 0, 8>, k_sweep<1, 0, 6>);
  else if (a.row_pairs)
    launch(k_sweep<0, 1, 8>, k_sweep<0, 1, 6>);
  else
    launch(k_sweep<0, 0, 8>, k_sweep<0, 0, 6>);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ev_end) (void)hipEventRecord(ev_end, stream);
  if (!a.partial) return hipSuccess;  // the sweep wrote the terms
  k_finish<<<(unsigned)((nwg + kFinishPairs - 1) / kFinishPairs), 64, 0, stream>>>(a, (int)nwg);
  return hipGetLastError();
}

hipError_t launch_eval_batch(const EvalArgs* jobs_dev, const int* wg_off_dev, int n_jobs, int per_xcd, int total_finish,
                             size_t lds, int rows, hipStream_t stream) {
  if (per_xcd <= 0) return hipSuccess;
  auto* kernel = rows == 0 ? k_sweep_batch<0> : (rows == 1 ? k_sweep_batch<1> : k_sweep_batch<2>);
  sweep_slices(8 * (int64_t)per_xcd,
               [&](unsigned wgs, int first) { kernel<<<wgs, kWG, lds, stream>>>(jobs_dev, wg_off_dev, n_jobs, first); });
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_finish_batch<<<(unsigned)total_finish, 64, 0, stream>>>(jobs_dev, wg_off_dev + (n_jobs + 1), n_jobs);
  return hipGetLastError();
}

hipError_t launch_full_reduce(const DevProblem& pr, int S, const double* terms, double* obj, hipStream_t stream) {
  k_full_reduce<<<S, kWG, 0, stream>>>(pr, terms, obj);
  return hipGetLastError();
}

hipError_t launch_pack_bordered(const float* raw, float* out, int Dx, int Dy, int Dz, BorderedLayout bl,
                                hipStream_t stream) {
  const int64_t n = bl.elements();
  const int blocks = (int)std::min<int64_t>((n + 255) / 256, 65536);
  k_pack_bordered<<<blocks, 256, 0, stream>>>(raw, out, Dx, Dy, Dz, bl);
  return hipGetLastError();
}

// Voxels of a tetrahedron (on average) per workgroup of k_transform: setting
// one up takes about as long as 1000 voxels (2048 voxels each: 305 us at
// 512x512x100, 8192: 297 us), and tetrahedra of more fill the device only if
// they are split (27 tetrahedra of 42000 voxels a cube at 200^3).
constexpr int kTransformVoxels = 8192;
// k_transform_clear looks at the grid before it clears where that is the
// shorter: clearing takes 2.5 us per million voxels, the look (every point and
// tetrahedron, by each workgroup) 6 us for 2430 tetrahedra.
constexpr int64_t kCheckVoxels = 1024;

hipError_t launch_transform(const DevProblem& pr, int own, const float* X2, float* dvf, float* warped,
                            hipStream_t stream) {
  if (!dvf && !warped) return hipSuccess;
  const int64_t V = (int64_t)pr.DxDy * pr.D[2];
  const int64_t nd = dvf ? 3 * V : 0, nw = warped ? V : 0;
  const int check = V >= (1 << 20) + kCheckVoxels * (int64_t)pr.T;
  k_transform_clear<<<(unsigned)std::min<int64_t>((nd + nw + 1023) / 1024, check ? 256 : 1024), 1024, 0, stream>>>(
      pr, own, X2, check, (uint32_t*)dvf, nd, (uint32_t*)warped, nw);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int parts = (int)std::max<int64_t>(1, std::min<int64_t>(64, V / pr.T / kTransformVoxels));
  k_transform<<<8u * (((unsigned)pr.T * parts + 7) / 8), kWG, 0, stream>>>(pr, own, X2, parts, dvf, warped);
  return hipGetLastError();
}

hipError_t launch_owner(const DevProblem& pr, const float* Xg, int* owner, int* overlap, hipStream_t stream) {
  const int64_t V = (int64_t)pr.DxDy * pr.D[2];
  k_fill_i32<<<(unsigned)std::min<int64_t>((V + 255) / 256, 4096), 256, 0, stream>>>(owner, V, -1);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  k_fill_i32<<<1, 64, 0, stream>>>(overlap, 1, 0);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  k_owner<<<pr.T, kWG, 0, stream>>>(pr, Xg, owner, overlap);
  return hipGetLastError();
}

}  // namespace dsm
