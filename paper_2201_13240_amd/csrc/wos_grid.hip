// Geometry on the device: inside tests of query points and of the sigma' sample, the sample
// itself, and the construction of the candidate grids of polygons and triangle meshes.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <type_traits>

#include "wos_device.h"
#include "wos_launch.h"

namespace wos {

// ------------------------------------------------------------------ inside tests (FP64)

template <int DIM>
__device__ __forceinline__ bool finite_point(const double* x) {
  bool f = true;
#pragma unroll
  for (int i = 0; i < DIM; ++i) f = f && isfinite(x[i]);
  return f;
}

template <int DIM, int GEOM>
__device__ __forceinline__ bool inside_analytic(G<DevGeometry<double>>& g, const double* x) {
  if (!finite_point<DIM>(x)) return false;
  if (GEOM == GK_BALL) {
    double r2 = 0;
    for (int i = 0; i < DIM; ++i) r2 += (x[i] - g.center[i]) * (x[i] - g.center[i]);
    return r2 < g.radius * g.radius;
  } else if (GEOM == GK_BOX) {
    for (int i = 0; i < DIM; ++i)
      if (!(x[i] > g.lo[i] && x[i] < g.hi[i])) return false;
    return true;
  } else {
    int act;
    return sdf_value<double, DIM>(g, x, &act) < 0.0;
  }
}

// What primitive j adds to the inside test at x: polygons count the crossings of a horizontal
// ray (even-odd), meshes sum signed solid angles (generalized winding number; Van Oosterom
// and Strackee: tan(Omega/2) = det[a b c] / (|a||b||c| + (a.b)|c| + (a.c)|b| + (b.c)|a|)).
template <int GEOM>
__device__ __forceinline__ double inside_term(G<DevGeometry<double>>& g, const double* x, int j) {
  if (GEOM == GK_POLYGON) {
    const WOS_GLOBAL double* s = gptr(g.prims) + (size_t)j * kPrimStride2;
    const double ay = s[1], by = s[3];
    if ((ay > x[1]) != (by > x[1])) {
      const double xi = s[0] + (x[1] - ay) * (s[2] - s[0]) / (by - ay);
      if (x[0] < xi) return 1.0;
    }
    return 0.0;
  }
  const WOS_GLOBAL double* t = gptr(g.prims) + (size_t)j * kPrimStride3;
  double a[3], b[3], c[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    a[i] = t[i] - x[i];
    b[i] = t[3 + i] - x[i];
    c[i] = t[6 + i] - x[i];
  }
  // every rounding is written out: on the surface the sum's last bits decide, and left to the
  // compiler they depend on the kernel around it
  auto dot = [](const double* u, const double* v) {
    return __builtin_fma(u[2], v[2], __builtin_fma(u[0], v[0], u[1] * v[1]));
  };
  auto minor = [&](int i, int j) { return __builtin_fma(b[i], c[j], -(c[i] * b[j])); };
  const double la = sqrt(dot(a, a)), lb = sqrt(dot(b, b)), lc = sqrt(dot(c, c));
  const double det = __builtin_fma(a[2], minor(0, 1), __builtin_fma(a[0], minor(1, 2), -(a[1] * minor(0, 2))));
  const double ab = dot(a, b), ac = dot(a, c), bc = dot(b, c);
  const double den = __builtin_fma(bc, la, __builtin_fma(ac, lb, __builtin_fma(la * lb, lc, ab * lc)));
  return 2.0 * atan2(det, den);
}

template <int GEOM>
__device__ __forceinline__ bool inside_sum(double w) {
  return GEOM == GK_POLYGON ? ((int64_t)w & 1) != 0 : fabs(w) > 2.0 * M_PI;
}

// Inside test of one finite point by a whole wave, over every primitive. On the surface of a mesh
// the angles add up to 2 pi, the threshold, and rounding decides: sums that close to it (n
// roundings of angles below 2 pi) are taken again in the primitives' order, so that the answer
// does not depend on how the lanes share them.
template <int GEOM>
__device__ __forceinline__ bool inside_wave(G<DevGeometry<double>>& g, const double* x) {
  const int lane = (int)__lane_id();
  double w = 0;
  for (int j = lane; j < g.n_prims; j += 64) w += inside_term<GEOM>(g, x, j);
  for (int off = 32; off > 0; off >>= 1) w += __shfl_xor(w, off);
  if (GEOM == GK_TRIMESH && fabs(fabs(w) - 2.0 * M_PI) <= 1e-13 * (double)(g.n_prims + 64)) {
    w = 0;
    for (int j0 = 0; j0 < g.n_prims; j0 += 64) {
      const int n = min(64, g.n_prims - j0);
      const double t = lane < n ? inside_term<GEOM>(g, x, j0 + lane) : 0.0;
      for (int k = 0; k < n; ++k) w += __shfl(t, k);
    }
  }
  return inside_sum<GEOM>(w);
}

// Class of a point from its grid cell: 0 outside, 1 inside, kCellMixed undecided. Points
// outside the grid lie outside the domain; a mesh that is not closed has no classes.
template <int DIM>
__device__ __forceinline__ int cell_class_of(G<DevGeometry<double>>& g, const double* x) {
  if (!finite_point<DIM>(x)) return 0;
  if (!g.cell_class) return kCellMixed;
  const int nn[3] = {g.grid_nx, g.grid_ny, g.grid_nz};
  int64_t c = 0;
  bool in = true;
#pragma unroll
  for (int i = DIM - 1; i >= 0; --i) {
    const double f = (x[i] - g.grid_lo[i]) * g.grid_inv_h;
    in = in && f >= 0.0 && f < (double)nn[i];
    c = c * nn[i] + (in ? (int64_t)f : 0);
  }
  return in ? (int)gptr(g.cell_class)[c] : 0;
}

// Points to classify: an array, or the cell centres of a sampling grid.
template <int DIM>
struct ArrayPoints {
  const double* pts;
  __device__ __forceinline__ void get(int64_t k, double* x) const {
    for (int i = 0; i < DIM; ++i) x[i] = pts[k * DIM + i];
  }
};

template <int DIM>
struct SamplePoints {
  double lo[3], h[3];
  int grid;
  int64_t first;   // sample of k = 0
  __device__ __forceinline__ void get(int64_t k, double* x) const {
    k += first;
#pragma unroll
    for (int i = 0; i < DIM; ++i) {
      x[i] = __builtin_fma(h[i], (double)(k % grid) + 0.5, lo[i]);
      k /= grid;
    }
  }
};

// Analytic and SDF domains: one point per thread.
template <int DIM, int GEOM, typename SRC>
__global__ void classify_analytic_kernel(const DevProblem<double>* P, SRC src, int64_t n, int8_t* inside) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  double x[DIM];
  src.get(i, x);
  inside[i] = inside_analytic<DIM, GEOM>(gptr(P)->geom, x) ? 1 : 0;
}

// Polygons and meshes: 64 points per block of 256 threads. The first wave looks up their cells;
// the points that lie in a cell of the boundary (2-10% of a slice) go through every
// primitive, a wave each. One point per thread over every primitive, as before, is a serial
// chain of n_prims terms: 15.7 ms for 131,000 points of a 20,480-triangle mesh, 156 us on
// average for the polygons of a batch.
constexpr int kClassifyPoints = 64;

// Classifies the block's points first .. first + 63 (those below n); returns for threads
// below 64 whether theirs is inside. Called by the whole block.
template <int DIM, int GEOM, typename SRC>
__device__ __forceinline__ bool classify_block(G<DevGeometry<double>>& g, const SRC& src, int64_t first, int64_t n) {
  __shared__ double s_x[kClassifyPoints][DIM];
  __shared__ int s_todo[kClassifyPoints];
  __shared__ int s_n;
  __shared__ int s_in[kClassifyPoints];
  const int t = (int)threadIdx.x, wave = t >> 6;
  if (wave == 0) {
    int c = 0;
    if (first + t < n) {
      double x[DIM];
      src.get(first + t, x);
      c = cell_class_of<DIM>(g, x);
#pragma unroll
      for (int k = 0; k < DIM; ++k) s_x[t][k] = x[k];
    }
    s_in[t] = c == 1;
    const uint64_t todo = __ballot(c == kCellMixed);
    if (c == kCellMixed) s_todo[__popcll(todo & ((1ull << t) - 1ull))] = t;
    if (t == 0) s_n = __popcll(todo);
  }
  __syncthreads();
  for (int k = wave; k < s_n; k += (int)(blockDim.x >> 6)) {
    const int p = s_todo[k];
    double x[DIM];
#pragma unroll
    for (int c = 0; c < DIM; ++c) x[c] = s_x[p][c];
    const bool in = inside_wave<GEOM>(g, x);
    if (__lane_id() == 0) s_in[p] = in;
  }
  __syncthreads();
  return wave == 0 && s_in[t] != 0;
}

template <int DIM, int GEOM, typename SRC>
__global__ void __launch_bounds__(256) classify_cells_kernel(const DevProblem<double>* P, SRC src, int64_t n,
                                                             int8_t* inside) {
  const int64_t first = (int64_t)blockIdx.x * kClassifyPoints;
  const bool in = classify_block<DIM, GEOM>(gptr(P)->geom, src, first, n);
  if (threadIdx.x < kClassifyPoints && first + threadIdx.x < n) inside[first + threadIdx.x] = in ? 1 : 0;
}

// ------------------------------------------------------------------ preparing a job
//
// One launch per kPrepItems items classifies their points, evaluates gamma(x0) (the same for
// all walks of a point, so each walk starts from it), and leaves everything else the walker
// finds in memory: the item table, which comes with the launch's arguments and needs no copy
// or wait, the launch parameters, cleared slots and tile counters. As five launches, a copy
// and a wait for it, this was 60 of the 350 us of a solve of 16 points x 128 walks.
template <typename T, int DIM, int GEOM>
__global__ void __launch_bounds__(256) prep_kernel(PrepArgs a) {
  constexpr bool kCells = GEOM == GK_POLYGON || GEOM == GK_TRIMESH;
  constexpr int kPoints = kCells ? kClassifyPoints : 256;
  const int t = (int)threadIdx.x;
  if (blockIdx.x == 0) {
    constexpr int kWords = (int)(sizeof(DevItem) / sizeof(uint32_t));
    if (a.table)
      for (int w = t; w < a.n * kWords; w += 256) ((uint32_t*)a.table)[w] = ((const uint32_t*)a.item)[w];
    if (a.counters && t < (int)(kTileQueues * kTileQueueStride)) a.counters[t] = 0;
    if (a.lp && t == 0) {
      a.lp->seed = a.seed;
      a.lp->walk_offset_add = 0;
    }
  }
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + t; i < a.slot_words; i += (uint64_t)gridDim.x * 256) a.slots[i] = 0;
  int k = 0;
  while (k + 1 < a.n && blockIdx.x >= a.block0[k + 1]) ++k;
  const DevItem& it = a.item[k];
  const int64_t first = (int64_t)(blockIdx.x - a.block0[k]) * kPoints, i = first + t;
  const DevProblem<double>* P64 = (const DevProblem<double>*)a.problem64[k];
  bool in = false;
  if constexpr (kCells) {
    in = classify_block<DIM, GEOM>(gptr(P64)->geom, ArrayPoints<DIM>{it.points}, first, it.n_points);
  } else if (i < it.n_points) {
    double x[DIM];
    ArrayPoints<DIM>{it.points}.get(i, x);
    in = inside_analytic<DIM, GEOM>(gptr(P64)->geom, x);
  }
  const bool mine = t < kPoints && i < it.n_points;
  if (mine) {
    ((int8_t*)it.inside)[i] = in ? 1 : 0;
    T g = 0;
    if (in) {
      T x[DIM];
#pragma unroll
      for (int c = 0; c < DIM; ++c) x[c] = (T)it.points[i * DIM + c];
      g = point_gamma<T, DIM>(*gptr((const DevProblem<T>*)it.problem), x);
    }
    ((T*)it.gamma0)[i] = g;
  }
  if (it.counters) {
    const uint64_t m = __ballot(mine && !in);
    if (__lane_id() == 0 && m) atomicAdd((unsigned long long*)&it.counters[0], (unsigned long long)__popcll(m));
  }
}

// ------------------------------------------------------------------ sigma' sampling (FP64)
// out per block: [min sigma', max sigma', min alpha, min sigma, #non-finite, #samples]

template <int DIM>
__global__ void sigma_sample_kernel(const DevProblem<double>* P, SamplePoints<DIM> src, int64_t n, const int8_t* inside,
                                    double* out) {
  double mn = __builtin_huge_val(), mx = -__builtin_huge_val(), amin = __builtin_huge_val(),
         smin = __builtin_huge_val(), bad = 0, cnt = 0;
  for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n; k += (int64_t)gridDim.x * blockDim.x) {
    if (!inside[k]) continue;
    double x[DIM];
    src.get(k, x);
    G<DevProblem<double>>& PR = *gptr(P);
    const PointCoef<double> c = point_coef<double, DIM, false>(PR, x);
    const double sig = field_eval<double, DIM, false>(PR.sigma, x).v;
    cnt += 1;
    if (!isfinite(c.sigma_prime) || !isfinite(c.alpha)) {
      bad += 1;
      continue;
    }
    mn = fmin(mn, c.sigma_prime);
    mx = fmax(mx, c.sigma_prime);
    amin = fmin(amin, c.alpha);
    smin = fmin(smin, sig);
  }
  __shared__ double red[6][256];
  const int t = threadIdx.x;
  red[0][t] = mn; red[1][t] = mx; red[2][t] = amin; red[3][t] = smin; red[4][t] = bad; red[5][t] = cnt;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if (t < s) {
      red[0][t] = fmin(red[0][t], red[0][t + s]);
      red[1][t] = fmax(red[1][t], red[1][t + s]);
      red[2][t] = fmin(red[2][t], red[2][t + s]);
      red[3][t] = fmin(red[3][t], red[3][t + s]);
      red[4][t] += red[4][t + s];
      red[5][t] += red[5][t + s];
    }
    __syncthreads();
  }
  if (t == 0)
    for (int k = 0; k < 6; ++k) out[blockIdx.x * 6 + k] = red[k][0];
}

// ------------------------------------------------------------------ cell classes
//
// A cell that no primitive touches lies wholly inside or wholly outside a closed boundary,
// and so do two such cells that share a face. Cells are joined into components (union-find
// over faces, labels only ever shrink), the lowest cell of each component is tested against
// every primitive, and the others take its class.

__device__ __forceinline__ uint32_t load_label(const uint32_t* label, uint32_t c) {
  return __hip_atomic_load(label + c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint32_t find_root(const uint32_t* label, uint32_t c) {
  for (;;) {
    const uint32_t up = load_label(label, c);
    if (up == c) return c;
    c = up;   // up < c
  }
}

// Each turn either ends or replaces a by a smaller label, so the loop ends.
__device__ __forceinline__ void join(uint32_t* label, uint32_t a, uint32_t b) {
  for (;;) {
    a = find_root(label, a);
    b = find_root(label, b);
    if (a == b) return;
    if (a < b) {
      const uint32_t t = a;
      a = b;
      b = t;
    }
    const uint32_t old = atomicMin(label + a, b);
    if (old == a) return;
    a = old;
  }
}

// A cell's first label: the start of its run of untouched cells in x, as far as its wave
// reaches, so that a row is not one chain of labels (one cell per link: 3.2 ms of joins for
// 655,000 cells).
__global__ void __launch_bounds__(256) label_init_kernel(const double* best, double reach, int64_t ncell, int nx,
                                                         uint32_t* label, uint32_t* n_roots) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c == 0) *n_roots = 0;
  const int lane = (int)__lane_id();
  const bool open = c < ncell && sqrt(best[c]) > reach;
  const uint64_t all = __ballot(open);
  const bool left = lane > 0 && (all >> (lane - 1) & 1ull) && c % nx != 0;
  const uint64_t starts = __ballot(open && !left) & (~0ull >> (63 - lane));
  if (c < ncell) label[c] = open ? (uint32_t)(c - (lane - (63 - __clzll(starts)))) : kNoLabel;
}

// Joins across the ends of those runs and to the next row and layer; of two rows' common
// stretch only the first pair is joined, the runs hold the others together.
__global__ void __launch_bounds__(256) label_join_kernel(uint32_t* label, int nx, int ny, int nz) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  auto open = [&](int64_t u) { return load_label(label, (uint32_t)u) != kNoLabel; };
  if (c >= (int64_t)nx * ny * nz || !open(c)) return;
  const int64_t layer = (int64_t)nx * ny;
  const int i = (int)(c % nx), j = (int)(c / nx % ny), k = (int)(c / layer);
  const bool left = i > 0 && open(c - 1);
  if (left && (c & 63) == 0) join(label, (uint32_t)c, (uint32_t)(c - 1));
  if (j + 1 < ny && open(c + nx) && !(left && open(c + nx - 1))) join(label, (uint32_t)c, (uint32_t)(c + nx));
  if (k + 1 < nz && open(c + layer) && !(left && open(c + layer - 1)))
    join(label, (uint32_t)c, (uint32_t)(c + layer));
}

__global__ void label_roots_kernel(const uint32_t* label, int64_t ncell, uint32_t* roots, uint32_t* n_roots) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c < ncell && label[c] == (uint32_t)c) roots[atomicAdd(n_roots, 1u)] = (uint32_t)c;
}

template <int GEOM>
__global__ void __launch_bounds__(256) root_class_kernel(const DevProblem<double>* P, GridShape s, const uint32_t* roots,
                                                         const uint32_t* n_roots, uint8_t* cls) {
  __shared__ double s_w[4];
  G<DevGeometry<double>>& g = gptr(P)->geom;
  const uint32_t n = *n_roots;
  for (uint32_t r = blockIdx.x; r < n; r += gridDim.x) {
    const uint32_t c = roots[r];
    const double x[3] = {s.lo[0] + ((double)(c % (uint32_t)s.nx) + 0.5) * s.h,
                         s.lo[1] + ((double)(c / (uint32_t)s.nx % (uint32_t)s.ny) + 0.5) * s.h,
                         s.lo[2] + ((double)(c / ((uint32_t)s.nx * (uint32_t)s.ny)) + 0.5) * s.h};
    double w = 0;
    for (int j = (int)threadIdx.x; j < g.n_prims; j += (int)blockDim.x) w += inside_term<GEOM>(g, x, j);
    for (int off = 32; off > 0; off >>= 1) w += __shfl_xor(w, off);
    if (__lane_id() == 0) s_w[threadIdx.x >> 6] = w;
    __syncthreads();
    if (threadIdx.x == 0) cls[c] = inside_sum<GEOM>(s_w[0] + s_w[1] + s_w[2] + s_w[3]) ? 1 : 0;
    __syncthreads();
  }
}

__global__ void cell_class_kernel(const uint32_t* label, int64_t ncell, uint8_t* cls) {
  const int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (c >= ncell) return;
  const uint32_t l = label[c];
  if (l == kNoLabel) {
    cls[c] = kCellMixed;
  } else if (l != (uint32_t)c) {
    cls[c] = cls[find_root(label, l)];   // roots are written already
  }
}

// ------------------------------------------------------------------ candidate grids
//
// The construction of build_segment_grid and build_triangle_grid (bvh.h), one cell per
// thread, in their arithmetic: contraction is off from here on, so that distances, and with
// them the lists, come out as the host's. The host builds took 170 ms for 5120 triangles and
// 440 ms for 20,480 (16 threads), more than the solves that followed.
#pragma clang fp contract(off)

__device__ __forceinline__ double build_seg_dist2(const WOS_GLOBAL double* s, const double* p) {
  const double ex = s[2] - s[0], ey = s[3] - s[1];
  const double qx = p[0] - s[0], qy = p[1] - s[1];
  const double l2 = ex * ex + ey * ey;
  double t = l2 > 0 ? (qx * ex + qy * ey) / l2 : 0.0;
  t = fmin(1.0, fmax(0.0, t));
  const double dx = qx - t * ex, dy = qy - t * ey;
  return dx * dx + dy * dy;
}

__device__ __forceinline__ double build_dot3(const double* a, const double* b) {
  return a[0] * b[0] + a[1] * b[1] + a[2] * b[2];
}

__device__ __forceinline__ double build_edge_dist2(const double* a, const double* b, const double* p) {
  double e[3], q[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    e[k] = b[k] - a[k];
    q[k] = p[k] - a[k];
  }
  const double l2 = build_dot3(e, e);
  double t = l2 > 0 ? build_dot3(q, e) / l2 : 0.0;
  t = fmin(1.0, fmax(0.0, t));
#pragma unroll
  for (int k = 0; k < 3; ++k) q[k] -= t * e[k];
  return build_dot3(q, q);
}

__device__ __forceinline__ double build_tri_dist2(const WOS_GLOBAL double* t, const double* p) {
  double a[3], b[3], c[3], e0[3], e1[3], ap[3];
#pragma unroll
  for (int k = 0; k < 3; ++k) {
    a[k] = t[k];
    b[k] = t[3 + k];
    c[k] = t[6 + k];
    e0[k] = b[k] - a[k];
    e1[k] = c[k] - a[k];
    ap[k] = p[k] - a[k];
  }
  const double d00 = build_dot3(e0, e0), d01 = build_dot3(e0, e1), d11 = build_dot3(e1, e1);
  const double den = d00 * d11 - d01 * d01;
  if (den > 0) {
    const double d20 = build_dot3(ap, e0), d21 = build_dot3(ap, e1);
    const double v = (d11 * d20 - d01 * d21) / den, w = (d00 * d21 - d01 * d20) / den;
    if (v >= 0 && w >= 0 && v + w <= 1) {
      double q[3];
#pragma unroll
      for (int k = 0; k < 3; ++k) q[k] = ap[k] - v * e0[k] - w * e1[k];
      return build_dot3(q, q);
    }
  }
  return fmin(build_edge_dist2(a, b, p), fmin(build_edge_dist2(b, c, p), build_edge_dist2(c, a, p)));
}

template <int DIM>
__device__ __forceinline__ double build_box_dist2(const WOS_GLOBAL double* lo, const WOS_GLOBAL double* hi,
                                                  const double* p) {
  double s = 0;
#pragma unroll
  for (int k = 0; k < DIM; ++k) {
    const double e = fmax(fmax(lo[k] - p[k], p[k] - hi[k]), 0.0);
    s += e * e;
  }
  return s;
}

// Blocks of one wave. Far children wait on a stack in LDS (a column per lane) in trees of
// depth kBuildStack or less, else in private memory.
constexpr int kBuildStack = 20;
constexpr int kBuildStackDeep = 48;   // any tree the host accepts

// Visits every leaf primitive whose subtree box lies within sqrt(bound) of p, nearer boxes
// first; f(primitive, squared distance) may lower the bound.
template <int DIM, bool DEEP, typename F>
__device__ __forceinline__ void build_traverse(G<DevGeometry<double>>& g, const double* p, const double& bound,
                                               int32_t* s_node, double* s_dist, F&& f) {
  const WOS_GLOBAL BvhNode<double, DIM>* nodes = (const WOS_GLOBAL BvhNode<double, DIM>*)g.nodes;
  const WOS_GLOBAL double* prims = gptr(g.prims);
  int32_t d_node[DEEP ? kBuildStackDeep : 1];
  double d_dist[DEEP ? kBuildStackDeep : 1];
  int sp = 0;
  int32_t cur = g.root;
  for (;;) {
    if (cur < 0) {
      const int32_t code = -1 - cur, first = code >> 3, cnt = code & 7;
      for (int32_t i = first; i < first + cnt; ++i)
        f(i, DIM == 2 ? build_seg_dist2(prims + (size_t)i * kPrimStride2, p)
                      : build_tri_dist2(prims + (size_t)i * kPrimStride3, p));
    } else {
      G<BvhNode<double, DIM>>& n = nodes[cur];
      const double da = build_box_dist2<DIM>(n.lo[0], n.hi[0], p), db = build_box_dist2<DIM>(n.lo[1], n.hi[1], p);
      const int32_t ca = n.child[0], cb = n.child[1];
      const bool a_first = da <= db;
      const double near_d = a_first ? da : db, far_d = a_first ? db : da;
      if (far_d <= bound) {   // at most one entry per level above the current node
        if constexpr (DEEP) {
          d_node[sp] = a_first ? cb : ca;
          d_dist[sp] = far_d;
        } else {
          s_node[sp * 64] = a_first ? cb : ca;
          s_dist[sp * 64] = far_d;
        }
        ++sp;
      }
      if (near_d <= bound) {
        cur = a_first ? ca : cb;
        continue;
      }
    }
    double d;
    do {
      if (sp == 0) return;
      --sp;
      cur = DEEP ? d_node[DEEP ? sp : 0] : s_node[sp * 64];
      d = DEEP ? d_dist[DEEP ? sp : 0] : s_dist[sp * 64];
    } while (!(d <= bound));
  }
}

// Cell of this thread and its centre, or -1: a wave takes a block of 8 x 8 (3D: 4 x 4 x 4)
// cells, whose searches visit nearly the same nodes (64 cells of a row reach across the
// domain).
template <int DIM>
struct CellBlocks {
  static constexpr int kSide = DIM == 2 ? 8 : 4;
  static int64_t blocks(const GridShape& s) {
    const auto n = [](int64_t v) { return (v + kSide - 1) / kSide; };
    return n(s.nx) * n(s.ny) * (DIM == 2 ? 1 : n(s.nz));
  }
};

template <int DIM>
__device__ __forceinline__ int64_t block_cell(const GridShape& s, double* p) {
  constexpr int S = CellBlocks<DIM>::kSide;
  const int bx = (s.nx + S - 1) / S, by = (s.ny + S - 1) / S, b = (int)blockIdx.x, t = (int)threadIdx.x;
  const int i = b % bx * S + t % S, j = b / bx % by * S + t / S % S, k = DIM == 2 ? 0 : b / (bx * by) * S + t / (S * S);
  p[0] = s.lo[0] + ((double)i + 0.5) * s.h;
  p[1] = s.lo[1] + ((double)j + 0.5) * s.h;
  p[2] = s.lo[2] + ((double)k + 0.5) * s.h;
  return i < s.nx && j < s.ny && k < s.nz ? ((int64_t)k * s.ny + j) * s.nx + i : -1;
}

// The traversal stacks of a block and the list being collected, a column per lane.
template <bool DEEP, int KEEP>
struct BuildScratch {
  int32_t node[DEEP ? 1 : kBuildStack * 64];
  double dist[DEEP ? 1 : kBuildStack * 64];
  double d2[KEEP ? KEEP * 64 : 1];
  int32_t id[KEEP ? KEEP * 64 : 1];
};

// Squared distance of p and the nearest primitive.
template <int DIM, bool DEEP, typename S>
__device__ __forceinline__ double build_nearest(G<DevGeometry<double>>& g, const double* p, S& sc, int32_t* nearest) {
  const int t = DEEP ? 0 : (int)threadIdx.x;
  double best = 1e300;
  *nearest = 0;
  build_traverse<DIM, DEEP>(g, p, best, sc.node + t, sc.dist + t, [&](int32_t i, double d2) {
    if (d2 < best) {
      best = d2;
      *nearest = i;
    }
  });
  return best;
}

// Collects the primitives within r2 of p in the lane's column, in order of (distance, index):
// the max_list + 1 nearest, or, for a polygon with more, the deep_list + 1 nearest. Returns
// how many belong to the cell's list; *tail receives the distance of the next one, +inf where
// the list is complete.
template <int DIM, bool DEEP, typename S>
__device__ __forceinline__ int build_list(G<DevGeometry<double>>& g, const double* p, double r2, const GridRule& rule,
                                          S& sc, double* tail) {
  const int t = DEEP ? 0 : (int)threadIdx.x;
  double* ld = sc.d2 + threadIdx.x;
  int32_t* li = sc.id + threadIdx.x;
  double bound = r2;
  int n = 0, cap = rule.max_list + 1;
  bool over = false;
  build_traverse<DIM, DEEP>(g, p, bound, sc.node + t, sc.dist + t, [&](int32_t i, double d2) {
    if (!(d2 <= bound)) return;
    if (n == cap) {
      const double ed = ld[(n - 1) * 64];
      if (d2 > ed || (d2 == ed && i > li[(n - 1) * 64])) return;
      --n;
    }
    int k = n++;
    for (; k > 0; --k) {
      const double ed = ld[(k - 1) * 64];
      const int32_t ei = li[(k - 1) * 64];
      if (ed < d2 || (ed == d2 && ei < i)) break;
      ld[k * 64] = ed;
      li[k * 64] = ei;
    }
    ld[k * 64] = d2;
    li[k * 64] = i;
    if (n == cap) {
      if (DIM == 2 && !over) {
        over = true;
        cap = n = rule.deep_list + 1;
      }
      bound = ld[(n - 1) * 64];
    }
  });
  const int keep = DIM == 2 && over ? rule.deep_list : min(n, rule.max_list);
  *tail = n > keep ? sqrt(ld[keep * 64]) : __builtin_huge_val();
  return keep;
}

// Polygons: squared distance of each cell's centre, the length of its list, and how many lists
// are truncated.
template <bool DEEP>
__global__ void __launch_bounds__(64) segment_count_kernel(const DevProblem<double>* P, GridShape s, GridRule rule,
                                                           double* best_out, uint32_t* count, uint32_t* truncated) {
  __shared__ BuildScratch<DEEP, 0> sc;
  double p[3];
  const int64_t c = block_cell<2>(s, p);
  if (c < 0) return;
  G<DevGeometry<double>>& g = gptr(P)->geom;
  int32_t nearest;
  const double best = build_nearest<2, DEEP>(g, p, sc, &nearest);
  best_out[c] = best;
  const double r = sqrt(best) + 2 * rule.halfdiag + rule.margin, r2 = r * r;
  const uint32_t most = (uint32_t)rule.max_list + 1u;
  uint32_t n = 0;
  double bound = r2;
  const int t = DEEP ? 0 : (int)threadIdx.x;
  build_traverse<2, DEEP>(g, p, bound, sc.node + t, sc.dist + t, [&](int32_t, double d2) {
    if (d2 <= r2 && ++n >= most) bound = -1.0;   // enough is known
  });
  count[c] = n >= most ? (uint32_t)rule.deep_list : n;
  const uint64_t cut = __ballot(n >= most);
  if (cut && (int)__lane_id() == __ffsll((unsigned long long)cut) - 1) atomicAdd(truncated, (uint32_t)__popcll(cut));
}

// Polygons: every cell's list from its start, and its record in both precisions; distances
// are less the rounding margin.
template <bool DEEP>
__global__ void __launch_bounds__(64) segment_fill_kernel(const DevProblem<double>* P, GridShape s, GridRule rule,
                                                          const double* best_in, const uint32_t* start, GridOut o) {
  __shared__ BuildScratch<DEEP, kPolygonCellMax + 1> sc;
  double p[3];
  const int64_t c = block_cell<2>(s, p);
  if (c < 0) return;
  G<DevGeometry<double>>& g = gptr(P)->geom;
  const double r = sqrt(best_in[c]) + 2 * rule.halfdiag + rule.margin;
  double tail;
  const int keep = build_list<2, DEEP>(g, p, r * r, rule, sc, &tail);
  if (tail < __builtin_huge_val()) tail -= rule.margin;
  const double* ld = sc.d2 + threadIdx.x;
  const int32_t* li = sc.id + threadIdx.x;
  const uint32_t st = start[c];
  const WOS_GLOBAL double* prims = gptr(g.prims);
  for (int k = 0; k < keep; ++k) {
    const int32_t id = li[k * 64];
    const double dc = sqrt(ld[k * 64]) - rule.margin;
    o.prim[st + k] = id;
    float* l32 = o.list32 + (size_t)(st + k) * kListEntry;
    double* l64 = o.list64 + (size_t)(st + k) * kListEntry;
    l32[4] = (float)dc;
    l64[4] = dc;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const double v = prims[(size_t)id * kPrimStride2 + e];
      l32[e] = (float)v;
      l64[e] = v;
    }
  }
  if (tail < __builtin_huge_val()) {
    // the band of the list: its extent along the nearest segment and across it
    const WOS_GLOBAL double* q = prims + (size_t)li[0] * kPrimStride2;
    double ux = q[2] - q[0], uy = q[3] - q[1];
    const double l = sqrt(ux * ux + uy * uy);
    ux = l > 0 ? ux / l : 1.0;
    uy = l > 0 ? uy / l : 0.0;
    double t0 = 1e300, t1 = -1e300, w0 = 1e300, w1 = -1e300;
    for (int k = 0; k < keep; ++k)
      for (int v = 0; v < 4; v += 2) {
        const WOS_GLOBAL double* e = prims + (size_t)li[k * 64] * kPrimStride2 + v;
        const double t = (e[0] - q[0]) * ux + (e[1] - q[1]) * uy, w = (e[1] - q[1]) * ux - (e[0] - q[0]) * uy;
        t0 = fmin(t0, t);
        t1 = fmax(t1, t);
        w0 = fmin(w0, w);
        w1 = fmax(w1, w);
      }
    const double wm = 0.5 * (w0 + w1);
    const double a[4] = {q[0] + t0 * ux - wm * uy, q[1] + t0 * uy + wm * ux, (t1 - t0) * ux, (t1 - t0) * uy};
    auto band = [&](auto* b) {
      using T = typename std::remove_reference<decltype(b->radius)>::type;
      for (int e = 0; e < 4; ++e) b->axis[e] = (T)a[e];
      b->inv_len2 = t1 > t0 ? (T)(1.0 / ((t1 - t0) * (t1 - t0))) : (T)0;
      b->radius = (T)(0.5 * (w1 - w0) + 2 * rule.margin);   // the margin covers FP32 rounding here too
    };
    band((ListBand<float>*)(o.list32 + (size_t)st * kListEntry));
    band((ListBand<double>*)(o.list64 + (size_t)st * kListEntry));
  }
  auto record = [&](auto* rec) {
    using T = typename std::remove_reference<decltype(rec->tail)>::type;
    rec->count = (uint32_t)keep;
    rec->start = st;
    rec->tail = (T)tail;
    // inline entries beyond the list repeat its last candidate: their distance equals
    // that candidate's, so they never replace it as the nearest (strict comparison)
    for (int k = 0; k < kCellInline; ++k) {
      T sg[4] = {0, 0, 0, 0}, inv = 0;
      if (keep > 0) {
        const WOS_GLOBAL double* q = prims + (size_t)li[min(k, keep - 1) * 64] * kPrimStride2;
        sg[0] = (T)q[0];
        sg[1] = (T)q[1];
        sg[2] = (T)(q[2] - q[0]);
        sg[3] = (T)(q[3] - q[1]);
        const double ex = (double)sg[2], ey = (double)sg[3], l2 = ex * ex + ey * ey;
        inv = l2 > 0 ? (T)(1.0 / l2) : (T)0;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) rec->seg[k][e] = sg[e];
      rec->inv_len2[k] = inv;
    }
    rec->next_dc = keep > kCellInline ? (T)(sqrt(ld[kCellInline * 64]) - rule.margin) : (T)0;
  };
  record((CellRec<float>*)o.cells32 + c);
  record((CellRec<double>*)o.cells64 + c);
}

// Meshes: squared distance of each cell's centre, its record in both precisions, and the sum
// of the list lengths. The search deep inside, where many triangles are nearly equidistant,
// is most of the time; a list there would not decide anything, so the cell keeps the nearest
// triangle alone, with its distance as the tail (no triangle is nearer to the centre).
template <bool DEEP>
__global__ void __launch_bounds__(64) mesh_cells_kernel(const DevProblem<double>* P, GridShape s, GridRule rule,
                                                        double* best_out, GridOut o, uint32_t* total) {
  __shared__ BuildScratch<DEEP, kMeshCellList + 1> sc;
  double p[3];
  const int64_t c = block_cell<3>(s, p);
  int keep = 0;
  if (c >= 0) {
    G<DevGeometry<double>>& g = gptr(P)->geom;
    double* ld = sc.d2 + threadIdx.x;
    int32_t* li = sc.id + threadIdx.x;
    int32_t nearest;
    const double best = build_nearest<3, DEEP>(g, p, sc, &nearest), d = sqrt(best);
    best_out[c] = best;
    double tail = d;
    keep = 1;
    if (d >= rule.deep) {
      ld[0] = best;
      li[0] = nearest;
    } else {
      const double r = d + 2 * rule.halfdiag + rule.margin;
      keep = build_list<3, DEEP>(g, p, r * r, rule, sc, &tail);
    }
    if (tail < __builtin_huge_val()) tail -= rule.margin;
    auto record = [&](auto* rec) {
      using T = typename std::remove_reference<decltype(rec->tail)>::type;
      rec->count = (uint32_t)keep;
      rec->tail = (T)tail;
      for (int k = 0; k < kMeshCellList; ++k) {   // short lists repeat their last entry
        const int e = min(k, keep - 1) * 64;
        rec->id[k] = li[e];
        rec->dc[k] = (T)(sqrt(ld[e]) - rule.margin);
      }
    };
    record((MeshCell<float>*)o.cells32 + c);
    record((MeshCell<double>*)o.cells64 + c);
  }
  for (int off = 32; off > 0; off >>= 1) keep += __shfl_xor(keep, off);
  if (threadIdx.x == 0) atomicAdd(total, (uint32_t)keep);
}

// ------------------------------------------------------------------ SDF cells
//
// Rows that can decide the combined field somewhere in a cell. Every primitive field, and
// with it every minimum and maximum of them, changes by at most the half diagonal hd between
// the cell's centre and any of its points. A run of unions (or of intersections and
// subtractions) leaves the minimum (maximum) of its rows and of the field before it, so a
// row, or everything before the run, that stays 2 hd and a rounding margin away from that
// value at the centre never is the value itself. The row that is read first sets the field.
template <int DIM>
__global__ void __launch_bounds__(64) sdf_cells_kernel(const DevProblem<double>* P, GridShape s, double scale,
                                                       uint64_t* cells) {
  double p[3];
  const int64_t c = block_cell<DIM>(s, p);
  if (c < 0) return;
  G<DevGeometry<double>>& g = gptr(P)->geom;
  const WOS_GLOBAL double* rows = gptr(g.prims);
  const double hd = 0.5 * s.h * sqrt((double)DIM);
  auto field = [&](int k) {
    const WOS_GLOBAL double* r = rows + (size_t)k * kSdfStride;
    const double f = sdf_shape<double, DIM, false>(r, p, nullptr);
    return (int)r[0] == 2 ? -f : f;
  };
  // FP32 rounding of the point, the cell index and the two fields that are compared
  auto margin = [&](int k) {
    const WOS_GLOBAL double* r = rows + (size_t)k * kSdfStride;
    double m = scale;
    for (int e = 2; e < kSdfStride; ++e) m += fabs(r[e]);
    return 1e-5 * m;
  };
  double f = __builtin_huge_val(), reach = 0;   // reach: largest margin of the rows behind f
  uint64_t list = 0;
  int n = 0;
  for (int i0 = 0; i0 < g.n_prims;) {
    const bool uni = (int)rows[(size_t)i0 * kSdfStride] == 0;
    const double sg = uni ? 1.0 : -1.0;   // sg * value is minimised over the run
    int i1 = i0;
    double best = sg * f;
    for (; i1 < g.n_prims && ((int)rows[(size_t)i1 * kSdfStride] == 0) == uni; ++i1) {
      best = fmin(best, sg * field(i1));
      reach = fmax(reach, margin(i1));
    }
    if (sg * f > best + 2 * hd + 2 * reach) {
      list = 0;
      n = 0;
    }
    for (int i = i0; i < i1; ++i)
      if (sg * field(i) <= best + 2 * hd + 2 * reach) {
        if (n < kSdfCellRows) list |= (uint64_t)i << (8 * n + 8);
        ++n;
      }
    f = sg * best;
    i0 = i1;
  }
  cells[c] = n <= kSdfCellRows ? list | (uint64_t)n : 0xFFull;
}

// ------------------------------------------------------------------ prefix sum
// start[c] = count[0] + ... + count[c - 1] over n cells, and the total: sums of 4096 counts,
// their running sums, then the counts of each block again.
constexpr int kScanItems = 16;

__device__ __forceinline__ uint32_t block_scan(uint32_t v, uint32_t* s_wave, uint32_t* total) {
  uint32_t run = v;
  for (int off = 1; off < 64; off <<= 1) {
    const uint32_t u = __shfl_up(run, off);
    if ((int)__lane_id() >= off) run += u;
  }
  const int wave = threadIdx.x >> 6;
  if (__lane_id() == 63) s_wave[wave] = run;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (int w = 0; w < 4; ++w) {
    if (w < wave) before += s_wave[w];
    all += s_wave[w];
  }
  __syncthreads();
  *total = all;
  return before + run - v;
}

__global__ void __launch_bounds__(256) scan_sums_kernel(const uint32_t* count, int64_t n, uint32_t* sums) {
  __shared__ uint32_t s_wave[4];
  const int64_t b = ((int64_t)blockIdx.x * 256 + threadIdx.x) * kScanItems;
  uint32_t v = 0, total;
  for (int k = 0; k < kScanItems; ++k) v += b + k < n ? count[b + k] : 0u;
  block_scan(v, s_wave, &total);
  if (threadIdx.x == 0) sums[blockIdx.x] = total;
}

__global__ void __launch_bounds__(256) scan_blocks_kernel(uint32_t* sums, int n_blocks, uint32_t* total_out) {
  __shared__ uint32_t s_wave[4];
  uint32_t carry = 0;
  for (int b = 0; b < n_blocks; b += 256) {
    const int i = b + (int)threadIdx.x;
    const uint32_t v = i < n_blocks ? sums[i] : 0u;
    uint32_t total;
    const uint32_t e = block_scan(v, s_wave, &total);
    if (i < n_blocks) sums[i] = carry + e;
    carry += total;
  }
  if (threadIdx.x == 0) *total_out = carry;
}

__global__ void __launch_bounds__(256) scan_write_kernel(const uint32_t* count, int64_t n, const uint32_t* sums,
                                                         uint32_t* start) {
  __shared__ uint32_t s_wave[4];
  const int64_t b = ((int64_t)blockIdx.x * 256 + threadIdx.x) * kScanItems;
  uint32_t v = 0, total;
  for (int k = 0; k < kScanItems; ++k) v += b + k < n ? count[b + k] : 0u;
  uint32_t e = sums[blockIdx.x] + block_scan(v, s_wave, &total);
  for (int k = 0; k < kScanItems && b + k < n; ++k) {
    start[b + k] = e;
    e += count[b + k];
  }
}

// ====================================================================== launchers

static inline unsigned blocks_for(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }

template <int DIM, typename SRC>
static hipError_t classify_t(int geom, const void* P64, const SRC& src, int64_t n, int8_t* inside, hipStream_t st) {
  const DevProblem<double>* P = (const DevProblem<double>*)P64;
  const dim3 b(256), ga(blocks_for(n, 256)), gc(blocks_for(n, kClassifyPoints));
  if (geom == GK_BALL)
    hipLaunchKernelGGL((classify_analytic_kernel<DIM, GK_BALL, SRC>), ga, b, 0, st, P, src, n, inside);
  else if (geom == GK_BOX)
    hipLaunchKernelGGL((classify_analytic_kernel<DIM, GK_BOX, SRC>), ga, b, 0, st, P, src, n, inside);
  else if (geom == GK_SDF)
    hipLaunchKernelGGL((classify_analytic_kernel<DIM, GK_SDF, SRC>), ga, b, 0, st, P, src, n, inside);
  else if (geom == (DIM == 2 ? GK_POLYGON : GK_TRIMESH))
    hipLaunchKernelGGL((classify_cells_kernel<DIM, DIM == 2 ? GK_POLYGON : GK_TRIMESH, SRC>), gc, b, 0, st, P, src, n,
                       inside);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_classify(int dim, int geom, const void* P64, const double* pts, int64_t n, int8_t* inside,
                           hipStream_t st) {
  if (n == 0) return hipSuccess;
  return dim == 2 ? classify_t<2>(geom, P64, ArrayPoints<2>{pts}, n, inside, st)
                  : classify_t<3>(geom, P64, ArrayPoints<3>{pts}, n, inside, st);
}

template <typename T, int DIM>
static hipError_t prep_t(int geom, const dim3& g, const PrepArgs& a, hipStream_t st) {
  const dim3 b(256);
  if (geom == GK_BALL) hipLaunchKernelGGL((prep_kernel<T, DIM, GK_BALL>), g, b, 0, st, a);
  else if (geom == GK_BOX) hipLaunchKernelGGL((prep_kernel<T, DIM, GK_BOX>), g, b, 0, st, a);
  else if (geom == GK_SDF) hipLaunchKernelGGL((prep_kernel<T, DIM, GK_SDF>), g, b, 0, st, a);
  else if (geom == (DIM == 2 ? GK_POLYGON : GK_TRIMESH))
    hipLaunchKernelGGL((prep_kernel<T, DIM, DIM == 2 ? GK_POLYGON : GK_TRIMESH>), g, b, 0, st, a);
  else return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_prep(int fp64, int dim, int geom, PrepArgs& a, hipStream_t st) {
  const int points = geom == GK_POLYGON || geom == GK_TRIMESH ? kClassifyPoints : 256;
  a.block0[0] = 0;
  for (int k = 0; k < a.n; ++k) a.block0[k + 1] = a.block0[k] + blocks_for(a.item[k].n_points, points);
  // at least one block writes the tables; slots beyond the points' share get blocks of their own
  const uint64_t clear = std::min<uint64_t>((a.slot_words + 2047) / 2048, 4096);
  const dim3 g((unsigned)std::max<uint64_t>(std::max<uint64_t>(a.block0[a.n], clear), 1));
  if (fp64) return dim == 2 ? prep_t<double, 2>(geom, g, a, st) : prep_t<double, 3>(geom, g, a, st);
  return dim == 2 ? prep_t<float, 2>(geom, g, a, st) : prep_t<float, 3>(geom, g, a, st);
}

template <int DIM>
static hipError_t sigma_t(int geom, const void* P64, const double* lo, const double* h, int grid, int64_t first,
                          int64_t n, int nblocks, int8_t* inside, double* out, hipStream_t st) {
  SamplePoints<DIM> src;
  for (int i = 0; i < 3; ++i) {
    src.lo[i] = lo[i];
    src.h[i] = h[i];
  }
  src.grid = grid;
  src.first = first;
  const hipError_t e = classify_t<DIM>(geom, P64, src, n, inside, st);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((sigma_sample_kernel<DIM>), dim3(nblocks), dim3(256), 0, st, (const DevProblem<double>*)P64, src,
                     n, inside, out);
  return hipGetLastError();
}

hipError_t launch_sigma_sample(int dim, int geom, const void* P64, const double* lo, const double* h, int grid,
                               int64_t first, int64_t n, int nblocks, int8_t* inside, double* out, hipStream_t st) {
  return dim == 2 ? sigma_t<2>(geom, P64, lo, h, grid, first, n, nblocks, inside, out, st)
                  : sigma_t<3>(geom, P64, lo, h, grid, first, n, nblocks, inside, out, st);
}

hipError_t launch_segment_count(int depth, const void* P64, const GridShape& s, const GridRule& rule, double* best,
                                uint32_t* count, uint32_t* sums, uint32_t* start, uint32_t* total, hipStream_t st) {
  const int64_t n = s.cells();
  const DevProblem<double>* P = (const DevProblem<double>*)P64;
  const dim3 g((unsigned)CellBlocks<2>::blocks(s)), b(64);
  hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(256), 0, st, (uint32_t*)nullptr, 0, total + 1);   // = 0
  if (depth > kBuildStack)
    hipLaunchKernelGGL((segment_count_kernel<true>), g, b, 0, st, P, s, rule, best, count, total + 1);
  else
    hipLaunchKernelGGL((segment_count_kernel<false>), g, b, 0, st, P, s, rule, best, count, total + 1);
  const unsigned nb = blocks_for(n, 256 * kScanItems);
  hipLaunchKernelGGL(scan_sums_kernel, dim3(nb), dim3(256), 0, st, count, n, sums);
  hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(256), 0, st, sums, (int)nb, total);
  hipLaunchKernelGGL(scan_write_kernel, dim3(nb), dim3(256), 0, st, count, n, sums, start);
  return hipGetLastError();
}

hipError_t launch_segment_fill(int depth, const void* P64, const GridShape& s, const GridRule& rule, const double* best,
                               const uint32_t* start, const GridOut& out, hipStream_t st) {
  const DevProblem<double>* P = (const DevProblem<double>*)P64;
  const dim3 g((unsigned)CellBlocks<2>::blocks(s)), b(64);
  if (depth > kBuildStack) hipLaunchKernelGGL((segment_fill_kernel<true>), g, b, 0, st, P, s, rule, best, start, out);
  else hipLaunchKernelGGL((segment_fill_kernel<false>), g, b, 0, st, P, s, rule, best, start, out);
  return hipGetLastError();
}

hipError_t launch_mesh_cells(int depth, const void* P64, const GridShape& s, const GridRule& rule, double* best,
                             const GridOut& out, uint32_t* total, hipStream_t st) {
  const DevProblem<double>* P = (const DevProblem<double>*)P64;
  const dim3 g((unsigned)CellBlocks<3>::blocks(s)), b(64);
  hipLaunchKernelGGL(scan_blocks_kernel, dim3(1), dim3(256), 0, st, (uint32_t*)nullptr, 0, total);   // total = 0
  if (depth > kBuildStack) hipLaunchKernelGGL((mesh_cells_kernel<true>), g, b, 0, st, P, s, rule, best, out, total);
  else hipLaunchKernelGGL((mesh_cells_kernel<false>), g, b, 0, st, P, s, rule, best, out, total);
  return hipGetLastError();
}

hipError_t launch_cell_classes(int dim, const void* P64, const GridShape& s, double reach, const double* best,
                               uint32_t* label, uint32_t* roots, uint32_t* n_roots, uint8_t* cls, hipStream_t st) {
  const int64_t n = s.cells();
  const DevProblem<double>* P = (const DevProblem<double>*)P64;
  const dim3 g(blocks_for(n, 256)), b(256);
  hipLaunchKernelGGL(label_init_kernel, g, b, 0, st, best, reach, n, s.nx, label, n_roots);
  hipLaunchKernelGGL(label_join_kernel, g, b, 0, st, label, s.nx, s.ny, s.nz);
  hipLaunchKernelGGL(label_roots_kernel, g, b, 0, st, label, n, roots, n_roots);
  if (dim == 2)
    hipLaunchKernelGGL((root_class_kernel<GK_POLYGON>), dim3(512), b, 0, st, P, s, roots, n_roots, cls);
  else
    hipLaunchKernelGGL((root_class_kernel<GK_TRIMESH>), dim3(512), b, 0, st, P, s, roots, n_roots, cls);
  hipLaunchKernelGGL(cell_class_kernel, g, b, 0, st, label, n, cls);
  return hipGetLastError();
}

hipError_t launch_sdf_cells(int dim, const void* P64, const GridShape& s, double scale, uint64_t* cells, hipStream_t st) {
  const DevProblem<double>* P = (const DevProblem<double>*)P64;
  if (dim == 2)
    hipLaunchKernelGGL((sdf_cells_kernel<2>), dim3((unsigned)CellBlocks<2>::blocks(s)), dim3(64), 0, st, P, s, scale, cells);
  else
    hipLaunchKernelGGL((sdf_cells_kernel<3>), dim3((unsigned)CellBlocks<3>::blocks(s)), dim3(64), 0, st, P, s, scale, cells);
  return hipGetLastError();
}

size_t scan_sum_words(int64_t cells) { return blocks_for(cells, 256 * kScanItems); }

}  // namespace wos
