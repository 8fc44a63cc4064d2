// Lists of a candidate grid as the host reference builds them (csrc/bvh.cpp), with the
// library's sizes and margins.
//
// Usage: grid_total <tri|seg> <file of doubles: [n][12] triangles or [n][4] segments>
// Prints "nx NX ny NY nz NZ candidates C truncated T".
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <vector>

#include "bvh.h"

using namespace wos;

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  const bool tri = argv[1][0] == 't';
  const int dim = tri ? 3 : 2, stride = tri ? 12 : 4, nv = tri ? 3 : 2;
  FILE* f = std::fopen(argv[2], "rb");
  if (!f) return 2;
  std::vector<double> raw;
  double buf[12];
  while (std::fread(buf, sizeof(double), stride, f) == (size_t)stride) raw.insert(raw.end(), buf, buf + stride);
  std::fclose(f);
  const int64_t n = (int64_t)raw.size() / stride;
  std::vector<double> lo(n * dim), hi(n * dim), cen(n * dim);
  double scale = 0;
  for (int64_t j = 0; j < n; ++j)
    for (int k = 0; k < dim; ++k) {
      double mn = 1e300, mx = -1e300, s = 0;
      for (int v = 0; v < nv; ++v) {
        const double c = raw[stride * j + dim * v + k];
        mn = std::min(mn, c);
        mx = std::max(mx, c);
        s += c;
        scale = std::max(scale, std::fabs(c));
      }
      lo[j * dim + k] = mn;
      hi[j * dim + k] = mx;
      cen[j * dim + k] = s / nv;
    }
  const BvhTopology t = build_bvh(lo, hi, cen, dim, n, 4);
  std::vector<double> prims(n * stride), plo(n * dim), phi(n * dim), bounds;
  for (int64_t i = 0; i < n; ++i) {
    const int32_t s = t.order[i];
    for (int k = 0; k < stride; ++k) prims[stride * i + k] = raw[stride * s + k];
    for (int k = 0; k < dim; ++k) {
      plo[dim * i + k] = lo[dim * s + k];
      phi[dim * i + k] = hi[dim * s + k];
    }
  }
  bvh_child_bounds<double>(t, plo, phi, dim, bounds);
  const double margin = 4e-6 * (scale + 1.0);
  const SegmentGrid g =
      tri ? build_triangle_grid(prims, n, t, bounds, std::min<int64_t>(1 << 21, std::max<int64_t>(32768, 128 * n)),
                                margin, kMeshCellList, 4)
          : build_segment_grid(prims, n, t, bounds, std::min<int64_t>(1 << 20, std::max<int64_t>(4096, 64 * n)), margin,
                               kPolygonCellMax, kPolygonDeepList);
  int64_t truncated = 0;
  for (double v : g.tail) truncated += std::isfinite(v) ? 1 : 0;
  std::printf("nx %d ny %d nz %d candidates %lld truncated %lld\n", g.nx, g.ny, g.nz, (long long)g.prim.size(),
              (long long)truncated);
  return 0;
}
