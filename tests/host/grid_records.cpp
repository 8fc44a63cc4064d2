// The candidate grids that the device builds, cell by cell against the host reference
// (csrc/bvh.cpp): calls the library's own launchers on a BVH built here, with the library's
// sizes and margins, and copies the records and lists back.
//
// Usage: grid_records <tri|seg> <file of doubles: [n][12] triangles or [n][4] segments> [deep]
// (deep: with the construction's stacks in private memory, as for trees of more than 20 levels)
// Prints "cells N truncated T lists L order O tails X inline I floats F bands B": N cells, T of
// them with truncated lists, and the numbers of cells whose list differs in length, position,
// distances or members; lists out of order; tails, polygon records, FP32 copies and
// bands that are not what the list says.
#include <hip/hip_runtime_api.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <set>
#include <vector>

#include "bvh.h"
#include "wos_launch.h"
#include "wos_types.h"

using namespace wos;

static void hip(hipError_t e) {
  if (e == hipSuccess) return;
  std::fprintf(stderr, "%s\n", hipGetErrorString(e));
  std::exit(3);
}

template <typename T>
static T* upload(const std::vector<T>& v, size_t more = 0) {
  T* p = nullptr;
  hip(hipMalloc((void**)&p, (v.size() + more) * sizeof(T) + 16));
  if (!v.empty()) hip(hipMemcpy(p, v.data(), v.size() * sizeof(T), hipMemcpyHostToDevice));
  return p;
}

template <typename T>
static std::vector<T> download(const void* p, size_t n) {
  std::vector<T> v(n);
  hip(hipMemcpy(v.data(), p, n * sizeof(T), hipMemcpyDeviceToHost));
  return v;
}

template <int DIM>
static std::vector<BvhNode<double, DIM>> nodes_of(const BvhTopology& t, const std::vector<double>& b) {
  std::vector<BvhNode<double, DIM>> out(std::max<size_t>(1, t.child.size() / 2));
  for (size_t i = 0; i < t.child.size() / 2; ++i)
    for (int s = 0; s < 2; ++s) {
      for (int k = 0; k < DIM; ++k) {
        out[i].lo[s][k] = b[(i * 4 + s) * DIM + k];
        out[i].hi[s][k] = b[(i * 4 + 2 + s) * DIM + k];
      }
      out[i].child[s] = t.child[2 * i + s];
    }
  return out;
}

struct Counts {
  long long truncated = 0, lists = 0, order = 0, tails = 0, inlined = 0, floats = 0, bands = 0;
};

// A list against the reference's: distances exactly, in order; members up to equal distances.
static void check_list(const SegmentGrid& g, int64_t c, double margin, uint32_t count, const int32_t* id,
                       const std::vector<double>& dc, Counts& n) {
  const uint32_t st = g.start[c], want = g.start[c + 1] - st;
  if (count != want || dc.size() != want) {
    ++n.lists;
    return;
  }
  bool same = true, sorted = true;
  std::set<int32_t> seen;
  for (uint32_t k = 0; k < count; ++k) {
    same = same && dc[k] == g.dc[st + k] - margin && seen.insert(id[k]).second;
    sorted = sorted && (k == 0 || dc[k] >= dc[k - 1]);
    // another primitive than the reference's only where its distance is not told apart from a
    // neighbour's on the list, or from the first one off it
    if (id[k] != g.prim[st + k]) {
      const double d = g.dc[st + k];
      same = same && ((k > 0 && g.dc[st + k - 1] == d) || (k + 1 < count && g.dc[st + k + 1] == d) ||
                      (k + 1 == count && g.tail[c] == d));
    }
  }
  n.lists += !same;
  n.order += !sorted;
}

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
  const int64_t nc = g.cells();
  const int depth = argc > 3 ? 48 : t.depth;
  const GridRule rule = tri ? GridRule{cell_halfdiag(g, 3), margin, deep_distance(g), kMeshCellList, kMeshCellList}
                            : GridRule{cell_halfdiag(g, 2), margin, HUGE_VAL, kPolygonCellMax, kPolygonDeepList};

  DevProblem<double> P;
  std::memset((void*)&P, 0, sizeof(P));
  P.geom.n_prims = (int32_t)n;
  P.geom.n_nodes = (int32_t)(t.child.size() / 2);
  P.geom.root = t.root;
  P.geom.depth = t.depth;
  P.geom.prims = upload(prims);
  P.geom.nodes = tri ? (const void*)upload(nodes_of<3>(t, bounds)) : (const void*)upload(nodes_of<2>(t, bounds));
  const void* dP = upload(std::vector<DevProblem<double>>{P});
  double* best = upload(std::vector<double>(nc));
  uint32_t* total = upload(std::vector<uint32_t>(2, 0u));
  GridOut o{nullptr, nullptr, nullptr, nullptr, nullptr};
  Counts r;
  if (tri) {
    o.cells32 = upload(std::vector<MeshCell<float>>(nc));
    o.cells64 = upload(std::vector<MeshCell<double>>(nc));
    hip(launch_mesh_cells(depth, dP, g, rule, best, o, total, 0));
    const auto c32 = download<MeshCell<float>>(o.cells32, nc);
    const auto c64 = download<MeshCell<double>>(o.cells64, nc);
    for (int64_t c = 0; c < nc; ++c) {
      const MeshCell<double>& m = c64[c];
      if (m.count > (uint32_t)kMeshCellList || m.count == 0) {
        ++r.lists;
        continue;
      }
      check_list(g, c, margin, m.count, m.id, std::vector<double>(m.dc, m.dc + m.count), r);
      const bool cut = std::isfinite(g.tail[c]);
      r.truncated += cut;
      r.tails += m.tail != (cut ? g.tail[c] - margin : HUGE_VAL);
      bool pad = true, fl = c32[c].count == m.count && c32[c].tail == (float)m.tail;
      for (uint32_t k = 0; k < (uint32_t)kMeshCellList; ++k) {
        if (k >= m.count) pad = pad && m.id[k] == m.id[m.count - 1] && m.dc[k] == m.dc[m.count - 1];
        fl = fl && c32[c].id[k] == m.id[k] && c32[c].dc[k] == (float)m.dc[k];
      }
      r.inlined += !pad;
      r.floats += !fl;
    }
  } else {
    uint32_t *count = upload(std::vector<uint32_t>(nc)), *start = upload(std::vector<uint32_t>(nc)),
             *sums = upload(std::vector<uint32_t>(scan_sum_words(nc)));
    hip(launch_segment_count(depth, dP, g, rule, best, count, sums, start, total, 0));
    const std::vector<uint32_t> tot = download<uint32_t>(total, 2);
    const size_t nl = (size_t)tot[0] + kListGroup;
    o.cells32 = upload(std::vector<CellRec<float>>(nc));
    o.cells64 = upload(std::vector<CellRec<double>>(nc));
    o.prim = upload(std::vector<int32_t>(tot[0]));
    o.list32 = upload(std::vector<float>(nl * kListEntry));
    o.list64 = upload(std::vector<double>(nl * kListEntry));
    hip(launch_segment_fill(depth, dP, g, rule, best, start, o, 0));
    const auto c32 = download<CellRec<float>>(o.cells32, nc);
    const auto c64 = download<CellRec<double>>(o.cells64, nc);
    const auto prim = download<int32_t>(o.prim, tot[0]);
    const auto l32 = download<float>(o.list32, nl * kListEntry);
    const auto l64 = download<double>(o.list64, nl * kListEntry);
    for (int64_t c = 0; c < nc; ++c) {
      const CellRec<double>& m = c64[c];
      const uint32_t st = g.start[c], cnt = g.start[c + 1] - st;
      if (m.start != st || m.count != cnt || st + cnt > tot[0]) {
        ++r.lists;
        continue;
      }
      const bool cut = std::isfinite(g.tail[c]);
      r.truncated += cut;
      r.tails += m.tail != (cut ? g.tail[c] - margin : HUGE_VAL);
      // the first two entries of a truncated list hold its band: their distances are the
      // reference's where the members are
      std::vector<double> dc(cnt);
      bool rec = true, fl = c32[c].start == st && c32[c].count == cnt && c32[c].tail == (float)m.tail &&
                            c32[c].next_dc == (float)m.next_dc;
      for (uint32_t k = 0; k < cnt; ++k) {
        const double *e = &l64[(size_t)(st + k) * kListEntry], *s = &prims[4 * (size_t)prim[st + k]];
        const float* e32 = &l32[(size_t)(st + k) * kListEntry];
        if (cut && k < 2) {
          dc[k] = g.dc[st + k] - margin;
          continue;
        }
        dc[k] = e[4];
        rec = rec && std::equal(s, s + 4, e);
        for (int v = 0; v < kListEntry; ++v) fl = fl && e32[v] == (float)e[v];
      }
      check_list(g, c, margin, cnt, &prim[st], dc, r);
      for (int k = 0; cnt > 0 && k < kCellInline; ++k) {
        const double* s = &prims[4 * (size_t)prim[st + std::min<uint32_t>(k, cnt - 1)]];
        const double w[4] = {s[0], s[1], s[2] - s[0], s[3] - s[1]}, l2 = w[2] * w[2] + w[3] * w[3];
        for (int v = 0; v < 4; ++v) {
          rec = rec && m.seg[k][v] == w[v];
          fl = fl && c32[c].seg[k][v] == (float)w[v];
        }
        const double fx = (float)w[2], fy = (float)w[3], f2 = fx * fx + fy * fy;
        rec = rec && std::fabs(m.inv_len2[k] * l2 - 1.0) < 1e-15 * 4;
        fl = fl && std::fabs((double)c32[c].inv_len2[k] * f2 - 1.0) < 1.3e-7;
      }
      rec = rec && (cnt <= (uint32_t)kCellInline || m.next_dc == dc[kCellInline]);
      r.inlined += !rec;
      r.floats += !fl;
      if (cut) {
        // every listed segment within the band, in both precisions (ends suffice: it is convex)
        const ListBand<double> b = *(const ListBand<double>*)&l64[(size_t)st * kListEntry];
        const ListBand<float> b32 = *(const ListBand<float>*)&l32[(size_t)st * kListEntry];
        auto inside = [&](const auto& B, double slack) {
          const double e[2] = {(double)B.axis[2], (double)B.axis[3]};
          for (uint32_t k = 0; k < cnt; ++k)
            for (int v = 0; v < 4; v += 2) {
              const double* s = &prims[4 * (size_t)prim[st + k]];
              const double q[2] = {s[v] - (double)B.axis[0], s[v + 1] - (double)B.axis[1]};
              const double u = std::min(1.0, std::max(0.0, (q[0] * e[0] + q[1] * e[1]) * (double)B.inv_len2));
              if (std::hypot(q[0] - u * e[0], q[1] - u * e[1]) > (double)B.radius - slack) return false;
            }
          return true;
        };
        // half of the band's margin stays free for the rounding of a query in FP32
        r.bands += !inside(b, margin) || !inside(b32, margin);
      }
    }
  }
  hip(hipDeviceSynchronize());
  std::printf("cells %lld truncated %lld lists %lld order %lld tails %lld inline %lld floats %lld bands %lld\n",
              (long long)nc, r.truncated, r.lists, r.order, r.tails, r.inlined, r.floats, r.bands);
  return 0;
}
