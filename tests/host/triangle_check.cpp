// Closest points of triangles (csrc/triangle.h) on the CPU, in FP64 and FP32, over triangles
// and points with small integer coordinates, where most tests of a region tie with another's.
//
// Usage: triangle_check <number of triangles> <seed>
// Every triangle is taken in all six vertex orders, with points drawn from the lattice, at its
// vertices, on its edges and straight above them. A wrong point is one further than `tol` from
// the closest point by brute force (the face where the projection falls inside it, else the
// nearest of the three edges, in long double); triangles of zero area are left out. Prints
// "tests N ties T wrong64 W wrong32 V".
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <random>

namespace wos {
inline float m_fma(float a, float b, float c) { return std::fma(a, b, c); }
inline double m_fma(double a, double b, double c) { return std::fma(a, b, c); }
inline float m_div(float a, float b) { return a * (1.0f / b); }   // the device multiplies by a reciprocal
inline double m_div(double a, double b) { return a / b; }
}  // namespace wos

#include "triangle.h"

using V = long double;

static V dot(const V* a, const V* b) { return a[0] * b[0] + a[1] * b[1] + a[2] * b[2]; }

static V edge_point(const V* a, const V* b, const V* p, V* q) {
  V e[3], w[3], d = 0;
  for (int k = 0; k < 3; ++k) {
    e[k] = b[k] - a[k];
    w[k] = p[k] - a[k];
  }
  const V t = std::fmin(1.0L, std::fmax(0.0L, dot(w, e) / dot(e, e)));
  for (int k = 0; k < 3; ++k) {
    q[k] = a[k] + t * e[k];
    d += (p[k] - q[k]) * (p[k] - q[k]);
  }
  return d;
}

static void brute(const V t[3][3], const V* p, V* q) {
  V ab[3], ac[3], ap[3];
  for (int k = 0; k < 3; ++k) {
    ab[k] = t[1][k] - t[0][k];
    ac[k] = t[2][k] - t[0][k];
    ap[k] = p[k] - t[0][k];
  }
  const V d00 = dot(ab, ab), d01 = dot(ab, ac), d11 = dot(ac, ac), d20 = dot(ap, ab), d21 = dot(ap, ac);
  const V den = d00 * d11 - d01 * d01, v = (d11 * d20 - d01 * d21) / den, w = (d00 * d21 - d01 * d20) / den;
  if (v >= 0 && w >= 0 && v + w <= 1) {
    for (int k = 0; k < 3; ++k) q[k] = t[0][k] + v * ab[k] + w * ac[k];
    return;
  }
  V best = HUGE_VALL, c[3];
  for (int e = 0; e < 3; ++e) {
    const V d = edge_point(t[e], t[(e + 1) % 3], p, c);
    if (d < best) {
      best = d;
      for (int k = 0; k < 3; ++k) q[k] = c[k];
    }
  }
}

template <typename T>
static bool wrong(const double t[3][3], const double* p, const V* want, V tol) {
  T tri[9], x[3], q[3];
  for (int v = 0; v < 3; ++v)
    for (int k = 0; k < 3; ++k) tri[3 * v + k] = (T)t[v][k];
  for (int k = 0; k < 3; ++k) x[k] = (T)p[k];
  wos::triangle_closest<T>(x, (const T*)tri, q);
  for (int k = 0; k < 3; ++k)
    if (!(std::fabs((V)q[k] - want[k]) <= tol)) return true;
  return false;
}

int main(int argc, char** argv) {
  if (argc < 3) return 2;
  const int n = std::atoi(argv[1]);
  std::mt19937_64 rng((uint64_t)std::atoll(argv[2]));
  auto lattice = [&](int r) { return (double)((int)(rng() % (uint64_t)(2 * r + 1)) - r); };
  long long tests = 0, ties = 0, w64 = 0, w32 = 0;
  static const int kOrder[6][3] = {{0, 1, 2}, {0, 2, 1}, {1, 0, 2}, {1, 2, 0}, {2, 0, 1}, {2, 1, 0}};
  for (int i = 0; i < n; ++i) {
    double t[3][3], nrm[3];
    for (auto& v : t)
      for (double& c : v) c = lattice(3);
    for (int k = 0; k < 3; ++k) {
      const int a = (k + 1) % 3, b = (k + 2) % 3;
      nrm[k] = (t[1][a] - t[0][a]) * (t[2][b] - t[0][b]) - (t[1][b] - t[0][b]) * (t[2][a] - t[0][a]);
    }
    if (nrm[0] == 0 && nrm[1] == 0 && nrm[2] == 0) continue;
    for (int j = 0; j < 24; ++j) {
      double p[3];
      const int v = j % 3, u = (v + 1) % 3;
      const double up = j < 6 ? 0.0 : lattice(2);
      for (int k = 0; k < 3; ++k)
        p[k] = j >= 12   ? lattice(5)                                              // anywhere
               : j % 6 < 3 ? t[v][k] + up * nrm[k]                                 // at or above a vertex
                           : 0.5 * (t[v][k] + t[u][k]) + up * nrm[k];              // at or above an edge
      V tv[3][3], pv[3], want[3];
      for (int a = 0; a < 3; ++a)
        for (int k = 0; k < 3; ++k) tv[a][k] = t[a][k];
      for (int k = 0; k < 3; ++k) pv[k] = p[k];
      brute(tv, pv, want);
      for (int a = 0; a < 3; ++a)
        if (want[0] == tv[a][0] && want[1] == tv[a][1] && want[2] == tv[a][2]) ++ties;
      for (const auto& o : kOrder) {
        double s[3][3];
        for (int a = 0; a < 3; ++a)
          for (int k = 0; k < 3; ++k) s[a][k] = t[o[a]][k];
        ++tests;
        // every product is a multiple of 1/4 below 2^22, exact in both types; a region's
        // quotient and the two roundings after it lose a few units of the last place of
        // numbers up to 12
        w64 += wrong<double>(s, p, want, 1e-13L);
        w32 += wrong<float>(s, p, want, 1e-5L);
      }
    }
  }
  std::printf("tests %lld ties %lld wrong64 %lld wrong32 %lld\n", tests, ties, w64, w32);
  return 0;
}
