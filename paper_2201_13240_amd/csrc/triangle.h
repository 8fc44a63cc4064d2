// Closest point of a triangle (Sec. 7.1). Included by wos_device.h, whose m_fma and m_div it
// takes; a host program that defines those two can compile it too.
#pragma once

#if defined(__HIPCC__)
#define WOS_TRIANGLE_FN __device__ __forceinline__
#else
#define WOS_TRIANGLE_FN inline
#endif

namespace wos {

// x . y, its products added in the order 1, 0, 2 (one rounding each after the first).
template <typename T>
WOS_TRIANGLE_FN T dot3(const T* x, const T* y) {
  return m_fma(x[2], y[2], m_fma(x[0], y[0], x[1] * y[1]));
}

// Closest point of triangle (a, b, c) = (tri[0..2], tri[3..5], tri[6..8]) to p, by the
// Voronoi regions of its vertices, edges and face (Ericson, Real-Time Collision
// Detection, Sec. 5.1.5). Every region's point is a + s1 ab, rounded, plus s2 times ac (or
// ac - ab on the edge bc), so the regions select numbers instead of branching: lanes of a
// wave are spread over all of them, and as seven nested branches a triangle took twice as
// long.
template <typename T, typename PT>
WOS_TRIANGLE_FN void triangle_closest(const T* p, PT tri, T* q) {
  T a[3], ab[3], ac[3], ap[3], bp[3], cp[3];
#pragma unroll
  for (int i = 0; i < 3; ++i) {
    a[i] = tri[i];
    ab[i] = tri[3 + i] - a[i];
    ac[i] = tri[6 + i] - a[i];
    ap[i] = p[i] - a[i];
    bp[i] = ap[i] - ab[i];
    cp[i] = ap[i] - ac[i];
  }
  const T d1 = dot3(ab, ap), d2 = dot3(ac, ap), d3 = dot3(ab, bp), d4 = dot3(ac, bp), d5 = dot3(ab, cp),
          d6 = dot3(ac, cp);
  const T vc = m_fma(d1, d4, -(d3 * d2)), vb = m_fma(d5, d2, -(d1 * d6)), va = m_fma(d3, d6, -(d5 * d4));
  const T t1 = d4 - d3, t2 = d5 - d6;
  // face, then the other regions from the last tested to the first: num / den is 1 / (va + vb +
  // vc) on the face and the edge's parameter on an edge
  T num = 1, den = va + vb + vc;
  const bool on_ac = vb <= (T)0 && d2 >= (T)0 && d6 <= (T)0;
  const bool at_c = d6 >= (T)0 && d5 <= d6;
  // the edge bc, unless ac or c wins: on a tie (p straight above c, or in the plane through c
  // across bc) their tests hold as well, and the direction of s2 has to be theirs
  const bool bc = va <= (T)0 && t1 >= (T)0 && t2 >= (T)0 && !on_ac && !at_c;
  num = bc ? t1 : num;
  den = bc ? t1 + t2 : den;
  num = on_ac ? d2 : num;
  den = on_ac ? d2 - d6 : den;
  const bool on_ab = vc <= (T)0 && d1 >= (T)0 && d3 <= (T)0;
  num = on_ab ? d1 : num;
  den = on_ab ? d1 - d3 : den;
  const T r = m_div(num, den);
  const bool at_a = d1 <= (T)0 && d2 <= (T)0, at_b = d3 >= (T)0 && d4 <= d3;
  T s1 = bc ? (T)1 : vb * r, s2 = bc ? r : vc * r;
  s1 = on_ac ? (T)0 : s1;
  s2 = on_ac ? r : s2;
  s1 = at_c ? (T)0 : s1;
  s2 = at_c ? (T)1 : s2;
  s1 = on_ab ? r : s1;
  s2 = on_ab ? (T)0 : s2;
  s1 = at_b ? (T)1 : s1;
  s2 = at_b ? (T)0 : s2;
  s1 = at_a ? (T)0 : s1;
  s2 = at_a ? (T)0 : s2;
#pragma unroll
  for (int i = 0; i < 3; ++i) q[i] = m_fma(s2, bc ? ac[i] - ab[i] : ac[i], m_fma(s1, ab[i], a[i]));
}

}  // namespace wos
