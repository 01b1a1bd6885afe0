// Random chains of rotations about bonds, composed root to leaf in FP32 in two
// ways (products fused into sums, and every operation rounded), as two kernels'
// forward kinematics may be compiled: the nodes that corner_range gives for one
// placement, widened by fk_spread, hold the cell of the other.  Frames up to
// 1e6 Angstrom from the origin, spacings from 0.02 to 1 Angstrom.  Prints
//   missed N far N fixed N   (misses; cases whose cells differ; of those, misses
//                             of a margin of a hundredth of a cell alone)
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

#include "dock_internal.h"

template <bool FUSED>
static float dot4(const float* m, const float* v, float t) {
#pragma clang fp contract(off)
  if (FUSED) return std::fma(m[0], v[0], std::fma(m[1], v[1], std::fma(m[2], v[2], t)));
  return ((m[0] * v[0] + m[1] * v[1]) + m[2] * v[2]) + t;
}

struct Tf {
  float m[9], t[3];
};

template <bool FUSED>
static Tf compose(const Tf& a, const Tf& b) {
  Tf c;
  for (int i = 0; i < 3; ++i) {
    for (int j = 0; j < 3; ++j) {
      const float col[3] = {b.m[j], b.m[3 + j], b.m[6 + j]};
      c.m[3 * i + j] = dot4<FUSED>(a.m + 3 * i, col, 0.f);
    }
    c.t[i] = dot4<FUSED>(a.m + 3 * i, b.t, a.t[i]);
  }
  return c;
}

template <bool FUSED>
static Tf bond(const float* u, const float* xb, float th) {
  const float s = std::sin(th), c = std::cos(th), oc = 1.f - c;
  Tf f;
  const float m[9] = {c + u[0] * u[0] * oc,        u[0] * u[1] * oc - u[2] * s, u[0] * u[2] * oc + u[1] * s,
                      u[1] * u[0] * oc + u[2] * s, c + u[1] * u[1] * oc,        u[1] * u[2] * oc - u[0] * s,
                      u[2] * u[0] * oc - u[1] * s, u[2] * u[1] * oc + u[0] * s, c + u[2] * u[2] * oc};
  for (int i = 0; i < 9; ++i) f.m[i] = m[i];
  for (int i = 0; i < 3; ++i) f.t[i] = xb[i] - dot4<FUSED>(f.m + 3 * i, xb, 0.f);
  return f;
}

int main() {
  std::mt19937 rng(7);
  std::uniform_real_distribution<float> uni(-1.f, 1.f);
  long missed = 0, far = 0, fixed = 0;
  for (int it = 0; it < 500000; ++it) {
    const float frame = it % 4 == 0 ? 0.f : std::pow(10.f, 2.f + 4.f * std::fabs(uni(rng)));
    const float h = std::pow(10.f, -1.7f * std::fabs(uni(rng))), reach = 4.f + 26.f * std::fabs(uni(rng));
    const int n = 33, depth = rng() % 20;
    float T[3], ang[3], a[3], o[3], hi[3];
    for (int c = 0; c < 3; ++c) {
      o[c] = frame * uni(rng);
      hi[c] = float(double(o[c]) + double(h) * (n - 1));
      T[c] = o[c] + 0.5f * h * (n - 1) * (1.f + uni(rng));
      ang[c] = 3.14f * uni(rng);
      a[c] = reach * uni(rng);
    }
    const float sa = std::sin(ang[0]), ca = std::cos(ang[0]), sb = std::sin(ang[1]), cb = std::cos(ang[1]),
                sg = std::sin(ang[2]), cg = std::cos(ang[2]);
    Tf w[2];
    const Tf root{{ca * cb, ca * sb * sg - sa * cg, ca * sb * cg + sa * sg, sa * cb, sa * sb * sg + ca * cg,
                   sa * sb * cg - ca * sg, -sb, cb * sg, cb * cg},
                  {T[0], T[1], T[2]}};
    // root o ((b1 o b2) o ...), as pointer jumping composes it
    Tf local[2];
    for (int k = 0; k < depth; ++k) {
      float u[3], xb[3], len = 0.f;
      for (int c = 0; c < 3; ++c) {
        u[c] = uni(rng) + 1e-3f;
        len += u[c] * u[c];
        xb[c] = reach * uni(rng);
      }
      for (float& v : u) v /= std::sqrt(len);
      const float th = 3.14f * uni(rng);
      const Tf f0 = bond<false>(u, xb, th), f1 = bond<true>(u, xb, th);
      local[0] = k ? compose<false>(local[0], f0) : f0;
      local[1] = k ? compose<true>(local[1], f1) : f1;
    }
    w[0] = depth ? compose<false>(root, local[0]) : root;
    w[1] = depth ? compose<true>(root, local[1]) : root;
    for (int c = 0; c < 3; ++c) {
      const float p = dot4<false>(w[0].m + 3 * c, a, w[0].t[c]), q = dot4<true>(w[1].m + 3 * c, a, w[1].t[c]);
      const float inv_h = 1.0f / h;
      auto cell = [&](float v) { return std::min(int((std::min(std::max(v, o[c]), hi[c]) - o[c]) * inv_h), n - 2); };
      const int cp = cell(p), cq = cell(q);
      if (cp == cq) continue;
      ++far;
      int lo, up;
      dock::corner_range(p, dock::fk_spread(p, T[c], reach), o[c], hi[c], inv_h, n, lo, up);
      if (cq < lo || cq + 1 > up) ++missed;
      dock::corner_range(p, 0.f, o[c], hi[c], inv_h, n, lo, up);
      if (cq < lo || cq + 1 > up) ++fixed;
    }
  }
  std::printf("missed %ld far %ld fixed %ld\n", missed, far, fixed);
  return missed != 0;
}
