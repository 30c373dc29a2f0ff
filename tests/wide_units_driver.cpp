// Grids of nodes with units of their own (node_grid), on the host: whatever an
// object's distance and size, its planes contain its boxes and are within 2^-17
// of the distance from the grid's middle, or its own size, and walks that read
// them enter no box late and leave none early, from origins anywhere.
#include <cmath>
#include <cstdio>
#include <random>

#include "../paper_2111_06906_amd/csrc/pv_device.h"

static float half_value(uint32_t h) {
  const uint32_t e = (h >> 10) & 31u, m = h & 1023u;
  const float s = (h >> 15) ? -1.0f : 1.0f;
  if (e == 31u) return s * INFINITY;
  return e ? s * std::ldexp(1.0f + (float)m / 1024.0f, (int)e - 15) : 0.0f;
}

int main() {
  std::mt19937_64 g(11);
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  long bad = 0, units = 0;
  for (long i = 0; i < 1500000; ++i) {
    const bool fine = i & 1;  // no static world
    const float world = (float)std::ldexp(1.0 + std::fabs(U(g)), (int)(g() % 16) - 8);
    float lo3[3], hi3[3];
    for (int k = 0; k < 3; ++k) {
      const float m = fine ? 0.0f : (float)(U(g) * world * 3.0);
      lo3[k] = m - world;
      hi3[k] = m + world;
    }
    const pv::PlaneGrid p = pv::plane_grid(lo3, hi3, true);
    // an object: middle, half extent; a box inside it, one axis of it
    const float half = (float)(world * std::exp(U(g) * 9.0));
    float at[3];
    for (int k = 0; k < 3; ++k) at[k] = (float)(p.qm[k] + U(g) * world * std::exp(U(g) * 9.0));
    const pv::NodeGrid n = pv::node_grid(p.qc, p.qm, p.qs, at, half, fine);
    units += n.e != 0;
    const float lo = (float)(at[0] + U(g) * half), hi = lo + (float)std::fabs(U(g) * half * 0.1);
    const uint32_t w = pv::wide_planes(lo, hi, n.c[0], n.s, n.f[0], n.e ? pv::kUnitSlack : p.slack);
    const float a = half_value(w & 0xFFFFu), b = half_value(w >> 16);
    const double base = n.e ? p.qm[0] : p.qc[0];
    const double pa = base + ((double)a + n.f[0]) / n.s, pb = base + ((double)b + n.f[0]) / n.s;
    double far = half;
    for (int k = 0; k < 3; ++k) far = std::fmax(far, std::fabs((double)at[k] - p.qm[k]));
    // one FP16 step at the box's distance from the origin (the object's half
    // extent, or half a unit) and the slack; nodes in the grid's step add its
    const double tol = 2e-3 * half + far * std::ldexp(1.0, -16) + (n.e ? 0.0 : (p.slack + 40e-3) / p.qs);
    if (!(pa <= lo && pb >= hi && lo - pa <= tol && pb - hi <= tol) && ++bad < 10)
      std::printf("planes: e %d at %g half %g world %g: %.9g %.9g of %.9g %.9g\n", n.e, at[0], half, world, pa, pb, lo, hi);
    // a walk that reads units, from anywhere
    const float o = (float)(p.qm[0] + U(g) * world * std::exp(U(g) * 10.0));
    const float d = (float)std::copysign(std::exp(U(g) * 3.0 - 3.0), U(g)), tmin = (float)(1e-4 * std::fabs(U(g)));
    float inv = 1.0f / d;
    const int ulp = (int)(g() % 3) - 1;
    if (ulp) inv = std::nextafter(inv, ulp > 0 ? INFINITY : -INFINITY);
    const float k = 1.0f / 1099511627776.0f, q = inv * (p.qinv * k);
    const float oi = ((p.qm[0] - o) * inv - tmin) * k, u = std::ldexp(oi, -n.e), og = (float)n.o[0] - 128.0f;
    const float on = std::fmaf(og, q, std::fmaf(-pv::kWiden, std::fabs(u), u)), of = std::fmaf(og, q, std::fmaf(pv::kWiden, std::fabs(u), u));
    const float n0 = std::fmaf(d > 0 ? a : b, q, on), f0 = std::fmaf(d > 0 ? b : a, q, of);
    const double t0 = ((double)(d > 0 ? lo : hi) - o) / d, t1 = ((double)(d > 0 ? hi : lo) - o) / d;
    if (t0 > tmin && t0 < 1e6) {
      const float ts = std::ldexp(((float)t0 - tmin) * k, -n.e);
      if (!(n0 <= ts) && ++bad < 20) std::printf("entered late: e %d lo %.9g hi %.9g o %.9g d %.9g\n", n.e, lo, hi, o, d);
    }
    if (!((double)f0 >= std::ldexp((t1 - tmin) * k, -n.e)) && ++bad < 20)
      std::printf("left early: e %d lo %.9g hi %.9g o %.9g d %.9g\n", n.e, lo, hi, o, d);
  }
  std::printf("units checked (%ld of them not the step), %ld wrong\n", units, bad);
  return bad != 0;
}
