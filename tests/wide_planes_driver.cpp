// Checks of the four-wide nodes' FP16 planes on the host: a plane rounds
// outwards, is never a subnormal and is at most one step away, for every FP16
// value, its FP32 neighbours and random FP32 values; a quantised box contains
// its FP32 box in any grid.
#include <cmath>
#include <cstdio>
#include <cstring>
#include <random>

#include "../paper_2111_06906_amd/csrc/pv_device.h"

static float half_value(uint32_t h) {
  const uint32_t e = (h >> 10) & 31u, m = h & 1023u;
  const float s = (h >> 15) ? -1.0f : 1.0f;
  if (e == 31u) return m ? NAN : s * INFINITY;
  return e ? s * std::ldexp(1.0f + (float)m / 1024.0f, (int)e - 15) : s * std::ldexp((float)m, -24);
}

static long bad = 0;
static void check(float x) {
  if (!std::isfinite(x)) return;
  const uint32_t d = pv::half_down(x), u = pv::half_up(x);
  const float a = half_value(d), b = half_value(u);
  const float tiny = 6.103515625e-5f, step = std::max(std::fabs(x) * 9.8e-4f, tiny);
  const bool in = a <= x && x <= b;
  const bool normal = (((d >> 10) & 31u) || !(d & 1023u)) && (((u >> 10) & 31u) || !(u & 1023u));
  const bool near_ = std::fabs(x) > 65504.0f || (x - a <= step && b - x <= step);
  if (!(in && normal && near_) && ++bad < 10) std::printf("x %.9g down %.9g up %.9g\n", x, a, b);
}

int main() {
  for (uint32_t h = 0; h < 65536; ++h) {
    const float v = half_value(h);
    check(v);
    check(std::nextafterf(v, INFINITY));
    check(std::nextafterf(v, -INFINITY));
  }
  std::mt19937 g(5);
  for (int i = 0; i < 2000000; ++i) {
    uint32_t w = (uint32_t)g();
    float x;
    std::memcpy(&x, &w, 4);
    check(x);
  }
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  for (int i = 0; i < 2000000; ++i) {
    const float size = std::ldexp(1.0f, (int)(g() % 24) - 8), c = (float)(U(g) * size * 4.0);
    int ex;
    std::frexp(size, &ex);
    const float s = std::ldexp(1.0f, 8 - ex);
    const float lo = (float)(c + U(g) * size), hi = lo + (float)std::fabs(U(g) * size);
    const uint32_t w = pv::wide_planes(lo, hi, c, s);
    const double a = half_value(w & 0xFFFFu) / (double)s + (double)c, b = half_value(w >> 16) / (double)s + (double)c;
    if (!(a <= lo && hi <= b) && ++bad < 20) std::printf("box %.9g %.9g c %.9g s %g: %.9g %.9g\n", lo, hi, c, s, a, b);
  }
  // with a node's origin: a box inside a grid of 256 steps, origin near its
  // middle (or clamped, for boxes outside), planes relative to it
  for (int i = 0; i < 2000000; ++i) {
    const float half = std::ldexp(1.0f, (int)(g() % 24) - 8);
    const float s = 128.0f / half, c = (float)(U(g) * half * 4.0) - half;
    const float size = half * std::ldexp(1.0f, -(int)(g() % 16));
    const float lo = (float)(c + (i % 8 ? 2.0 : 5.0) * half * std::fabs(U(g))), hi = lo + (float)std::fabs(U(g) * size);
    const uint32_t o = pv::wide_origin(0.5f * lo + 0.5f * hi, c, s);
    const uint32_t w = pv::wide_planes(lo, hi, c, s, (float)o);
    const double a = (half_value(w & 0xFFFFu) + (double)o) / (double)s + (double)c;
    const double b = (half_value(w >> 16) + (double)o) / (double)s + (double)c;
    // inside the grid: within an FP16 step of the distance to the origin, and
    // the slack
    const double reach = std::max(std::fabs((lo - (double)c) * s - o), std::fabs((hi - (double)c) * s - o));
    const double slack = (reach * 2e-3 + 4e-4) / s;
    const bool tight = a >= lo - slack && b <= hi + slack;
    if (!(o <= 255u && a <= lo && hi <= b && tight) && ++bad < 30)
      std::printf("box %.9g %.9g c %.9g s %g origin %u: %.9g %.9g\n", lo, hi, c, s, o, a, b);
  }
  std::printf("planes checked, %ld wrong\n", bad);
  return bad != 0;
}
