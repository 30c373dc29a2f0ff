// The slab parameters that a walk forms from FP16 planes, on the host: the chain
// of FP32 roundings of the box tests (csrc/pv_device.h), with the reciprocal up
// to an ulp off either way, never lets a box be entered late or left early, for
// ray origins up to kRayReach steps from the grid's base along an axis.
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
  std::mt19937_64 g(7);
  std::uniform_real_distribution<double> U(-1.0, 1.0);
  long bad = 0;
  for (long i = 0; i < 4000000; ++i) {
    const bool origins = i & 1;
    // largest half extent of the static world, its grid, a box inside
    const float half = (float)std::ldexp(i % 8 < 4 ? 0.9999 : 0.75 + 0.25 * U(g), (int)(g() % 12) - 4);
    int ex;
    (void)std::frexp(half, &ex);
    const float s = std::ldexp(1.0f, (origins ? 7 : 8) - ex), inv_s = 1.0f / s;
    const float mid = (float)(U(g) * half * 4.0), c = mid - (origins ? 128.0f * inv_s : 0.0f);
    // boxes and origins anywhere, or near opposite ends, where roundings are largest
    const bool ends = i % 32 >= 16;
    const double side = std::copysign(1.0, U(g)), near_end = 1.0 - 0.02 * std::fabs(U(g));
    float lo = (float)(mid + (ends ? side * near_end : U(g)) * half);
    float hi = lo + (float)std::fabs(U(g) * half * std::ldexp(1.0, -(int)(g() % 12)));
    const uint32_t org = origins ? pv::wide_origin(0.5f * lo + 0.5f * hi, c, s) : 0u;
    // the box with the same planes whose lower (upper) bound is closest to them
    auto planes = [&](float l, float h) { return pv::wide_planes(l, h, c, s, (float)org, pv::kPlaneSlack); };
    const uint32_t w = planes(lo, hi);
    float l0 = lo - half * 4e-3f, h1 = hi + half * 4e-3f;
    for (int step = 0; step < 40; ++step) {
      const float ml = 0.5f * (l0 + lo), mh = 0.5f * (h1 + hi);
      if (((planes(ml, hi) ^ w) & 0xFFFFu) == 0) lo = ml; else l0 = ml;
      if ((planes(lo, mh) ^ w) >> 16 == 0) hi = mh; else h1 = mh;
    }
    // a ray from inside the world or as far out as the planes reach
    const float reach = (i % 4 < 2 ? half : pv::kRayReach * inv_s);
    const float o = i % 4 < 2 ? (float)(mid + (ends ? -side * near_end : U(g)) * half) : (float)(c + (i % 16 < 4 ? std::copysign(0.9999, U(g)) : U(g)) * reach);
    const float d = (float)std::copysign(std::exp(U(g) * 3.0 - 3.0), U(g)), tmin = (float)(1e-4 * std::fabs(U(g)));
    float inv = 1.0f / d;
    const int ulp = (int)(g() % 3) - 1;
    if (ulp) inv = std::nextafter(inv, ulp > 0 ? INFINITY : -INFINITY);
    const float k = 1.0f / 1099511627776.0f, q = inv * (inv_s * k);
    float oi = ((c - o) * inv - tmin) * k;
    if (origins) oi = std::fmaf((float)org, q, oi);
    const float a = std::fmaf(half_value(w & 0xFFFFu), q, oi), b = std::fmaf(half_value(w >> 16), q, oi);
    const float near_ = std::fmin(a, b), far_ = std::fmax(a, b);
    const double t0 = ((double)(d > 0 ? lo : hi) - o) / d, t1 = ((double)(d > 0 ? hi : lo) - o) / d;
    if (t0 > tmin) {
      const float ts = ((float)t0 - tmin) * k;  // a crossing on the near side as the interval's end
      if (!(near_ <= ts) && ++bad < 10)
        std::printf("entered late: origins %d lo %.9g hi %.9g o %.9g d %.9g half %g\n", origins, lo, hi, o, d, half);
    }
    if (!((double)far_ >= (t1 - tmin) * k) && ++bad < 10)
      std::printf("left early: origins %d lo %.9g hi %.9g o %.9g d %.9g half %g\n", origins, lo, hi, o, d, half);
  }
  std::printf("slabs checked, %ld wrong\n", bad);
  return bad != 0;
}
