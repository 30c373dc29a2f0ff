// Host checks of a dynamic object's current hierarchy, on arrays copied back
// from the device (pv_object_hierarchy_info).
#pragma once
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <vector>

#include "pv_device.h"

namespace pv {

inline float half_float(uint32_t h) {
  const uint32_t e = (h >> 10) & 31u, m = h & 1023u;
  const float s = (h >> 15) ? -1.0f : 1.0f;
  if (e == 31u) return m ? NAN : s * INFINITY;
  return e ? s * std::ldexp(1.0f + (float)m / 1024.0f, (int)e - 15) : s * std::ldexp((float)m, -24);
}

// What the planes of a scene's four-wide nodes count from; scaled: the frame
// reads the nodes' own units.
struct PlanesOf {
  const float *qc, *qm;
  float qs;
  uint32_t shift;
  bool scaled;
};

// The four-wide form below 'root': every one of the object's triangle records
// [first, first + n) is in exactly one leaf, lies inside every box on the way to
// it as a walk of the frame decodes it, and unused slots are never entered.
// tris: the object's records.
inline bool check_wide(const Wide* wide, uint32_t n_wide, int32_t root, const PlanesOf& P, const Tri* tris,
                       uint32_t first, uint32_t n) {
  struct Item {
    int32_t code;
    double lo[3], hi[3];
  };
  std::vector<uint8_t> seen(n, 0);
  Item top{root, {-INFINITY, -INFINITY, -INFINITY}, {INFINITY, INFINITY, INFINITY}};
  std::vector<Item> st{top};
  uint32_t visits = 0;
  while (!st.empty()) {
    const Item it = st.back();
    st.pop_back();
    if (it.code < 0) {
      const int32_t code = it.code >> P.shift;
      const uint32_t f = leaf_first(code), c = leaf_count(code);
      for (uint32_t i = f; i < f + c; ++i) {
        if (i < first || i - first >= n || seen[i - first]) return false;
        seen[i - first] = 1;
        for (int v = 0; v < 3; ++v)
          for (int k = 0; k < 3; ++k) {
            const double x = tris[i - first].v[v][k];
            if (!(it.lo[k] <= x && x <= it.hi[k])) return false;
          }
      }
      continue;
    }
    const uint32_t node = (uint32_t)it.code >> P.shift;
    if (node >= n_wide || ++visits > n) return false;
    const Wide& w = wide[node];
    const int e = P.shift && P.scaled ? (int)(int8_t)(w.child[3] & 255) : 0;
    if (P.shift && !P.scaled && (w.child[3] & 255)) return false;  // a unit that no walk of the frame reads
    for (int s = 0; s < 4; ++s) {
      if (w.plane[3 * s] == kPlanesNone && w.plane[3 * s + 1] == kPlanesNone && w.plane[3 * s + 2] == kPlanesNone) continue;
      Item ch{w.child[s], {}, {}};
      for (int k = 0; k < 3; ++k) {
        const uint32_t p = w.plane[3 * s + k];
        const double org = P.shift ? (double)(w.child[k] & 255) - (P.scaled ? kOriginMid : 0.0) : 0.0;
        const double base = P.shift && P.scaled ? P.qm[k] : P.qc[k], step = std::ldexp(1.0, e) / P.qs;
        ch.lo[k] = std::max(it.lo[k], base + (org + half_float(p & 0xFFFFu)) * step);
        ch.hi[k] = std::min(it.hi[k], base + (org + half_float(p >> 16)) * step);
      }
      st.push_back(ch);
    }
  }
  return std::all_of(seen.begin(), seen.end(), [](uint8_t s) { return s != 0; });
}

// Whether 'order' (records counted from the object's first, in the depth-first
// order of a rebuilt hierarchy's leaves) is the stable order by 30-bit Morton
// code of the triangles' centroids in their box.
inline bool check_code_order(const std::vector<uint32_t>& order, const Tri* tris, uint32_t n) {
  if (order.size() != n) return false;
  std::vector<float> sum(3 * (size_t)n);
  const float third = 1.0f / 3.0f;
  float lo[3] = {INFINITY, INFINITY, INFINITY}, hi[3] = {-INFINITY, -INFINITY, -INFINITY};
  for (uint32_t i = 0; i < n; ++i)
    for (int k = 0; k < 3; ++k) {
      const float a = tris[i].v[0][k] + tris[i].v[1][k] + tris[i].v[2][k], x = a * third;
      sum[3 * (size_t)i + k] = a;
      lo[k] = std::min(lo[k], x);
      hi[k] = std::max(hi[k], x);
    }
  std::vector<uint32_t> code(n, 0), want(n);
  for (uint32_t i = 0; i < n; ++i) {
    want[i] = i;
    for (int k = 0; k < 3; ++k) {
      const float ext = hi[k] - lo[k], u = ext > 0.0f ? std::fma(sum[3 * (size_t)i + k], third, -lo[k]) / ext : 0.0f;
      const uint32_t q = std::min((uint32_t)std::max(u * 1024.0f, 0.0f), 1023u);
      for (int b = 0; b < 10; ++b) code[i] |= ((q >> b) & 1u) << (3 * b + 2 - k);
    }
  }
  std::stable_sort(want.begin(), want.end(), [&](uint32_t a, uint32_t b) { return code[a] < code[b]; });
  return want == order;
}

}  // namespace pv
