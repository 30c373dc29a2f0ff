// The host checks of an object's hierarchy (csrc/pv_check.h) accept a right
// four-wide form and order and refuse each planted mistake.
#include <cstdio>
#include <random>

#include "../paper_2111_06906_amd/csrc/pv_check.h"

using namespace pv;

static std::vector<Tri> tris;
static std::vector<Wide> wide;
static const uint32_t kFirst = 5;  // records before the object's
static PlanesOf P;
static PlaneGrid grid;

// one node over four leaves of two triangles each, in a grid with origins
static void build(int unit) {
  tris.clear();
  std::mt19937 g(3);
  std::uniform_real_distribution<float> U(-0.5f, 0.5f);
  for (uint32_t i = 0; i < 8; ++i) {
    float v[9];
    for (int k = 0; k < 9; ++k) v[k] = U(g) + 0.3f * (float)(k % 3);
    tris.push_back(make_tri(v, i));
  }
  const float lo[3] = {-1, -1, -1}, hi[3] = {1, 1, 1};
  grid = plane_grid(lo, hi, true);
  P = PlanesOf{grid.qc, grid.qm, grid.qs, kOriginShift, unit != 0};
  const float s = std::ldexp(grid.qs, -unit);
  Wide w{};
  for (uint32_t c = 0; c < 4; ++c) {
    for (int k = 0; k < 3; ++k) {
      float l = INFINITY, h = -INFINITY;
      for (uint32_t i = 2 * c; i < 2 * c + 2; ++i)
        for (int v = 0; v < 3; ++v) {
          l = std::min(l, tris[i].v[v][k]);
          h = std::max(h, tris[i].v[v][k]);
        }
      w.plane[3 * c + k] = unit ? wide_planes(l, h, grid.qm[k], s, 0.0f) : wide_planes(l, h, grid.qc[k], s, 128.0f);
    }
    w.child[c] = wide_code(leaf_code(kFirst + 2 * c, 2), kOriginShift) | (c < 3 ? 128 : (unit & 255));
  }
  wide.assign(1, w);
}

static long bad = 0;
static bool valid(int32_t root = 0) {
  return check_wide(wide.data(), (uint32_t)wide.size(), root, P, tris.data(), kFirst, (uint32_t)tris.size());
}
static void expect(bool want, bool got, const char* what) {
  if (want != got) std::printf("%s: %d\n", what, got), ++bad;
}

int main() {
  for (int unit : {0, 3, -2}) {
    build(unit);
    expect(true, valid(), "a right node");
    wide[0].plane[4] = (wide[0].plane[4] & 0xFFFF0000u) | ((wide[0].plane[4] >> 16) & 0x7FFFu);  // lower = upper
    expect(false, valid(), "a plane inside the box");
    build(unit);
    wide[0].child[1] += 1;  // the origin's y
    expect(false, valid(), "an origin off by a step");
    build(unit);
    wide[0].child[3] = (wide[0].child[3] & ~255) | ((unit - 1) & 255);
    expect(false, valid(), "a unit too small, or one that is not read");
    build(unit);
    std::swap(wide[0].child[0], wide[0].child[1]);
    expect(false, valid(), "children exchanged");
    build(unit);
    wide[0].child[2] = wide_code(leaf_code(kFirst + 2, 2), kOriginShift) | 128;
    expect(false, valid(), "a leaf twice, another missing");
    build(unit);
    for (int k = 0; k < 3; ++k) wide[0].plane[9 + k] = kPlanesNone;
    expect(false, valid(), "a leaf's slot empty");
    build(unit);
    wide[0].child[0] = wide_code(0, kOriginShift) | 128;
    expect(false, valid(), "a node below itself");
  }
  build(0);
  P.scaled = true;  // the step read as a unit of 2^0
  expect(true, valid(), "the step as a unit");
  // order: codes by centroid, equal codes by record
  std::vector<Tri> t;
  const float at[6] = {0.9f, 0.1f, 0.5f, 0.1f, 0.0f, 1.0f};
  for (uint32_t i = 0; i < 6; ++i) {
    float v[9];
    for (int k = 0; k < 9; ++k) v[k] = k % 3 == 0 ? at[i] : 0.0f;
    t.push_back(make_tri(v, i));
  }
  expect(true, check_code_order({4, 1, 3, 2, 0, 5}, t.data(), 6), "the order of the codes");
  expect(false, check_code_order({4, 3, 1, 2, 0, 5}, t.data(), 6), "equal codes exchanged");
  expect(false, check_code_order({4, 1, 3, 0, 2, 5}, t.data(), 6), "codes out of order");
  std::printf("checks checked, %ld wrong\n", bad);
  return bad != 0;
}
