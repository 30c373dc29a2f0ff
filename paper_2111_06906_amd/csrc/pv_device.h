// Device-side data structures and inline routines of the path-verification
// library (gfx950).  Included by every .hip translation unit of the library.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/pv.h"

namespace pv {

// Pointers read from the scene descriptor are generic; casting them to the
// global address space lets the compiler emit global (not flat) memory
// instructions, which do not make LDS accesses (the traversal stack) wait for
// outstanding memory loads.
#if defined(__HIP_DEVICE_COMPILE__)
#define PV_GLOBAL __attribute__((address_space(1)))
#define PV_LDS __attribute__((address_space(3)))
#else
#define PV_GLOBAL
#define PV_LDS
#endif
template <typename T>
__device__ __forceinline__ PV_GLOBAL T* G(T* p) {
  return (PV_GLOBAL T*)p;
}
template <typename T>
__device__ __forceinline__ const PV_GLOBAL T* G(const T* p) {
  return (const PV_GLOBAL T*)p;
}

constexpr int kBlock = 256;        // threads per block of the streaming kernels
// Traversal stack: entries per lane, all in LDS (dynamic shared memory sized
// per launch from the scene's hierarchy depths).  A depth-first walk of a
// binary hierarchy holds at most one entry per internal ancestor of the node
// it visits, plus the sentinel at the bottom, and writes the far child one
// slot above the top: a walk through a top-level tree of depth t into a
// hierarchy of depth d needs t + d + 2 entries.  A four-wide walk leaves up to
// three entries per node; it gives up before it would pass the same number
// (walk_run) and the binary walk answers the query.
constexpr int kMaxStack = 40;
constexpr int kTopDepth = 7;  // top-level tree depth bound (the static root beside a median split of <= 64 objects)
constexpr int kMaxDepth = kMaxStack - kTopDepth - 2;
// the walk_run of a shallow scene: the sentinel, the entries of one full node
// and one slot above them
constexpr uint32_t kMinStack = 12;
static_assert((1 << (kTopDepth - 1)) >= PV_MAX_OBJECTS, "top-level depth bound");
__host__ __device__ inline uint32_t stack_entries(uint32_t top_depth, uint32_t depth) {
  const uint32_t n = top_depth + depth + 2;
  return n > kMinStack ? n : kMinStack;
}
constexpr uint32_t kHitNone = 0xFFFFFFFFu;

// ---------------------------------------------------------------------------
// information word (Section 4): 22-bit cell, 4-bit count, 4-bit start,
// replace bit, reuse-light bit
__host__ __device__ inline uint32_t info_nseg(uint32_t w) { return (w >> 22) & 15u; }
__host__ __device__ inline uint32_t info_start(uint32_t w) { return (w >> 26) & 15u; }
__host__ __device__ inline uint32_t info_replace(uint32_t w) { return (w >> 30) & 1u; }
__host__ __device__ inline uint32_t info_reuse(uint32_t w) { return (w >> 31) & 1u; }
__host__ __device__ inline uint32_t info_cell(uint32_t w) { return w & 0x3fffffu; }
__host__ __device__ inline uint32_t info_pack(uint32_t cell, uint32_t nseg, uint32_t start,
                                              uint32_t replace, uint32_t reuse) {
  return (cell & 0x3fffffu) | ((nseg & 15u) << 22) | ((start & 15u) << 26) | ((replace & 1u) << 30) |
         ((reuse & 1u) << 31);
}

// ---------------------------------------------------------------------------
// BVH2 node: both child boxes stored in the parent (one 64-byte line).
//   a = lo0.xyz hi0.x, b = hi0.yz lo1.xy, c = lo1.z hi1.xyz, d = (child0, child1, parent, -)
// child >= 0: internal node index; child < 0: leaf, ~child = first_tri << 3 | (count-1)
struct alignas(16) Node {
  float4 a, b, c;
  int4 d;
};

__host__ __device__ inline int leaf_code(uint32_t first, uint32_t count) {
  return ~(int)((first << 3) | (count - 1));
}
__host__ __device__ inline uint32_t leaf_first(int code) { return ((uint32_t)~code) >> 3; }
__host__ __device__ inline uint32_t leaf_count(int code) { return (((uint32_t)~code) & 7u) + 1u; }

// Four-wide node of one 64-byte line: the walks' own form of the hierarchies.
// Planes are FP16 in the scene's grid, (coordinate - qc) * qs with qs a power
// of two, less the node's origin, rounded outwards, so a quantised box contains
// its FP32 box; child k's planes are words 3 k .. 3 k + 2, (lower plane | upper
// plane << 16) per axis.  Child words are a walk's codes: those of Node shifted
// left by 8 (wide_code), and the low bytes of the first three are the origin's
// x, y, z in whole grid steps, of which the static world spans up to 256, and
// that of the fourth the exponent of the node's own unit (node_grid; 0 unless
// a dynamic object lies outside that span).  In scenes too large for 24-bit
// codes they are the plain codes and the origin is 0, the grid's centre.
//
// Why an origin per node: FP16 around the scene's centre leaves a wall's box a
// thousandth of the scene thick, so nearly every ray that starts on a wall
// walked down to that wall again (paths in a 300k-triangle interior, counted on
// the host: 16.5 nodes and 3.9 triangles a ray, 13.4 and 1.9 with FP32 planes,
// 13.7 and 1.9 with origins).  An unused slot holds +inf as its lower and
// -inf as its upper planes, which no query enters.
struct alignas(64) Wide {
  uint32_t plane[12];
  int32_t child[4];
};
constexpr uint32_t kPlanesNone = 0xFC007C00u;  // +inf, -inf
constexpr uint32_t kSlotNone = 0xFFFFFFFFu;

__host__ __device__ inline uint32_t float_bits(float x) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __float_as_uint(x);
#else
  uint32_t u;
  __builtin_memcpy(&u, &x, 4);
  return u;
#endif
}

// the largest FP16 value not above x, never a subnormal (a plane between 0
// and the smallest normal value goes outwards to one of the two)
__host__ __device__ inline uint32_t half_down(float x) {
  if (!(x < 65504.0f)) return 0x7BFFu;
  if (x < -65504.0f) return 0xFC00u;
  const uint32_t u = float_bits(x), m = u & 0x7FFFFFFFu;
  if (m < 0x38800000u) return (u >> 31) && m ? 0x8400u : 0u;
  const uint32_t h = (m - 0x38000000u) >> 13;
  return (u >> 31) ? 0x8000u | (h + ((m & 0x1FFFu) ? 1u : 0u)) : h;
}
__host__ __device__ inline uint32_t half_up(float x) { return half_down(-x) ^ 0x8000u; }

// Planes go outwards beyond their boxes' padding, for the roundings of a walk's
// slab parameters.  With every rounding 2^-24 of its result, and in distances
// along the axis, a plane P seen from a ray's origin o is off by at most
// 8 |qc - o| + |origin - qc| + 4 |P - qc| times 2^-24: qc - o, its product with
// 1 / d and that less tmin; the origin's multiply-add; the plane's multiply-add,
// the hardware reciprocal (2) and the interval's end.  The part of the box is
// kPlaneRel of its distance to qc (those 5, one for the wider slabs of
// WALK_SCALED, 2 for wide_planes' own subtractions, and one more).  The part of
// the ray is a constant, kPlaneSlack grid steps: for origins up to kRayReach
// steps from qc along every axis, four or more times the largest half extent;
// in scenes of less than half a unit at least kPlaneSlackMin units, which covers
// origins up to the 5 units that the FP32 boxes' padding covered.  Rays from
// further out are WALK_SCALED's, or not answered by these planes
// (SceneDev::wtop[2]).
constexpr float kPlaneSlack = 4.8828125e-4f;  // 2^-11
constexpr float kRayReach = 1024.0f;          // 8 x 1024 = 2^-11 x 2^24
constexpr float kPlaneSlackMin = 2.4e-6f;     // 8 x 5 x 2^-24
constexpr float kUnitSlack = 6.1035156e-5f;   // 2^-14, of a node's own unit: the ray's part is the wider slabs'
constexpr float kPlaneRel = 5.3644180e-7f;    // 9 x 2^-24

// planes of one axis of a box [lo, hi] in the grid (c, s), less the origin o and
// going outwards by 'slack' (both in units of 1 / s); the subtractions'
// roundings (2^-24 of their results) go outwards too
__host__ __device__ inline uint32_t wide_planes(float lo, float hi, float c, float s, float o = 0.0f,
                                                float slack = 0.0f) {
  const float a = (lo - c) * s, b = (hi - c) * s;
  const float da = a - o, db = b - o;
  const float ra = __builtin_fabsf(a) + __builtin_fabsf(da), rb = __builtin_fabsf(b) + __builtin_fabsf(db);
  return half_down(da - (ra * kPlaneRel + slack)) | (half_up(db + (rb * kPlaneRel + slack)) << 16);
}

// The same for object-space forms, in their own grids: a world segment mapped
// by the inverse transform is off by up to 12 x 2^-24 of the larger of its
// ends' object-space coordinates besides (the translation's subtraction, and
// three products of rounded factors and their sums), for ends and corner within
// kObjReach steps, at least 97 half extents of the object.
constexpr float kObjSlack = 0.015625f;   // 2^-6
constexpr float kObjReach = 12483.0f;    // 21 x 12483 <= 2^-6 x 2^24

// Node origins: whole grid steps 0 .. 255 from the grid's corner (qc, then 128
// steps below the scene's centre), where codes fit 24 bits.
constexpr uint32_t kOriginShift = 8;
constexpr uint32_t kOriginTris = (1u << 20) - 1;  // triangles of a scene whose nodes have origins
constexpr float kOriginMid = 128.0f;

// one axis of a node's origin: the grid step nearest to x
__host__ __device__ inline uint32_t wide_origin(float x, float c, float s) {
  const float m = (x - c) * s + 0.5f;
  return m >= 0.0f ? (m < 255.0f ? (uint32_t)m : 255u) : 0u;
}

// The planes' grid of a box: its middle qm in whole steps, so that the corner
// qc, 128 steps below it, is exact too; the step a power of two by which the
// largest half extent is 64 to 128 steps, the reach of the origins, or, in
// scenes without origins, 128 to 256 from qc = qm.
struct PlaneGrid {
  float qc[3], qm[3], qs, qinv, slack;
};

__host__ inline PlaneGrid plane_grid(const float* lo, const float* hi, bool origins) {
  PlaneGrid g;
  float half = 0.0f;
  for (int k = 0; k < 3; ++k) half = fmaxf(half, 0.5f * (hi[k] - lo[k]));
  int ex = 0;
  if (half > 0.0f && half < __builtin_inff()) (void)__builtin_frexpf(half, &ex);
  ex = (origins ? 7 : 8) - ex;
  g.qs = __builtin_ldexpf(1.0f, ex < -100 ? -100 : (ex > 100 ? 100 : ex));
  g.qinv = 1.0f / g.qs;
  g.slack = fmaxf(kPlaneSlack, kPlaneSlackMin * g.qs);
  for (int k = 0; k < 3; ++k) {
    const float m = __builtin_rintf((0.5f * lo[k] + 0.5f * hi[k]) * g.qs) * g.qinv;
    g.qm[k] = m - m == 0.0f ? m : 0.0f;
    g.qc[k] = g.qm[k] - (origins ? kOriginMid * g.qinv : 0.0f);
  }
  return g;
}

// Grid of one node's planes: lower corner c and scale s of the planes, and the
// origin, as the bytes that the node holds and as the float that is subtracted.
// The unit is the grid's step, 2^0, or 2^e steps, counted from the grid's
// middle, where the step does not serve: for what lies more than 16 steps
// beyond the origins' range, whose planes would lose digits with their distance
// from the last origin and be infinite past 65,504 steps (a walk through
// objects a thousand half extents out took 100 times as long), and for what
// reaches so far out that rays from it would begin beyond kRayReach.  With
// 'fine' (no static world sets the step) also for what the step is too coarse
// for.  All planes are then within 2^-18 of the distance from the middle.
struct NodeGrid {
  float c[3], s, f[3];
  uint32_t o[3];
  int e;
};

// ceil(log2(x)) of a positive finite x, within +-40 (slab parameters of a ray
// along an axis are near 2^60 and take the unit's factor)
__host__ __device__ inline int ceil_exp(float x) {
  const uint32_t u = float_bits(x);
  const int e = (int)(u >> 23) - 127 + ((u & 0x7FFFFFu) ? 1 : 0);
  return e < -40 ? -40 : (e > 40 ? 40 : e);
}

// at, half: middle and largest half extent of what the node's planes bound
__host__ __device__ inline NodeGrid node_grid(const float* qc, const float* qm, float qs, const float* at, float half,
                                              bool fine) {
  float need = 0.0f;
  for (int k = 0; k < 3; ++k) need = __builtin_fmaxf(need, __builtin_fabsf((at[k] - qm[k]) * qs));
  const float hs = half * qs;
  NodeGrid g;
  g.e = 0;
  const bool inside = need <= 144.0f && need + hs <= kRayReach - kOriginMid;
  if (!inside || (fine && (hs < 0.0625f || need + hs < 1.0f))) {
    const int e = ceil_exp(__builtin_fmaxf(need, hs) * (1.0f / 128.0f));
    g.e = fine && inside ? e : (e > 1 ? e : 1);
  }
  g.s = g.e ? __builtin_ldexpf(qs, -g.e) : qs;
  for (int k = 0; k < 3; ++k) {
    g.c[k] = g.e ? qm[k] : qc[k];
    g.o[k] = g.e ? wide_origin(at[k] - qm[k], -kOriginMid / g.s, g.s) : wide_origin(at[k], qc[k], qs);
    g.f[k] = (float)g.o[k] - (g.e ? kOriginMid : 0.0f);
  }
  return g;
}

// a code of Node as a walk's
__host__ __device__ inline int32_t wide_code(int32_t code, uint32_t shift) {
  return code == INT32_MIN ? code : (int32_t)((uint32_t)code << shift);
}

// Triangle record in BVH leaf order, one 64-byte line: each vertex as x, y, z,
// x, y, so that a query reads its three coordinates in any cyclic order (its
// own axis order of the watertight test) with one 12-byte load and no
// selection but that of the sign, and the global triangle id.
struct alignas(64) Tri {
  float v[3][5];
  uint32_t gid;
};

__host__ __device__ inline Tri make_tri(const float* w9, uint32_t gid) {
  Tri t;
  for (int i = 0; i < 3; ++i)
    for (int k = 0; k < 5; ++k) t.v[i][k] = w9[3 * i + k % 3];
  t.gid = gid;
  return t;
}

// ---------------------------------------------------------------------------
// scene as seen by kernels (one entry per scene of a batch; plain calls use one)
struct ObjDev {
  uint32_t gbase;      // global triangle id of its first triangle (upload order)
  uint32_t n_tris;
  uint32_t tri_base;   // first record of the object in the object-space vertex arrays
  uint32_t node_base;  // first node of its hierarchy in the scene's node array
  uint32_t n_nodes;    // internal nodes of its hierarchy
  int32_t root;        // root child code in the scene's node / triangle arrays (current hierarchy)
  int32_t sah_root;    // root of the upload-time topology (refit each frame)
  uint32_t lbvh_base;  // first node of its region for the per-frame rebuilt radix tree
  int32_t oroot;       // root of the four-wide upload-time topology with object-space boxes
  int32_t wroot;       // root of the current hierarchy's four-wide form
  int32_t sah_wroot;   // the same of the upload-time topology
  uint32_t lbvh_wbase; // first four-wide node of its region for the rebuilt radix tree
  float centre[3], half[3];  // its object-space box: middle and half extents
  float og[3], oinv;         // grid of its object-space form: corner (qc), 1 / scale
};

struct LightDev {
  float half[2];
  float power[3];
  float e1[3];      // photon power of Section 3, power / path_count
  uint32_t path_base, path_count;
  int32_t kind;     // PV_LIGHT_AREA / PV_LIGHT_SPOT / PV_LIGHT_CAMERA
  float param[2];   // spot: cos of the cone half-angle; camera: tan of the half field of view along u, v
  uint32_t pad[3];
};

struct LeafRec {          // a leaf of a hierarchy built on the host
  uint32_t first, count;  // triangle records
  int32_t parent;         // parent node, -1 when the leaf is the root
  uint32_t side;          // 0 = child0 of its parent, 1 = child1
};

// One hierarchy per scene: the static world's nodes, then every object's
// nodes, then two top-level trees rebuilt each frame (one over the static root
// and all object roots, one over the moved objects only).  Child codes and
// leaf triangle indices are absolute in the scene's node and triangle arrays,
// so one traversal loop serves every query.
constexpr uint32_t kTopNodes = PV_MAX_OBJECTS;  // internal nodes of one top-level tree
constexpr int32_t kRootNone = INT32_MIN;        // empty tree; never a leaf code (< 2^28 triangles)

struct SceneDev {
  Node* nodes;            // [static][objects][2 x kTopNodes]
  Tri* tris;              // [static][objects], leaf order
  int32_t* top;           // [2] per frame: root of the whole scene, root of the moved objects
  uint32_t top_base;      // first top-level node
  uint32_t n_static;
  int32_t sroot;          // static root code (kRootNone without static triangles)
  // the four-wide form: [static][objects][rebuilt objects][2 x kTopNodes][objects in object space]
  Wide* wide;
  // [3] per frame: four-wide roots of the whole scene and of the moved objects,
  // and the reach of the nodes' planes (bits of a float; kRayReach steps,
  // infinite or kReachNone)
  int32_t* wtop;
  uint32_t wtop_base;     // first four-wide top-level node
  int32_t swroot;         // static root code in 'wide'
  // grid of the planes: corner, middle, scale (a power of two), 1 / scale
  float qc[3], qm[3], qs, qinv;
  float qslack;           // their slack, in steps
  uint32_t wshift;        // kOriginShift: the nodes have origins; 0: they have none
  float sbox[6];          // static world box (lo, hi)
  // dynamic objects
  const float* dlocal;    // [n][9] object-space vertices in leaf order
  const uint32_t* dtri_gid;  // [n] global id of each leaf-order triangle
  float4* pyr;            // pyramid of box unions over the dynamic triangles (as LbvhWork's)
  uint32_t n_dyn;         // dynamic triangles
  uint32_t pyr_full;      // 1: an object's ranges need the pyramid above its low levels
  const ObjDev* objs;
  uint32_t n_obj;
  float* obj_aabb;        // [n_obj][6] world boxes (lo, hi)
  float* obj_xf_cur;      // [n_obj][12]
  uint32_t* obj_moved;    // [n_obj]
  // per internal node of the objects' upload-time topologies (nodes
  // [obj_node_first, obj_node_first + n_obj_nodes) of the scene): the
  // dynamic-record ranges of its two children (a subtree holds a contiguous
  // run of the leaf order), and its object
  const uint4* dspan;
  const uint32_t* dspan_obj;
  uint32_t obj_node_first, n_obj_nodes;
  // where the box of each child of those nodes goes in the four-wide form:
  // four-wide node * 4 + slot, kSlotNone for a child whose own children took
  // its place
  const uint2* wslot;
  // lights
  const LightDev* lights;
  float* light_xf_cur;    // [L][12]
  uint32_t* light_moved;  // [L]
  uint32_t n_lights;
  // materials
  const float* albedo;      // [M][3]
  const uint32_t* tri_mat;  // [T] by global id
  uint32_t n_tris_total;
  // store
  float4* pos;
  float4* energy;
  float* origin;
  uint32_t* info;
  uint32_t stride, n_paths, B;
  uint32_t verify_boxes;  // 1: a segment that reaches a moved object's box is invalid (no triangle test)
  uint32_t energy_test;   // Equation 2's E_N: PV_ENERGY_ALBEDO or PV_ENERGY_COSINE_RATIO
  const uint32_t* rec_mat;  // [T] material of each record of the leaf-order triangle array
  const uint32_t* gid_rec;  // [T] record of each global triangle id in the leaf-order triangle array
  float eps_end, eps_close, radius;
  uint32_t gpath_base;    // offset of this scene's paths in the work-queue id space
  uint32_t n_blocks;      // path blocks of the bound store
  uint32_t count_base;    // first entry of this scene's (row, block) photon counts
  uint32_t tile_base;     // first path tile (block of kBlock paths) of this scene
  uint32_t task_base;     // first entry of this scene's tile regions of verification tasks
  uint32_t* state;        // [2] first frame to come; a frame so far was read as WALK_SCALED
  // distribution maps (Section 3.1): grid {gu, gv, rings, sectors}, dm[0] = 0
  // when none; first cell of each light in the maps of all lights
  int32_t dm[4];
  uint32_t dm_off[PV_MAX_LIGHTS + 1];
};

// How walks read four-wide nodes.
enum WalkForm : int {
  WALK_PLAIN,   // no origins
  WALK_ORIGIN,  // an origin, the unit is the grid's step
  WALK_SCALED   // an origin and a unit of its own in every node; any ray origin
};

// SceneDev::wtop[2]: how far from plane_base a query may begin in this frame,
// along every axis.  With origins it is kRayReach steps, which no query needs to
// look at (nothing that the frame's rays begin on lies further out), or
// infinite: the nodes are read as WALK_SCALED.
constexpr float kReachNone = -1.0f;  // no query: without origins, and objects beyond FP16

// Grid of all nodes of an object placed by the rows m: its origin is the
// placed middle of the object's box.
template <typename M>
__device__ inline NodeGrid object_grid(const SceneDev& S, uint32_t o, M m) {
  const PV_GLOBAL ObjDev* ob = G(S.objs) + o;
  float at[3], half = 0.0f;
  for (int k = 0; k < 3; ++k) {
    const float a = m[4 * k], b = m[4 * k + 1], c = m[4 * k + 2];
    at[k] = a * ob->centre[0] + b * ob->centre[1] + c * ob->centre[2] + m[4 * k + 3];
    half = fmaxf(half, fabsf(a) * ob->half[0] + fabsf(b) * ob->half[1] + fabsf(c) * ob->half[2]);
  }
  return node_grid(S.qc, S.qm, S.qs, at, half, S.sroot == kRootNone);
}

// Writer of child boxes into four-wide slots.  Holds the grid and the array in
// registers: read from the descriptor at every write they would be loaded
// again after each store.  Each writer of an object's nodes finds their grid by
// itself (object_grid); the few top-level nodes have the grid's middle as their
// origin, and a unit of 2^e steps.
struct PlaneWriter {
  PV_GLOBAL Wide* wide;
  uint32_t shift;
  float slack0, slack;
  NodeGrid g;
  __device__ PlaneWriter(const SceneDev& S, int e) : wide(G(S.wide)), shift(S.wshift), slack0(S.qslack) {
    g.e = shift ? e : 0;
    g.s = g.e ? __builtin_ldexpf(S.qs, -g.e) : S.qs;
    for (int k = 0; k < 3; ++k) {
      g.c[k] = g.e ? S.qm[k] : S.qc[k];
      g.o[k] = shift ? (uint32_t)kOriginMid : 0u;
      g.f[k] = shift && !g.e ? kOriginMid : 0.0f;
    }
    slack = g.e ? kUnitSlack : slack0;
  }
  __device__ PlaneWriter(const SceneDev& S, uint32_t o, const float* xf) : PlaneWriter(S, 0) {
    if (shift) g = object_grid(S, o, G(xf) + 12 * o);
    slack = g.e ? kUnitSlack : slack0;
  }
  __device__ uint32_t low_byte(uint32_t k) const {
    return k == 0 ? g.o[0] : (k == 1 ? g.o[1] : (k == 2 ? g.o[2] : (uint32_t)g.e & 255u));
  }
  __device__ void put(uint32_t slot, float lx, float ly, float lz, float hx, float hy, float hz) const {
    PV_GLOBAL uint32_t* w = wide[slot >> 2].plane + 3 * (slot & 3u);
    w[0] = wide_planes(lx, hx, g.c[0], g.s, g.f[0], slack);
    w[1] = wide_planes(ly, hy, g.c[1], g.s, g.f[1], slack);
    w[2] = wide_planes(lz, hz, g.c[2], g.s, g.f[2], slack);
  }
  __device__ void none(uint32_t slot) const {
    PV_GLOBAL uint32_t* w = wide[slot >> 2].plane + 3 * (slot & 3u);
    w[0] = w[1] = w[2] = kPlanesNone;
    child(slot, 0);
  }
  // code: a walk's (wide_code)
  __device__ void child(uint32_t slot, int32_t code) const {
    wide[slot >> 2].child[slot & 3u] = code | (shift ? (int32_t)low_byte(slot & 3u) : 0);
  }
  // a node's origin and unit beside child codes that stay
  __device__ void put_origin(uint32_t node) const {
    if (!shift) return;
    PV_GLOBAL uint8_t* b = (PV_GLOBAL uint8_t*)wide[node].child;
    for (uint32_t k = 0; k < 4; ++k) b[4 * k] = (uint8_t)low_byte(k);
  }
};

// Device scratch of the per-frame object hierarchy rebuild (linear BVH over
// 30-bit Morton codes): sort keys (object << 30 | Morton code of the
// triangle's centroid) and values (dynamic triangle record) in two buffers,
// per-tile digit counts (and their scan for large sorts), parent links of the
// radix trees, a pyramid of box unions over the sorted triangles (level l
// entry k: positions [k 2^l, (k+1) 2^l)), each object's tree depth and
// centroid box.
struct LbvhWork {
  uint64_t* key[2];
  uint32_t* val[2];
  uint32_t* hist;        // [256][tiles] digit counts of a sort pass
  uint32_t* hoff;        // their exclusive scan (sorts of more than kFusedTiles tiles)
  uint32_t* htotal;      // [1]
  uint32_t* scan_tmp;    // scan_tmp_words(256 * tiles)
  int32_t* parent_leaf;  // [n_dyn] by sorted position: parent node (scene index)
  int32_t* parent_node;  // [nodes] parent node, -1 at an object's root
  float4* pyr;           // [2 * pyr_entries]: lo, hi of each pyramid entry
  uint32_t* odepth;      // [n_obj] deepest leaf of each rebuilt tree
  float* cbox;           // [n_obj][6] centroid bounds
  uint32_t n_dyn;        // dynamic triangles of the scene
  uint32_t first_node;   // scene node index of the first rebuilt node
};

// first entry of pyramid level l over n positions (level sizes n, ceil(n/2), ...)
__host__ __device__ inline uint32_t pyr_level(uint32_t n, int l) {
  uint32_t off = 0, m = n;
  for (int i = 0; i < l; ++i) {
    off += m;
    m = (m + 1) / 2;
  }
  return off;
}
// entries of the whole pyramid (levels down to a single entry)
__host__ __device__ inline uint32_t pyr_entries(uint32_t n) {
  uint32_t off = 0, m = n;
  while (m > 1) {
    off += m;
    m = (m + 1) / 2;
  }
  return off + m;
}

// Verification work lists (device scratch).  A task is one segment whose ray
// reaches a moved object's box: (global path id << 4) | segment.  Each path
// tile first writes its tasks into a region of its own; a gather makes them
// one list.  No atomics are needed:
// device-wide atomics on one word from thousands of blocks serialise.
struct VerifyWork {
  uint32_t* tmp;     // tasks by tile: region of a tile = kBlock * B entries
  uint32_t* tasks;   // compacted tasks
  uint32_t* tcount;  // [tiles] tasks of each tile
  uint32_t* toff;    // [tiles] their offsets in the compacted list
  uint32_t* total;   // [1] tasks in all
  uint32_t* first;   // [paths] first invalid segment found so far (global path id)
  uint32_t* part;    // statistics of each tile: [tiles][4]
  uint32_t* deal;    // [kDealWords] refill counters of the traversal, zero between launches
};

// Persistent kernels take their work lists a refill at a time from one of
// kDealGroups counters (a wave uses counter wave mod kDealGroups, each
// counter on its own 128-byte line); counter g deals the list's chunks
// g, g + kDealGroups, ... in order.
constexpr uint32_t kDealGroups = 64;
constexpr uint32_t kDealStride = 32;
constexpr uint32_t kDealWords = (kDealGroups + 1) * kDealStride;  // and a line for the groups that are done

// ---------------------------------------------------------------------------
// small vector helpers (FP32)
__device__ inline float3 f3(float x, float y, float z) { return make_float3(x, y, z); }
__device__ inline float3 sub(float3 a, float3 b) { return f3(a.x - b.x, a.y - b.y, a.z - b.z); }
__device__ inline float3 add(float3 a, float3 b) { return f3(a.x + b.x, a.y + b.y, a.z + b.z); }
__device__ inline float3 mul(float3 a, float s) { return f3(a.x * s, a.y * s, a.z * s); }
__device__ inline float dot(float3 a, float3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
__device__ inline float3 cross(float3 a, float3 b) {
  return f3(a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x);
}
__device__ inline float length(float3 a) { return sqrtf(dot(a, a)); }
__device__ inline float3 xyz(float4 v) { return f3(v.x, v.y, v.z); }
__device__ inline float comp(float3 v, int k) { return k == 0 ? v.x : (k == 1 ? v.y : v.z); }

// ---------------------------------------------------------------------------
// ray / segment query state of the triangle tests (Woop, Benthin, Wald 2013):
// the direction's largest component is the test's third axis, the other two
// follow in cyclic order, exchanged when that component is negative
struct Ray {
  float3 ro;          // origin, components in the test's axis order
  float3 d;           // direction (not necessarily unit)
  float tmin;         // lower end of the open interval of the parameter
  uint32_t axes;      // first axis of the cyclic order, + 4 when exchanged
  float sx, sy, sz;   // shear constants
};

__device__ inline Ray make_ray(float3 o, float3 d, float tmin) {
  Ray r;
  r.d = d;
  r.tmin = tmin;
  const float ax = fabsf(d.x), ay = fabsf(d.y), az = fabsf(d.z);
  const int kz = (ax > ay) ? (ax > az ? 0 : 2) : (ay > az ? 1 : 2);
  const float dz = kz == 0 ? d.x : (kz == 1 ? d.y : d.z);
  const bool sw = dz < 0.0f;
  r.axes = (kz == 2 ? 0u : (uint32_t)kz + 1u) + (sw ? 4u : 0u);
  auto order = [&](float3 v) {
    const float3 c = kz == 2 ? v : (kz == 0 ? f3(v.y, v.z, v.x) : f3(v.z, v.x, v.y));
    return f3(sw ? c.y : c.x, sw ? c.x : c.y, c.z);
  };
  r.ro = order(o);
  const float3 e = order(d);
  r.sx = e.x / e.z;
  r.sy = e.y / e.z;
  r.sz = 1.0f / e.z;
  return r;
}

// the origin in world axis order
__device__ inline float3 ray_origin(const Ray& r) {
  const bool sw = (r.axes & 4u) != 0;
  const float x = sw ? r.ro.y : r.ro.x, y = sw ? r.ro.x : r.ro.y, z = r.ro.z;
  const uint32_t k = r.axes & 3u;
  return k == 0u ? f3(x, y, z) : (k == 1u ? f3(z, x, y) : f3(y, z, x));
}

// what box tests read of a query: slab parameters are fma(bound, inv, oi)
struct BoxRay {
  float3 inv;         // 1 / direction
  float3 oi;          // -origin / direction
  float tmin, tmax;
};

// components kept at least 'tiny' from zero, sign kept
__device__ inline float3 off_zero(float3 d) {
  const float tiny = 1e-30f;
  return f3(copysignf(fmaxf(fabsf(d.x), tiny), d.x), copysignf(fmaxf(fabsf(d.y), tiny), d.y),
            copysignf(fmaxf(fabsf(d.z), tiny), d.z));
}

// 1 / d from the hardware reciprocal (1 ulp): moves a slab parameter by about
// 1e-7 of itself, far inside the 1e-6 padding of every stored box
__device__ inline float3 rcp3(float3 d) {
  d = off_zero(d);
  return f3(__builtin_amdgcn_rcpf(d.x), __builtin_amdgcn_rcpf(d.y), __builtin_amdgcn_rcpf(d.z));
}

// Slab test of one box against the ray's current [tmin, tmax]; returns the
// entry parameter or +inf.  A slab parameter is one fused multiply-add,
// bound * (1/d) - o/d; its error (relative 2^-24 of o/d, i.e. about 6e-8 of
// the origin's coordinates in distance) stays far inside the 1e-6 padding of
// every stored box, so the test remains conservative.
__device__ inline float box_entry(float lx, float ly, float lz, float hx, float hy, float hz, const BoxRay& r,
                                  float tmax) {
  float tx0 = fmaf(lx, r.inv.x, r.oi.x), tx1 = fmaf(hx, r.inv.x, r.oi.x);
  float ty0 = fmaf(ly, r.inv.y, r.oi.y), ty1 = fmaf(hy, r.inv.y, r.oi.y);
  float tz0 = fmaf(lz, r.inv.z, r.oi.z), tz1 = fmaf(hz, r.inv.z, r.oi.z);
  float t0 = fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fmaxf(fminf(tz0, tz1), r.tmin));
  float t1 = fminf(fminf(fmaxf(tx0, tx1), fmaxf(ty0, ty1)), fminf(fmaxf(tz0, tz1), tmax));
  return t0 <= t1 ? t0 : __builtin_inff();
}

// entry parameter of a box regardless of the query's interval
__device__ inline float slab_entry(float lx, float ly, float lz, float hx, float hy, float hz, const BoxRay& r) {
  const float tx0 = fmaf(lx, r.inv.x, r.oi.x), tx1 = fmaf(hx, r.inv.x, r.oi.x);
  const float ty0 = fmaf(ly, r.inv.y, r.oi.y), ty1 = fmaf(hy, r.inv.y, r.oi.y);
  const float tz0 = fmaf(lz, r.inv.z, r.oi.z), tz1 = fmaf(hz, r.inv.z, r.oi.z);
  return fmaxf(fmaxf(fminf(tx0, tx1), fminf(ty0, ty1)), fminf(tz0, tz1));
}

// Watertight ray/triangle test (Woop, Benthin, Wald, JCGT 2013), two-sided.
// Returns true with *t when the triangle is crossed at a parameter strictly
// inside (tmin, tmax).  An edge function compiles to a product and a fused
// multiply-add (the _rn intrinsics do not keep the compiler from contracting), so
// triangles sharing an edge see opposite values up to the product's rounding, and
// exactly so only where the edge is read in the same order; results hang on these
// roundings.  Written without early exits (the caller's loop stays one predicated block);
// only an exactly zero edge function takes the double-precision branch.
// near_tb (may be null): set when the triangle is crossed past tmin within
// 2.5e-7 (relative) of tmax.
__device__ inline bool tri_hit(const Ray& r, const PV_GLOBAL Tri* __restrict__ tri, float tmax, float* t_out,
                               bool* near_tb) {
  struct V {
    float x, y, z;
  };
  const PV_GLOBAL float* base = &tri->v[0][0] + (r.axes & 3u);
  const V a = *(const PV_GLOBAL V*)base, b = *(const PV_GLOBAL V*)(base + 5), c = *(const PV_GLOBAL V*)(base + 10);
  const bool sw = (r.axes & 4u) != 0;
  const float Akz = a.z - r.ro.z, Bkz = b.z - r.ro.z, Ckz = c.z - r.ro.z;
  const float Ax = ((sw ? a.y : a.x) - r.ro.x) - r.sx * Akz, Ay = ((sw ? a.x : a.y) - r.ro.y) - r.sy * Akz;
  const float Bx = ((sw ? b.y : b.x) - r.ro.x) - r.sx * Bkz, By = ((sw ? b.x : b.y) - r.ro.y) - r.sy * Bkz;
  const float Cx = ((sw ? c.y : c.x) - r.ro.x) - r.sx * Ckz, Cy = ((sw ? c.x : c.y) - r.ro.y) - r.sy * Ckz;
  float U = __fsub_rn(__fmul_rn(Cx, By), __fmul_rn(Cy, Bx));
  float V = __fsub_rn(__fmul_rn(Ax, Cy), __fmul_rn(Ay, Cx));
  float W = __fsub_rn(__fmul_rn(Bx, Ay), __fmul_rn(By, Ax));
  if (U == 0.0f || V == 0.0f || W == 0.0f) {
    // exact-zero edge function: re-evaluate in double precision (same paper)
    U = (float)((double)Cx * (double)By - (double)Cy * (double)Bx);
    V = (float)((double)Ax * (double)Cy - (double)Ay * (double)Cx);
    W = (float)((double)Bx * (double)Ay - (double)By * (double)Ax);
  }
  const bool mixed = (U < 0.0f || V < 0.0f || W < 0.0f) && (U > 0.0f || V > 0.0f || W > 0.0f);
  float det = U + V + W;
  float Az = r.sz * Akz, Bz = r.sz * Bkz, Cz = r.sz * Ckz;
  float T = U * Az + V * Bz + W * Cz;
  const bool neg = det < 0.0f;
  T = neg ? -T : T;
  det = neg ? -det : det;
  const bool ok = !mixed && det != 0.0f && T > r.tmin * det && T < tmax * det;
  *t_out = T / det;
  if (near_tb)
    *near_tb = !mixed && det != 0.0f && T > r.tmin * det && fabsf(fmaf(-tmax, det, T)) <= 2.5e-7f * T;
  return ok;
}

// ---------------------------------------------------------------------------
// traversal stack column of one lane: entry i at col[i * kBlock] (a column per
// lane of a kBlock-wide LDS array, conflict-free)
using StackCol = PV_LDS int32_t*;

struct Hit {
  float t;       // ray parameter of the closest crossing (tmax when none)
  uint32_t gid;  // its global triangle id, kHitNone when none
  uint32_t rec;  // its record in the scene's triangle array
};
constexpr uint32_t kRecNone = 0xFFFFFFFFu;

// Depth-first walk of the scene hierarchy from a root (near child first), in
// resumable form for persistent kernels.  any = stop at the first crossing
// inside the ray's open interval; otherwise the closest crossing.  The state
// of one lane's query survives between calls, and a call returns as soon as
// this lane's walk is finished or fewer than 'min_active' lanes of the wave
// are still walking, so that finished lanes can take new work instead of
// idling until the longest walk of the wave ends (Aila and Laine 2009,
// dynamic ray fetch).
//
// The inner loop over internal nodes has no branch besides its exit: each
// further child is always written one slot above the top of the stack and the
// stack pointer moves past it when that child is entered; when none is, the
// top entry, read ahead, becomes the next node.  A sentinel at the bottom ends
// the walk.
struct Walk {
  int32_t cur;    // next node or leaf; kRootNone once the stack is exhausted
  int32_t leaf;   // a reached leaf whose test is postponed, 0 when none
  int sp;         // stack entries in use
  float tb;       // closest crossing so far (the ray's tmax initially)
  uint32_t rec;   // its record in the scene's triangle array, kRecNone when none
  bool redo;      // the binary walk must answer: near tie, or out of stack
};

__device__ inline bool is_leaf(int32_t c) { return (uint32_t)c > 0x80000000u; }  // c < 0, c != kRootNone

__device__ inline bool walk_done(const Walk& w) { return w.cur == kRootNone && w.leaf == 0; }

__device__ inline void walk_start(Walk& w, int32_t root, float tmax, StackCol col) {
  col[0] = kRootNone;
  w.sp = 1;
  w.cur = root;
  w.leaf = 0;
  w.tb = tmax;
  w.rec = kRecNone;
  w.redo = false;
}

// leaves a query to walk_exact
__device__ inline void walk_leave(Walk& w) {
  w.cur = kRootNone;
  w.leaf = 0;
  w.redo = true;
}

// Parameters of a query's box tests: 1 / direction and (centre - origin) /
// direction in the planes' grid, and per axis 16 where the direction is
// negative (the upper plane is then the nearer one).  They give a crossing's
// parameter t as (t - tmin) kTScale, so that the instructions' output clamp to
// [0, 1] is the interval's lower end at no cost; parameters past 1 / kTScale
// clamp too, which only enters a box the query has left behind.
constexpr float kTScale = 1.0f / 1099511627776.0f;  // 2^-40

constexpr float kWiden = 9.5367432e-7f;  // 2^-20, of |qm - o| / d with WALK_SCALED

struct Slab {
  float3 inv, oi;
  uint32_t rx, ry, rz;
};

__device__ inline Slab make_slab(float3 inv, float3 oi, float scale, float tmin) {
  Slab q;
  q.inv = mul(inv, scale * kTScale);
  q.oi = f3((oi.x - tmin) * kTScale, (oi.y - tmin) * kTScale, (oi.z - tmin) * kTScale);
  q.rx = inv.x < 0.0f ? 16u : 0u;
  q.ry = inv.y < 0.0f ? 16u : 0u;
  q.rz = inv.z < 0.0f ? 16u : 0u;
  return q;
}

// what a scene's planes count from: the grid's corner, or with WALK_SCALED its
// middle (the same without origins)
template <bool kScaled>
__device__ inline float3 plane_base(const SceneDev& S) {
  const float* q = kScaled ? S.qm : S.qc;
  return f3(q[0], q[1], q[2]);
}

// a world-space query from o against the scene's four-wide nodes; c: plane_base - o
__device__ inline Slab world_slab(const SceneDev& S, float3 c, float3 inv, float tmin) {
  return make_slab(inv, f3(c.x * inv.x, c.y * inv.y, c.z * inv.z), S.qinv, tmin);
}

__device__ inline float reach3(float3 v) { return fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fabsf(v.z)); }
__device__ inline float frame_reach(const SceneDev& S) { return __int_as_float(G(S.wtop)[2]); }

// whether a query without origins is left to walk_exact; c: plane_base - o
__device__ inline bool walk_far(const SceneDev& S, float3 c) { return !S.wshift && !(reach3(c) <= frame_reach(S)); }

// a condition as the wave's mask, and a mask's bit of this lane: conditions
// combined as masks are scalar work beside the vector pipeline
__device__ __forceinline__ uint64_t wave_mask(bool c) { return __builtin_amdgcn_ballot_w64(c); }
__device__ __forceinline__ bool lane_bit(uint64_t m) {
#if defined(__HIP_DEVICE_COMPILE__)
  return __builtin_amdgcn_inverse_ballot_w64(m);
#else
  return m != 0;
#endif
}

typedef _Float16 half2v __attribute__((ext_vector_type(2)));

// both parameters of an axis' planes, nearer one first: a rotation by the
// axis' sign instead of a minimum and a maximum, and mixed-precision fused
// multiply-adds that read the FP16 planes in place
__device__ __forceinline__ void plane_pair(uint32_t w, uint32_t rot, float inv, float on, float of, float* n, float* f) {
  const half2v h = __builtin_bit_cast(half2v, __builtin_amdgcn_alignbit(w, w, rot));
  *n = __builtin_fmaf((float)h.x, inv, on);
  *f = __builtin_fmaf((float)h.y, inv, of);
}

// Speculative traversal (Aila and Laine 2009): a lane that reaches a leaf
// while holding none keeps it pending and continues with the next stack
// entry, until most lanes still walking hold a leaf; then the wave tests
// leaves together.
//
// Nodes are four wide with FP16 planes: one 64-byte line, four 16-byte loads,
// per visit, as the binary FP32 node took, and about a fifth of the visits (22
// against 109 for a ray of the 3M-path, 380k-triangle interior), so a shorter
// chain of dependent loads and fewer of them.  Bound by vector issue: about
// 90 instructions a visit.  Measured there, one MI355X, four-wide against
// binary: full trace 4.85 against 5.66 ms, partial re-trace 1.98 against 2.30
// ms, verification traversal 178 against 224 us; with the clamp as the lower
// end (four instructions a visit) the full trace went from 4.11 to 4.03 ms, and
// with the nodes' origins (seven more instructions a visit, but 19.6 visits and
// 3.1 triangles a ray instead of 21.9 and 4.6) to 3.55 ms.  The origin as eight
// bytes of an array beside the nodes gave the same visits and 4.39 ms: its load,
// a fifth per visit, cost more than they saved.
//
// Boxes are tested with the slab parameters q and triangles with the ray r
// itself: a walk through a rigid object's hierarchy in its own object space
// passes the object-space parameters for the boxes, with the same parameter
// interval, while triangles stay in world space.
//
// w.redo asks the caller to take walk_exact's answer instead: set when a walk
// would leave more entries than 'limit' (the top's address there) allows, which
// leaves no crossing, and, with kTies, when the closest crossing and one of
// another leaf lie within 2.5e-7 of each other, twice the rounding that lets the
// order of their tests decide.
//
// With WALK_SCALED a node has its own unit, and the slabs are widened by 2^-20
// of |qm - o| / d, twice what the ray's part of their roundings is: for ray
// origins anywhere.
template <bool kTies, int kForm>
__device__ inline void walk_run(const PV_GLOBAL Wide* __restrict__ nodes, const PV_GLOBAL Tri* __restrict__ tris,
                                const Ray& r, const Slab& q, bool any, StackCol col, StackCol limit, Walk& w,
                                int min_active) {
  int32_t cur = w.cur, leaf = w.leaf;
  // top: the stack's top entry (entry sp - 1).  Once the sentinel itself is
  // taken top points one entry below the column's first, which every launch
  // allocates and nothing uses.
  StackCol top = col + (w.sp - 1) * kBlock;
  float tb = w.tb;
  uint32_t rec = w.rec;
  bool redo = w.redo;
  constexpr bool kOrigin = kForm != WALK_PLAIN, kScaled = kForm == WALK_SCALED;
  while (true) {
    const float ts = __builtin_canonicalizef((tb - r.tmin) * kTScale);  // tb as a slab parameter
    const int alive = __popcll(__ballot(1));
    while (cur >= 0) {
      const int32_t below = top[0], below2 = top[-kBlock];
      // node records are addressed by a 32-bit byte offset (arrays < 4 GiB); a
      // code's low byte is not its own
      const PV_GLOBAL uint4* np = (const PV_GLOBAL uint4*)((const PV_GLOBAL char*)nodes + (kOrigin ? ((uint32_t)cur >> kOriginShift) << 6 : (uint32_t)cur << 6));
      const uint4 na = np[0], nb = np[1], nc = np[2], nd = np[3];
      const uint32_t pl[12] = {na.x, na.y, na.z, na.w, nb.x, nb.y, nb.z, nb.w, nc.x, nc.y, nc.z, nc.w};
      int32_t c[4] = {(int32_t)nd.x, (int32_t)nd.y, (int32_t)nd.z, (int32_t)nd.w};
      float e[4];
      uint64_t h[4];  // entered children, as wave masks
      float3 on = q.oi, of;
      float te = ts;
      if (kScaled) {
        // in the node's unit: every parameter times 2^-x
        const int x = -(int)(int8_t)(nd.w & 255u);
        const float3 og = f3((float)(nd.x & 255u) - kOriginMid, (float)(nd.y & 255u) - kOriginMid,
                             (float)(nd.z & 255u) - kOriginMid);
        auto wide = [&](float oi, float w, float g, float inv) {
          const float u = __builtin_ldexpf(oi, x);
          return __builtin_fmaf(g, inv, __builtin_fmaf(w, fabsf(u), u));
        };
        of = f3(wide(on.x, kWiden, og.x, q.inv.x), wide(on.y, kWiden, og.y, q.inv.y), wide(on.z, kWiden, og.z, q.inv.z));
        on = f3(wide(on.x, -kWiden, og.x, q.inv.x), wide(on.y, -kWiden, og.y, q.inv.y), wide(on.z, -kWiden, og.z, q.inv.z));
        te = __builtin_canonicalizef(__builtin_ldexpf(ts, x));
      } else {
        if (kOrigin) {
          on.x = __builtin_fmaf((float)(nd.x & 255u), q.inv.x, on.x);
          on.y = __builtin_fmaf((float)(nd.y & 255u), q.inv.y, on.y);
          on.z = __builtin_fmaf((float)(nd.z & 255u), q.inv.z, on.z);
        }
        of = on;
      }
#pragma unroll
      for (int k = 0; k < 4; ++k) {
        float nx, ny, nz, fx, fy, fz;
        plane_pair(pl[3 * k], q.rx, q.inv.x, on.x, of.x, &nx, &fx);
        plane_pair(pl[3 * k + 1], q.ry, q.inv.y, on.y, of.y, &ny, &fy);
        plane_pair(pl[3 * k + 2], q.rz, q.inv.z, on.z, of.z, &nz, &fz);
        e[k] = __builtin_amdgcn_fmed3f(fmaxf(fmaxf(nx, ny), nz), 0.0f, 1.0f);
        const float ex = fminf(fminf(fx, fy), fz);
        // the slab interval meets [tmin, tb]
        h[k] = wave_mask(e[k] <= fminf(ex, te));
      }
      // nearest entered child first, the others nearly in order (a child not
      // entered comes last of its pair); exchanges of the masks are scalar work
      auto order = [&](int i, int j) {
        const uint64_t sw = h[j] & (~h[i] | wave_mask(e[j] < e[i]));
        const bool x = lane_bit(sw);
        const int32_t u = x ? c[j] : c[i], v = x ? c[i] : c[j];
        const uint64_t hu = h[i] | h[j], hv = h[i] & h[j];
        e[i] = x ? e[j] : e[i];
        c[i] = u, c[j] = v, h[i] = hu, h[j] = hv;
      };
      order(0, 1);
      order(2, 3);
      order(0, 2);
      top[kBlock] = c[3];
      const StackCol t0 = top - kBlock;
      top = lane_bit(h[3]) ? top + kBlock : top;
      top[kBlock] = c[2];
      top = lane_bit(h[2]) ? top + kBlock : top;
      top[kBlock] = c[1];
      top = lane_bit(h[1]) ? top + kBlock : top;
      top = lane_bit(h[0]) ? top : t0;
      // the entry that the next pop takes, from registers
      const int32_t pushed = lane_bit(h[1]) ? c[1] : (lane_bit(h[2]) ? c[2] : c[3]);
      int32_t next = lane_bit(h[0]) ? below : below2;
      next = lane_bit(h[1] | h[2] | h[3]) ? pushed : next;
      cur = lane_bit(h[0]) ? c[0] : below;
      if (top > limit) {  // rare: no room for another full node
        redo = true;
        rec = kRecNone;
        cur = kRootNone;
        leaf = 0;
        break;
      }
      // postpone a reached leaf and go on with the next stack entry (once the
      // sentinel itself was taken, cur is kRootNone and nothing is postponed)
      const bool post = leaf == 0 && is_leaf(cur);
      leaf = post ? cur : leaf;
      cur = post ? next : cur;
      top = post ? top - kBlock : top;
      // once at most a quarter of the lanes that began this descent are still
      // here without a leaf, the wave tests leaves: full trace 3.49 ms (3.55
      // with a third of those still here, 3.56 with half of all), 3M-path
      // partial re-trace frame 2.04 ms (2.07, 2.09)
      if (4 * __popcll(__ballot(leaf == 0)) <= alive) break;
    }
    if (leaf == 0 && is_leaf(cur)) {
      leaf = cur;
      cur = top[0];
      top -= kBlock;
    }
    bool found = false;
    while (leaf != 0) {
      const int32_t code = leaf >> (kOrigin ? kOriginShift : 0u);
      const uint32_t f = leaf_first(code), n = leaf_count(code);
      for (uint32_t i = f; i < f + n; ++i) {
        float t;
        bool near_tb = false;
        const bool hit = tri_hit(r, tris + i, tb, &t, kTies ? &near_tb : nullptr);
        // both walks test one leaf's triangles in the same order; a clearly
        // closer crossing ends a tie
        if (kTies) redo = (near_tb && rec - f >= n) || (redo && !(hit && !near_tb));
        tb = hit ? t : tb;
        rec = hit ? i : rec;
        found |= hit;
      }
      // the current entry may itself be a leaf: test it next
      const bool again = is_leaf(cur) && !(found && any);
      leaf = again ? cur : 0;
      if (again) {
        cur = top[0];
        top -= kBlock;
      }
    }
    if (found && any) cur = kRootNone;
    if (cur == kRootNone) break;
    if (__popcll(__ballot(1)) < min_active) break;
  }
  w.cur = cur;
  w.leaf = leaf;
  w.sp = (int)(top - col) / kBlock + 1;
  w.tb = tb;
  w.rec = rec;
  w.redo = redo;
}

// walk_run in the scene's form of nodes
template <bool kTies, bool kScaled>
__device__ inline void walk_scene(const SceneDev& S, const Ray& r, const Slab& q, bool any, StackCol col, StackCol limit,
                                  Walk& w, int min_active) {
  if (S.wshift)
    walk_run<kTies, kScaled ? WALK_SCALED : WALK_ORIGIN>(G(S.wide), G(S.tris), r, q, any, col, limit, w, min_active);
  else
    walk_run<kTies, WALK_PLAIN>(G(S.wide), G(S.tris), r, q, any, col, limit, w, min_active);
}

// The answer to a world-space query by the order that settles near ties: the
// binary FP32 hierarchy depth first, the child entered first (the first child
// when both at once) before the other, a later crossing taken only when
// strictly closer.  Two crossings within rounding of each other (an edge of a
// wall on a floor) are otherwise decided by the order of their tests, which
// the four-wide walk's looser boxes change.  any: stop at the first crossing.
//
// A tie is settled among the crossings near the one that w holds: boxes that end
// before or begin after it are left out, which changes neither the order of the
// others nor what is taken among them, and a descent to a point is left of the
// walk.  Two-sided assets hold every triangle twice: a full trace of 500k paths
// through a room of 50k such pairs took 2.29 ms with every tie walked again in
// full and takes 0.83 (0.72 without the copies; 1.10 with the binary walk alone).
__device__ inline void walk_exact(const PV_GLOBAL Node* __restrict__ nodes, const PV_GLOBAL Tri* __restrict__ tris,
                                  const Ray& r, float tmax, int32_t root, bool any, StackCol col, Walk& w) {
  const float3 o = ray_origin(r), d = r.d;
  BoxRay q;
  const float tiny = 1e-30f;
  q.inv = f3(1.0f / (fabsf(d.x) > tiny ? d.x : copysignf(tiny, d.x)),
             1.0f / (fabsf(d.y) > tiny ? d.y : copysignf(tiny, d.y)),
             1.0f / (fabsf(d.z) > tiny ? d.z : copysignf(tiny, d.z)));
  q.oi = f3(-(o.x * q.inv.x), -(o.y * q.inv.y), -(o.z * q.inv.z));
  const bool tie = w.rec != kRecNone;
  constexpr float kNear = 2e-6f;
  q.tmin = tie ? fmaxf(r.tmin, w.tb * (1.0f - kNear)) : r.tmin;
  q.tmax = tie ? fminf(tmax, w.tb * (1.0f + kNear)) : tmax;
  StackCol top = col;
  top[0] = kRootNone;
  int32_t cur = root;
  float tb = q.tmax;
  uint32_t rec = kRecNone;
  while (cur != kRootNone) {
    if (cur >= 0) {
      const Node nd = *(const PV_GLOBAL Node*)((const PV_GLOBAL char*)nodes + ((uint32_t)cur << 6));
      const float e0 = box_entry(nd.a.x, nd.a.y, nd.a.z, nd.a.w, nd.b.x, nd.b.y, q, tb);
      const float e1 = box_entry(nd.b.z, nd.b.w, nd.c.x, nd.c.y, nd.c.z, nd.c.w, q, tb);
      const bool h0 = e0 != __builtin_inff(), h1 = e1 != __builtin_inff();
      const bool near0 = h0 && (!h1 || slab_entry(nd.a.x, nd.a.y, nd.a.z, nd.a.w, nd.b.x, nd.b.y, q) <=
                                           slab_entry(nd.b.z, nd.b.w, nd.c.x, nd.c.y, nd.c.z, nd.c.w, q));
      if (h0 && h1) {
        top += kBlock;
        top[0] = near0 ? nd.d.y : nd.d.x;
      }
      cur = near0 ? nd.d.x : nd.d.y;
      if (h0 || h1) continue;
    } else {
      const uint32_t f = leaf_first(cur), n = leaf_count(cur);
      for (uint32_t i = f; i < f + n; ++i) {
        float t;
        if (tri_hit(r, tris + i, tb, &t, nullptr)) {
          tb = t;
          rec = i;
        }
      }
      if (any && rec != kRecNone) break;
    }
    cur = top[0];
    top -= kBlock;
  }
  if (tie && rec == kRecNone) return;
  w.tb = tb;
  w.rec = rec;
}

// ---------------------------------------------------------------------------
// Philox4x64-10 (Salmon, Moraes, Dror, Shaw, SC'11) from its published
// definition; uniforms are the top 24 bits of each word times 2^-24.
// The 128-bit products are formed from four 32 x 32 + 64 bit multiply-adds.
__device__ inline void mul64(uint64_t m, uint64_t c, uint64_t* lo, uint64_t* hi) {
  const uint32_t ml = (uint32_t)m, mh = (uint32_t)(m >> 32), cl = (uint32_t)c, ch = (uint32_t)(c >> 32);
  const uint64_t p0 = (uint64_t)ml * cl;
  const uint64_t p1 = (uint64_t)mh * cl + (p0 >> 32);
  const uint64_t p2 = (uint64_t)ml * ch + (uint32_t)p1;
  *hi = ((uint64_t)mh * ch + (p1 >> 32)) + (p2 >> 32);
  *lo = (p2 << 32) | (uint32_t)p0;
}

// a ^ b ^ c in one instruction per word
__device__ inline uint64_t xor3(uint64_t a, uint64_t b, uint64_t c) {
  const uint32_t l = (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)a, (uint32_t)b, (uint32_t)c, 0x96);
  const uint32_t h = (uint32_t)__builtin_amdgcn_bitop3_b32((uint32_t)(a >> 32), (uint32_t)(b >> 32),
                                                          (uint32_t)(c >> 32), 0x96);
  return ((uint64_t)h << 32) | l;
}

__device__ inline void philox4x64(uint64_t c[4], uint64_t k0, uint64_t k1) {
  const uint64_t M0 = 0xD2E7470EE14C6C93ull, M1 = 0xCA5A826395121157ull;
  const uint64_t W0 = 0x9E3779B97F4A7C15ull, W1 = 0xBB67AE8584CAA73Bull;
#pragma unroll
  for (int r = 0; r < 10; ++r) {
    uint64_t lo0, hi0, lo1, hi1;
    mul64(M0, c[0], &lo0, &hi0);
    mul64(M1, c[2], &lo1, &hi1);
    const uint64_t n0 = xor3(hi1, c[1], k0), n2 = xor3(hi0, c[3], k1);
    c[0] = n0;
    c[1] = lo1;
    c[2] = n2;
    c[3] = lo0;
    k0 += W0;
    k1 += W1;
  }
}

__device__ inline void draw4(uint64_t seed, uint64_t path, uint64_t frame, uint64_t vertex, uint64_t tag,
                             float u[4]) {
  uint64_t c[4] = {path, frame, vertex, tag};
  // the round keys follow from the uniform seed by scalar additions; kept from
  // being computed ahead of a caller's loop, where they would spill
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile("" : "+s"(seed));
#endif
  philox4x64(c, seed, 0);
#pragma unroll
  for (int i = 0; i < 4; ++i) u[i] = (float)(uint32_t)(c[i] >> 40) * (1.0f / 16777216.0f);
}

// Shirley-Chiu concentric map to the unit disk, lifted to the cosine-weighted
// hemisphere (Malley): local (x, y, z).
__device__ inline float3 cosine_local(float u1, float u2) {
  const float a = 2.0f * u1 - 1.0f, b = 2.0f * u2 - 1.0f;
  const float PI4 = 0.78539816339744830962f;
  const bool zero = a == 0.0f && b == 0.0f, wide = fabsf(a) > fabsf(b);
  const float q = (wide ? b : a) / (wide ? a : b);  // one division for both wedges
  const float r = zero ? 0.0f : (wide ? a : b);
  const float phi = zero ? 0.0f : (wide ? PI4 * q : 2.0f * PI4 - PI4 * q);
  float sn, cs;
  sincosf(phi, &sn, &cs);
  const float x = r * cs, y = r * sn;
  // height above the disk point at radius |r|; (1-|r|) is exact for |r| >= 1/2
  float ar = fabsf(r);
  float z2 = (1.0f - ar) * (1.0f + ar);
  return f3(x, y, z2 > 0.0f ? sqrtf(z2) : 0.0f);
}

// ---------------------------------------------------------------------------
// Distribution maps (Section 3.1).  A light's emission is partitioned into
// cells: for a rectangle, a gu x gv grid over its local (u, v) times a grid of
// directions; for a point light, the directions only.  Directions are cut on
// the unit disk of their local (x, y) components (cosine-weighted emission is
// uniform there): 'rings' rings of equal area (equal steps of x^2 + y^2) and
// 'sectors' sectors of equal angle, so that every cell is equally likely.
// Cell index ((iu * gv + iv) * rings + ring) * sectors + sector.

__host__ __device__ inline bool dm_point(const float half[2]) { return half[0] == 0.0f && half[1] == 0.0f; }

__host__ __device__ inline uint32_t dm_cells(const float half[2], int32_t kind, const int32_t dm[4]) {
  if (kind == PV_LIGHT_CAMERA) return (uint32_t)dm[0] * (uint32_t)dm[1];  // pixel grid of the near plane
  return (uint32_t)(dm_point(half) ? 1 : dm[0] * dm[1]) * (uint32_t)dm[2] * (uint32_t)dm[3];
}

// squared radius of a light's direction disk: 1, or sin^2 of a spot's cone
__device__ inline float dm_disk2(int32_t kind, const float param[2]) {
  return kind == PV_LIGHT_SPOT ? (1.0f - param[0]) * (1.0f + param[0]) : 1.0f;
}

// DM_T: a light's paths spread evenly over its cells, the first N mod C
// cells one more
__host__ __device__ inline uint32_t dm_target(uint32_t n_paths, uint32_t cells, uint32_t c) {
  return n_paths / cells + (c < n_paths % cells ? 1u : 0u);
}

constexpr float kPiF = 3.14159265358979323846f;

// The cell of a light sample (origin x0 on the light, unit direction w), or
// -1 when the parametrisation has no value for it (origin off the rectangle,
// direction not on the emitting side).  xf: the light's 3x4 transform
// (columns eu, ev, n, centre).
__device__ inline int32_t dm_cell(const float* xf, const LightDev& lt, const int32_t dm[4], float3 x0, float3 w) {
  const float* half = lt.half;
  const float3 eu = f3(xf[0], xf[4], xf[8]), ev = f3(xf[1], xf[5], xf[9]);
  const float3 c = f3(xf[3], xf[7], xf[11]);
  float3 n = f3(xf[2], xf[6], xf[10]);
  n = mul(n, 1.0f / length(n));
  if (lt.kind == PV_LIGHT_CAMERA) {
    const float z = dot(w, n);
    if (!(z > 0.0f)) return -1;
    const float fu = (dot(w, eu) / z + lt.param[0]) / (2.0f * lt.param[0]) * (float)dm[0];
    const float fv = (dot(w, ev) / z + lt.param[1]) / (2.0f * lt.param[1]) * (float)dm[1];
    if (!(fu >= 0.0f && fu <= (float)dm[0] && fv >= 0.0f && fv <= (float)dm[1])) return -1;
    return min((int32_t)floorf(fu), dm[0] - 1) * dm[1] + min((int32_t)floorf(fv), dm[1] - 1);
  }
  const float s2 = dm_disk2(lt.kind, lt.param);
  const bool point = dm_point(half);
  const int32_t gu = point ? 1 : dm[0], gv = point ? 1 : dm[1], nr = dm[2], ns = dm[3];
  int32_t iu = 0, iv = 0;
  if (!point) {
    const float3 r = sub(x0, c);
    const float u = dot(r, eu), v = dot(r, ev);
    const float fu = (u + half[0]) / (2.0f * half[0]) * (float)gu;
    const float fv = (v + half[1]) / (2.0f * half[1]) * (float)gv;
    if (!(fu >= 0.0f && fu <= (float)gu && fv >= 0.0f && fv <= (float)gv)) return -1;
    iu = min((int32_t)floorf(fu), gu - 1);
    iv = min((int32_t)floorf(fv), gv - 1);
  }
  const float x = dot(w, eu), y = dot(w, ev), z = dot(w, n);
  if (!(z > 0.0f)) return -1;
  const float rho2 = x * x + y * y;
  const float fr = rho2 / s2 * (float)nr;
  if (lt.kind == PV_LIGHT_SPOT && !(fr <= (float)nr)) return -1;  // outside the cone
  const int32_t ring = min((int32_t)floorf(fr), nr - 1);
  const float phi = atan2f(y, x);  // [-pi, pi]
  const float fs = (phi + kPiF) / (2.0f * kPiF) * (float)ns;
  const int32_t sector = max(0, min((int32_t)floorf(fs), ns - 1));
  return ((iu * gv + iv) * nr + ring) * ns + sector;
}

// A new light sample inside cell 'cell' (Section 3.1, filling DM_C:
// sampling restricted to the cell): position uniform in the cell's part of
// the rectangle, disk point uniform in the cell's ring (in x^2 + y^2) and
// sector (in angle), lifted to the hemisphere; u: one Philox draw (tag 0).
__device__ inline void dm_sample(const float* xf, const LightDev& lt, const int32_t dm[4], uint32_t cell,
                                 const float u[4], float3* x0, float3* w) {
  const float* half = lt.half;
  const float3 eu = f3(xf[0], xf[4], xf[8]), ev = f3(xf[1], xf[5], xf[9]);
  const float3 c = f3(xf[3], xf[7], xf[11]);
  float3 n = f3(xf[2], xf[6], xf[10]);
  n = mul(n, 1.0f / length(n));
  if (lt.kind == PV_LIGHT_CAMERA) {
    // uniform in the pixel's part of the near plane
    const uint32_t iu = cell / (uint32_t)dm[1], iv = cell % (uint32_t)dm[1];
    const float x = -lt.param[0] + ((float)iu + u[0]) * (2.0f * lt.param[0] / (float)dm[0]);
    const float y = -lt.param[1] + ((float)iv + u[1]) * (2.0f * lt.param[1] / (float)dm[1]);
    *x0 = c;
    *w = mul(add(add(mul(eu, x), mul(ev, y)), n), 1.0f / sqrtf(x * x + y * y + 1.0f));
    return;
  }
  const float s2 = dm_disk2(lt.kind, lt.param);
  const bool point = dm_point(half);
  const uint32_t gu = point ? 1u : (uint32_t)dm[0], gv = point ? 1u : (uint32_t)dm[1];
  const uint32_t nr = (uint32_t)dm[2], ns = (uint32_t)dm[3];
  const uint32_t sector = cell % ns, ring = (cell / ns) % nr, pc = cell / (ns * nr);
  const uint32_t iv = pc % gv, iu = pc / gv;
  if (point) {
    *x0 = c;
  } else {
    const float a = -half[0] + ((float)iu + u[0]) * (2.0f * half[0] / (float)gu);
    const float b = -half[1] + ((float)iv + u[1]) * (2.0f * half[1] / (float)gv);
    *x0 = add(c, add(mul(eu, a), mul(ev, b)));
  }
  const float rho2 = ((float)ring + u[2]) / (float)nr * s2, rho = sqrtf(rho2);
  const float phi = -kPiF + ((float)sector + u[3]) * (2.0f * kPiF / (float)ns);
  // height over the disk point, sqrt(1 - rho^2), formed without cancellation
  // near the disk's rim: 1 - rho^2 = (1 - s2) + s2 (1 - t) for rho^2 = s2 t,
  // with 1 - t = ((nr - ring) - u) / nr and 1 - s2 the squared cone cosine
  const float om = ((float)(nr - ring) - u[2]) / (float)nr;
  const float c2 = lt.kind == PV_LIGHT_SPOT ? lt.param[0] * lt.param[0] : 0.0f;
  const float lx = rho * cosf(phi), ly = rho * sinf(phi), lz = sqrtf(fmaxf(c2 + s2 * om, 0.0f));
  *w = add(add(mul(eu, lx), mul(ev, ly)), mul(n, lz));
}

// Tangent frame of a unit normal (Duff et al., JCGT 2017).
__device__ inline void onb(float3 n, float3* t, float3* b) {
  float sign = n.z >= 0.0f ? 1.0f : -1.0f;
  float a = -1.0f / (sign + n.z);
  float c = n.x * n.y * a;
  *t = f3(1.0f + sign * n.x * n.x * a, sign * c, -sign * n.x);
  *b = f3(c, sign + n.y * n.y * a, -n.y);
}

}  // namespace pv
