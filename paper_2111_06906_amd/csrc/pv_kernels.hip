// HIP kernels of the path-verification hot path (gfx950).
//
//   k_verify_*      Section 3.1 origin update + Section 3.2 dynamic occlusions,
//                   first invalid segment
//   k_scan          exclusive scan of per-block counts (single block)
//   k_queue_hist / k_queue_scatter   stable re-trace work queue and its order
//   k_mark_all      full invalidation (baseline / frame 0)
//   k_retrace       persistent re-trace over the device work queue
//   k_photon_count / k_photon_scatter   compaction of existing photons
//   k_energy_fwd / k_energy_bwd / k_energy_sum   differentiation form
#include "pv_device.h"
#include "pv_launch.h"

namespace pv {

__device__ inline uint32_t lane_id() { return threadIdx.x & 63u; }
__device__ inline uint64_t lanemask_lt() { return (1ull << lane_id()) - 1ull; }

// block-wide sum of one value per thread (kBlock threads), result to all
__device__ inline unsigned long long block_sum_u64(unsigned long long v, unsigned long long* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  if (lane_id() == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  unsigned long long t = 0;
  for (int w = 0; w < kBlock / 64; ++w) t += sh[w];
  __syncthreads();
  return t;
}

// ---------------------------------------------------------------------------
// sparse transform update (one wave, n <= 64): row ids[i] of dst takes the 12
// floats m[i]; when an id repeats, its last entry wins; ids >= n_rows are
// skipped

__global__ __launch_bounds__(64) void k_scatter_xf(float* __restrict__ dst, uint32_t n_rows,
                                                   const uint32_t* __restrict__ ids,
                                                   const float* __restrict__ m, uint32_t n) {
  __shared__ uint32_t sid[64];
  const uint32_t i = threadIdx.x;
  const uint32_t id = i < n ? ids[i] : 0xFFFFFFFFu;
  sid[i] = id;
  __syncthreads();
  if (i >= n || id >= n_rows) return;
  for (uint32_t j = i + 1; j < n; ++j)
    if (sid[j] == id) return;
  for (int c = 0; c < 12; ++c) dst[12 * (size_t)id + c] = m[12 * (size_t)i + c];
}

hipError_t launch_scatter_xf(float* dst, uint32_t n_rows, const uint32_t* ids, const float* m, uint32_t n,
                             hipStream_t s) {
  if (n == 0) return hipSuccess;
  if (n > 64) return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_scatter_xf, dim3(1), dim3(64), 0, s, dst, n_rows, ids, m, n);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// verification (Sections 3.1 and 3.2)

// Moved objects of a scene in LDS: box corners with the object's global
// triangle id range in the w components (lo.w = first id, hi.w = count), and
// the same id ranges merged where consecutive moved objects' ids adjoin
// (run[k] = {first id, count}; one run when every object moves).
struct MovedSet {
  int n, nr;
  float4 lo[PV_MAX_OBJECTS], hi[PV_MAX_OBJECTS];
  uint2 run[PV_MAX_OBJECTS];
};

// the moved objects of the scene, compacted in object order by the first wave
// (at most PV_MAX_OBJECTS = 64 objects: one lane each)
__device__ inline void load_moved(const SceneDev& S, MovedSet& M) {
  static_assert(PV_MAX_OBJECTS <= 64, "one lane per object");
  if (threadIdx.x < 64) {
    const uint32_t o = threadIdx.x;
    const bool have = o < S.n_obj;
    const bool mv = have && G(S.obj_moved)[o] != 0;
    const uint64_t m = __ballot(mv);
    ObjDev ob{};
    if (have) ob = G(S.objs)[o];
    if (mv) {
      const uint32_t i = (uint32_t)__popcll(m & lanemask_lt());
      const PV_GLOBAL float* b = G(S.obj_aabb) + 6 * o;
      M.lo[i] = make_float4(b[0], b[1], b[2], __uint_as_float(ob.gbase));
      M.hi[i] = make_float4(b[3], b[4], b[5], __uint_as_float(ob.n_tris));
    }
    // runs: a moved object continues the run of the object before it when
    // that one moved too and its ids end where this one's begin
    const uint32_t end = ob.gbase + ob.n_tris;
    const uint32_t prev_end = __shfl_up(end, 1, 64);
    const bool cont = mv && o > 0 && ((m >> (o - 1)) & 1ull) && prev_end == ob.gbase;
    const bool start = mv && !cont;
    const uint64_t cm = __ballot(cont), sm = __ballot(start);
    const uint64_t after = o < 63 ? ~cm >> (o + 1) : 0ull;  // lanes past o that end a run
    const uint32_t last = o + (after ? (uint32_t)__ffsll((long long)after) - 1u : 63u - o);
    const uint32_t run_end = __shfl(end, (int)last, 64);
    if (start) M.run[__popcll(sm & lanemask_lt())] = make_uint2(ob.gbase, run_end - ob.gbase);
    if (o == 0) {
      M.n = (int)__popcll(m);
      M.nr = (int)__popcll(sm);
    }
  }
  __syncthreads();
}

// whether a stored hit id lies on a moved object (no early exit: the loop
// count is uniform over the block)
__device__ inline bool on_moved(const MovedSet& M, uint32_t hit) {
  bool mv = false;
  for (int k = 0; k < M.nr; ++k) mv |= hit - M.run[k].x < M.run[k].y;
  return mv;
}

// whether a segment's query reaches box [lo, hi] within its interval: the
// same decision as box_entry(...) != inf when tmin <= tmax, with the interval
// entering by comparisons (the slab parameters are fma results, so the
// min/max need no operand canonicalisation)
__device__ inline bool slab_hit(float4 lo, float4 hi, const BoxRay& r) {
  const float x0 = fmaf(lo.x, r.inv.x, r.oi.x), x1 = fmaf(hi.x, r.inv.x, r.oi.x);
  const float y0 = fmaf(lo.y, r.inv.y, r.oi.y), y1 = fmaf(hi.y, r.inv.y, r.oi.y);
  const float z0 = fmaf(lo.z, r.inv.z, r.oi.z), z1 = fmaf(hi.z, r.inv.z, r.oi.z);
  const float e = fmaxf(fmaxf(fminf(x0, x1), fminf(y0, y1)), fmaxf(fminf(z0, z1), r.tmin));
  const float x = fminf(fminf(fmaxf(x0, x1), fmaxf(y0, y1)), fminf(fmaxf(z0, z1), r.tmax));
  return e <= x;
}

// whether a ray reaches any moved object's box within its interval
__device__ inline bool reaches_moved_box(const MovedSet& M, const BoxRay& r) {
  bool h = false;
  for (int i = 0; i < M.n; ++i) {
    const float4 lo = M.lo[i], hi = M.hi[i];
    h |= box_entry(lo.x, lo.y, lo.z, hi.x, hi.y, hi.z, r, r.tmax) != __builtin_inff();
  }
  return h;
}

__device__ inline Ray segment_ray(float3 a, float3 b, float eps, float* tmax) {
  float3 d = sub(b, a);
  float L = length(d);
  float tmin = L > 0.0f ? eps / L : 1.0f;
  *tmax = 1.0f - tmin;
  return make_ray(a, d, tmin);
}

// The box-test part of segment_ray, for filters only: 1/d from the hardware
// reciprocal (1 ulp) and the end tolerance shortened by 1e-5 relative.  Both
// move slab parameters by about 1e-7 of the segment or widen the tested
// interval, far inside the 1e-6 padding of every stored box, so a segment that
// crosses a triangle inside a box always reaches that box.
__device__ inline BoxRay segment_box_ray(float3 a, float3 b, float eps) {
  BoxRay r;
  const float3 d = sub(b, a);
  r.inv = rcp3(d);
  r.oi = f3(-(a.x * r.inv.x), -(a.y * r.inv.y), -(a.z * r.inv.z));
  const float L2 = dot(d, d);
  r.tmin = L2 > 0.0f ? eps * __builtin_amdgcn_rsqf(L2) * (1.0f - 1e-5f) : 1.0f;
  r.tmax = 1.0f - r.tmin;
  return r;
}

__device__ inline float uniform(float x) { return __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(x))); }

// plane_base of a single-scene launch's scene, in scalar registers
template <bool kScaled>
__device__ inline float3 scene_base(const SceneDev& S) {
  const float3 b = plane_base<kScaled>(S);
  return f3(uniform(b.x), uniform(b.y), uniform(b.z));
}

// Whether a launch's nodes are read as WALK_SCALED: where the frame of any of
// its scenes asks for it (called by whole workgroups; the other scenes' nodes
// read the same way).  A kernel holds its persistent loop twice, once for each
// form, so that the usual one's registers and code are its own: as a branch
// inside the walk the rare form made the re-trace spill 13 registers instead of
// 2 (full trace 3.54 ms instead of 3.46, paper-scale frame 2.06 instead of 2.01).
template <bool kSingle>
__device__ inline bool any_scaled(const SceneDev* scenes, int n_scenes) {
  if (kSingle) return uniform(frame_reach(scenes[0])) == __builtin_inff();
  bool scaled = false;
  for (int i = (int)threadIdx.x; i < n_scenes; i += (int)blockDim.x) scaled |= frame_reach(scenes[i]) == __builtin_inff();
  return __syncthreads_or(scaled) != 0;
}

__device__ inline int light_of(const SceneDev& S, uint32_t p) {
  const PV_GLOBAL LightDev* lights = G(S.lights);
  for (uint32_t l = 0; l < S.n_lights; ++l)
    if (p - lights[l].path_base < lights[l].path_count) return (int)l;
  return -1;
}

// Section 3.1 for a rectangular area light: keep the outgoing direction and
// intersect it with the light's current plane.  A light with both half
// extents 0 is a point light: the sample becomes the light's new position and
// segment 0 is re-aimed at the first photon, which must lie on the emitting
// side farther than eps_end; *vis then asks for segment 0 to be tested
// against every triangle (the visibility the paper reads from a shadow map).
__device__ inline bool light_update(const SceneDev& S, int l, float3 x0, float3 x1, float3* out, bool* vis) {
  const PV_GLOBAL float* xf = G(S.light_xf_cur) + 12 * l;
  float3 eu = f3(xf[0], xf[4], xf[8]), ev = f3(xf[1], xf[5], xf[9]);
  float3 n = f3(xf[2], xf[6], xf[10]), c = f3(xf[3], xf[7], xf[11]);
  const PV_GLOBAL LightDev* lt = G(S.lights) + l;
  if (lt->half[0] == 0.0f && lt->half[1] == 0.0f) {
    const float3 w = sub(x1, c);
    const float z = dot(w, n);
    if (!(dot(w, w) > S.eps_end * S.eps_end) || !(z > 0.0f)) return false;
    const int32_t kind = lt->kind;
    if (kind == PV_LIGHT_SPOT) {
      // inside the cone: z / |w| >= cos of the half-angle
      if (!(z * __builtin_amdgcn_rsqf(dot(w, w) * dot(n, n)) >= lt->param[0])) return false;
    } else if (kind == PV_LIGHT_CAMERA) {
      // through the near plane: |u / z| <= tan_u, |v / z| <= tan_v (n unit length)
      const float zn = z * __builtin_amdgcn_rsqf(dot(n, n));
      if (!(fabsf(dot(w, eu)) <= lt->param[0] * zn && fabsf(dot(w, ev)) <= lt->param[1] * zn)) return false;
    }
    *out = c;
    *vis = true;
    return true;
  }
  // hardware reciprocal and reciprocal square root (about 1 ulp): the
  // decisions match the FP64 update outside its 1e-6 band, the new origin
  // within the position tolerance
  n = mul(n, __builtin_amdgcn_rsqf(dot(n, n)));
  float3 w = sub(x1, x0);
  const float l2 = dot(w, w);
  if (!(l2 > 0.0f)) return false;
  w = mul(w, __builtin_amdgcn_rsqf(l2));
  const float dn = dot(w, n);
  if (!(dn > 0.0f)) return false;
  const float sdist = dot(sub(x1, c), n) * __builtin_amdgcn_rcpf(dn);
  if (!(sdist > S.eps_end)) return false;
  float3 p = sub(x1, mul(w, sdist));
  float3 r = sub(p, c);
  float u = dot(r, eu), v = dot(r, ev);
  if (!(fabsf(u) <= lt->half[0] && fabsf(v) <= lt->half[1])) return false;
  *out = p;
  return true;
}

// The scene bases of a multi-scene launch (gbase[0..n_scenes]) copied to LDS
// by the whole block, so that the binary search of scene_of reads LDS (up to
// kLdsScenes scenes; larger batches keep reading global memory).  Ends with a
// barrier.
constexpr int kLdsScenes = 256;
__device__ inline const uint32_t* stage_gbase(const uint32_t* gbase, int n_scenes, uint32_t* sg) {
  if (n_scenes > kLdsScenes) return gbase;
  for (int i = (int)threadIdx.x; i <= n_scenes; i += (int)blockDim.x) sg[i] = gbase[i];
  __syncthreads();
  return sg;
}

// scene of a global path id: gbase[s] <= gp < gbase[s + 1]
__device__ inline uint32_t scene_of(const uint32_t* gbase, int n_scenes, uint32_t gp) {
  int lo = 0, hi = n_scenes;  // gbase[s] <= gp < gbase[s+1]
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (gbase[mid] <= gp)
      lo = mid;
    else
      hi = mid;
  }
  return (uint32_t)lo;
}

// Work lists are dealt to the waves of a persistent grid dynamically, a
// refill at a time: a wave whose idle lanes want work adds their number to its
// group's counter (one device atomic per refill) and takes that many entries
// of the group's share, chunks g, g + kDealGroups, ... of kChunk entries, in
// list order.  Static shares per wave left a wave idle for 12% of a re-trace
// launch on average (the sums of ~340 path costs differ from wave to wave);
// one counter for all waves serialised the atomics on one word; with 64
// groups each counter sees a few hundred refills per launch.  The group's
// n-th entry (groups: kDealGroups, or one per wave for grids of fewer waves):
constexpr uint32_t kChunk = 64;
__device__ inline uint32_t group_entry(uint32_t g, uint32_t groups, uint32_t n) {
  return ((n / kChunk) * groups + g) * kChunk + n % kChunk;
}

constexpr uint32_t kNoEntry = 0xFFFFFFFFu;

// The entry a lane that wants work takes (kNoEntry once its group's share is
// exhausted).  Called by every lane of the wave.
__device__ inline uint32_t deal(uint32_t* __restrict__ ctrs, uint32_t wave, uint32_t count, bool want) {
  const uint64_t m = __ballot(want);
  if (!m) return kNoEntry;
  const uint32_t groups = min(kDealGroups, gridDim.x * (blockDim.x / 64));
  const uint32_t g = wave % groups;
  const uint32_t leader = (uint32_t)__ffsll((long long)m) - 1u;
  uint32_t base = 0;
  if (lane_id() == leader) base = atomicAdd(ctrs + g * kDealStride, (uint32_t)__popcll(m));
  base = __shfl(base, (int)leader, 64);
  if (!want) return kNoEntry;
  const uint32_t idx = group_entry(g, groups, base + (uint32_t)__popcll(m & lanemask_lt()));
  return idx < count ? idx : kNoEntry;
}

// A list shorter than the lanes of 'waves' waves is spread over that many
// waves instead: wave w takes entries [w q, (w + 1) q) with its first q lanes,
// q = ceil(count / waves), and nothing is dealt.  (64: the list is dealt.)
// A wave's time is the sum over its rounds of the longest walk among its
// lanes, so that few lanes per wave finish sooner as long as waves share no
// SIMD with many others, and all of them are there from the start.
//
// Re-traced paths of a 50k-triangle interior spread over four workgroups per
// compute unit, against dealt, in us: 77k 266 and 334, 103k 300 and 314, 129k
// 320 and 326, 155k 323 and 335, 181k 335 and 355, 215k 348 and 355, camera
// paths 96k 303 and 330, 193k 356 and 371, 225k 371 and 386; lists of up to 51k
// within 3%.  So spreading is the better of the two up to the 64 lanes at which
// it ends.  Over three workgroups the same lists take up to 7% longer; where
// only three fit beside each other (the largest stacks: 24 rebuilt objects, 45k
// paths) a fourth makes it about 400 us instead of 302.  Verification tasks over two
// workgroups: 59k 61 and 67 us, 88k 72 and 78, 118k 80 and 83 (over four 61, 72
// and 78, but 29k 65 instead of 58).
constexpr uint32_t kSpreadRetrace = 4, kSpreadVerify = 2;  // workgroups per compute unit, as far as they fit
__device__ inline uint32_t wave_quota(uint32_t count, uint32_t waves) {
  return min(64u, max(1u, (count + waves - 1) / waves));
}

// Lanes below which a walk yields.  While there is work to deal, min_active.
// Once the wave has asked in vain nothing takes a finished lane's place and
// that number, sooner or later above the lanes left, would stop the walk after
// every descent for the state machine: then a share of the lanes still walking
// (half of what min_active is of a full wave).  With it a 60k-path
// frame took 506 us instead of 547, a 300k-path camera frame 431 instead of
// 463, a 750k-path spot frame 1015 instead of 1120, full trace 3.44 ms instead
// of 3.49; a yield at the last lane only, 3.49.
__device__ inline int yield_below(int min_active, bool drained, int walking) {
  return drained ? max(1, walking * min_active / 128) : min_active;
}

// The counters are zero between launches: the last workgroup to end a launch
// that dealt from them clears them again (arrivals are counted per group, then
// over the groups, so that no word takes more than a few dozen additions).
// Called by every thread of the workgroup, after its last deal().
__device__ inline void deal_done(uint32_t* __restrict__ ctrs) {
  __shared__ uint32_t last;
  __syncthreads();
  if (threadIdx.x == 0) {
    const uint32_t groups = min(kDealGroups, gridDim.x), g = blockIdx.x % groups;
    const uint32_t members = (gridDim.x - g + groups - 1) / groups;
    last = 0;
    if (atomicAdd(ctrs + g * kDealStride + 1, 1u) + 1 == members)
      last = atomicAdd(ctrs + kDealGroups * kDealStride, 1u) + 1 == groups ? 1u : 0u;
  }
  __syncthreads();
  if (!last) return;
  if (threadIdx.x < kDealGroups) {
    uint32_t* c = ctrs + threadIdx.x * kDealStride;
    __hip_atomic_store(c, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(c + 1, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  if (threadIdx.x == 0)
    __hip_atomic_store(ctrs + kDealGroups * kDealStride, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// sum of in[0 .. n) by the whole workgroup, result to all (n up to a few
// thousand: read with 16-byte loads, in is 16-byte aligned)
__device__ inline uint32_t block_prefix(const uint32_t* __restrict__ in, uint32_t n, uint32_t* sh) {
  uint32_t v = 0;
  const uint4* in4 = reinterpret_cast<const uint4*>(in);
#pragma unroll 4
  for (uint32_t i = threadIdx.x; i < n / 4; i += kBlock) {
    const uint4 q = in4[i];
    v += q.x + q.y + q.z + q.w;
  }
  if (threadIdx.x < n % 4) v += in[n / 4 * 4 + threadIdx.x];
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  __syncthreads();
  if (lane_id() == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  uint32_t t = 0;
  for (int w = 0; w < kBlock / 64; ++w) t += sh[w];
  return t;
}

// Verification runs as a short chain of kernels without atomics.
//  k_verify_scan (coalesced, lane per path, no traversal): origin update for
//    moved lights, the bounce rows read up front, endpoint test, and one task
//    per segment whose ray reaches a moved object's box, written into the
//    tile's own region; scanning stops at the first segment whose end photon
//    is on a moved object (that segment is invalid whatever lies before it).
//    Writes the information word as if no task were blocked (final for paths
//    without tasks).
//  k_verify_gather: one compact task list.
//  k_verify_trace: the tasks as independent any-hit queries against the
//    moved objects, every lane busy; a blocked segment lowers its path's
//    first invalid segment (atomic minimum on that path's own word).
//  k_verify_finish: information words of the paths with tasks, statistics.
// The result equals the in-order test of Section 3.2: the first invalid
// segment is the minimum over blocked segments and the first moved endpoint.

constexpr int kPreRows = 8;  // bounce rows a lane loads before testing
// task segment field of a point light's visibility test of segment 0 (real
// segments are 0..14)
constexpr uint32_t kVisTask = 15;
static_assert(PV_MAX_BOUNCES <= 15, "segment indices below kVisTask");

__global__ __launch_bounds__(kBlock) void k_verify_scan(const SceneDev* __restrict__ scenes,
                                                        const uint2* __restrict__ tiles, VerifyWork W,
                                                        pv_stats* stats) {
  __shared__ MovedSet M;
  __shared__ unsigned long long sred[kBlock / 64];
  __shared__ uint32_t swt[kBlock / 64];
  uint2 tile = tiles[blockIdx.x];
  const SceneDev& S = scenes[tile.x];
  load_moved(S, M);
  const uint32_t tid = threadIdx.x;
  const uint32_t p = tile.y + tid;
  const bool active = p < S.n_paths;
  const size_t stride = S.stride;
  uint32_t n = 0, cell = 0, cap = 0, mask = 0, lost = 0;
  bool vis = false;  // a point light moved: segment 0 against every triangle
  if (active) {
    const PV_GLOBAL float4* pos = G(S.pos);
    PV_GLOBAL float* org = G(S.origin);
    uint32_t w = G(S.info)[p];
    n = min(info_nseg(w), S.B);
    cell = info_cell(w);
    cap = n;
    // the path's rows (up to kPreRows) are all requested before the first
    // is used, so their loads are in flight together
    float4 rows[kPreRows];
    const uint32_t nload = M.n > 0 ? n : min(n, 1u);  // the light update needs the first hit only
#pragma unroll
    for (int j = 0; j < kPreRows; ++j) {
      rows[j] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      if ((uint32_t)j < nload) rows[j] = pos[(size_t)j * stride + p];
    }
    float3 a = f3(org[p], org[stride + p], org[2 * stride + p]);
    int l = light_of(S, p);
    if (l >= 0 && G(S.light_moved)[l]) {
      float3 na;
      if (n > 0 && light_update(S, l, a, xyz(rows[0]), &na, &vis)) {
        a = na;
        org[p] = na.x;
        org[stride + p] = na.y;
        org[2 * stride + p] = na.z;
      } else {
        lost = 1;
        cap = 0;
      }
    }
    if (!lost && M.n > 0) {
      // every segment of the path is tested (no early exit); the first
      // segment whose end photon lies on a moved object caps the scan.  The
      // loaded rows' segments are set up first, then each moved box is read
      // once and tested against all of them (rows past n are masked off).
      // Rows are tested up to the scene's bounce limit (uniform), not the
      // path's own count, so that no lane-dependent branch splits the loop.
      // Box hits are collected as wave masks (one per row, scalar registers).
      BoxRay rs[kPreRows];
      uint64_t hit[kPreRows];
      uint32_t mv = 0;
#pragma unroll
      for (int j = 0; j < kPreRows; ++j) {
        hit[j] = 0;
        if ((uint32_t)j < S.B) {
          const float3 b = xyz(rows[j]);
          rs[j] = segment_box_ray(a, b, S.eps_end);
          if (!(rs[j].tmin <= rs[j].tmax)) rs[j].tmin = __builtin_inff();  // nothing to test
          rs[j].tmin = __builtin_canonicalizef(rs[j].tmin);
          rs[j].tmax = __builtin_canonicalizef(rs[j].tmax);
          if (on_moved(M, __float_as_uint(rows[j].w))) mv |= 1u << j;
          a = b;
        }
      }
      for (int i = 0; i < M.n; ++i) {
        const float4 lo = M.lo[i], hi = M.hi[i];
#pragma unroll
        for (int j = 0; j < kPreRows; ++j)
          if ((uint32_t)j < S.B) hit[j] |= __builtin_amdgcn_ballot_w64(slab_hit(lo, hi, rs[j]));
      }
#pragma unroll
      for (int j = 0; j < kPreRows; ++j) mask |= (uint32_t)((hit[j] >> lane_id()) & 1ull) << j;
      uint32_t first_mv = min(n, mv ? (uint32_t)__ffs(mv) - 1u : n);
      for (uint32_t j = kPreRows; j < n; ++j) {
        const float4 row = pos[(size_t)j * stride + p];
        const float3 b = xyz(row);
        if (on_moved(M, __float_as_uint(row.w))) first_mv = min(first_mv, j);
        if (reaches_moved_box(M, segment_box_ray(a, b, S.eps_end))) mask |= 1u << j;
        a = b;
      }
      if (S.verify_boxes) {
        // Section 3.2's own test: the first segment that reaches a moved
        // box is invalid, no triangle is tested (rows past n masked off)
        mask &= (1u << n) - 1u;
        cap = min(first_mv, mask ? (uint32_t)__ffs(mask) - 1u : n);
        mask = 0;
      } else {
        cap = first_mv;
        mask &= (1u << cap) - 1u;
      }
    }
    // the visibility task (segment index kVisTask) replaces segment 0's own
    // test, which it covers; none when segment 0 is already invalid
    if (vis && cap > 0) mask = (mask & ~1u) | (1u << kVisTask);
  }
  // ---- tasks into the tile's region, in lane order
  const uint32_t nt = (uint32_t)__popc(mask);
  uint32_t x = nt;  // inclusive wave prefix of the task counts
  for (int o = 1; o < 64; o <<= 1) {
    uint32_t y = __shfl_up(x, o, 64);
    if ((int)lane_id() >= o) x += y;
  }
  const uint32_t wave = tid >> 6;
  if (lane_id() == 63) swt[wave] = x;
  __syncthreads();
  uint32_t before = 0, all = 0;
  for (uint32_t w = 0; w < kBlock / 64; ++w) {
    before += w < wave ? swt[w] : 0u;
    all += swt[w];
  }
  if (tid == 0) W.tcount[blockIdx.x] = all;
  if (nt > 0) {
    const uint32_t gp = S.gpath_base + p;
    W.first[gp] = cap;
    PV_GLOBAL uint32_t* region =
        G(W.tmp) + S.task_base + (size_t)(blockIdx.x - S.tile_base) * kBlock * S.B;
    uint32_t t = before + x - nt;
    for (uint32_t m = mask; m; m &= m - 1) region[t++] = (gp << 4) | (uint32_t)(__ffs(m) - 1);
  }
  // ---- information word as if no task were blocked
  uint32_t ex = 0, inv = 0;
  if (active) {
    uint32_t out;
    if (lost) {
      out = info_pack(cell, n, 0, 1, 0);
    } else if (cap < n) {
      out = info_pack(cell, n, cap, 1, 1);
      ex = cap + 1;
    } else {
      out = info_pack(cell, n, 0, 0, 0);
      ex = n;
    }
    G(S.info)[p] = out;
    inv = info_replace(out);
    if (nt > 0) ex = inv = 0;  // counted by k_verify_finish
  }
  if (stats) {
    // per-block counts go to their own slots and are summed by
    // k_verify_finish: one counter word shared by every block would serialise
    // thousands of atomics.  Each count is at most kBlock * 15 < 2^16 per
    // block, so the four travel as 16-bit fields of one sum.
    static_assert(kBlock * 15 < (1 << 16), "16-bit fields");
    const unsigned long long packed = (unsigned long long)ex | ((unsigned long long)inv << 16) |
                                      ((unsigned long long)lost << 32) | ((unsigned long long)nt << 48);
    const unsigned long long sum = block_sum_u64(packed, sred);
    if (tid == 0) {
      uint32_t* o = W.part + 4 * (size_t)blockIdx.x;
      o[0] = (uint32_t)(sum & 0xffffu);
      o[1] = (uint32_t)((sum >> 16) & 0xffffu);
      o[2] = (uint32_t)((sum >> 32) & 0xffffu);
      o[3] = (uint32_t)(sum >> 48);
    }
  }
}

// A workgroup moves the tasks of kGatherTiles path tiles, a wave a tile at a
// time, to their place in the compacted list.  The tiles' offsets come from
// 'toff', or, for a few thousand tiles, from the counts themselves: every
// workgroup sums the counts before its own (at most 64 KB from L2, 8 KB on
// average for 3M paths), which takes less than the launch of a scan (8 us).
constexpr uint32_t kGatherTiles = 8;
constexpr uint32_t kInlineTiles = 16384;

__global__ __launch_bounds__(kBlock) void k_verify_gather(const SceneDev* __restrict__ scenes,
                                                          const uint2* __restrict__ tiles, uint32_t n_tiles,
                                                          VerifyWork W, const uint32_t* __restrict__ toff) {
  __shared__ uint32_t sh[kBlock / 64];
  __shared__ uint32_t cnt[kGatherTiles], off[kGatherTiles];
  const uint32_t t0 = blockIdx.x * kGatherTiles, m = min(kGatherTiles, n_tiles - t0);
  const uint32_t before = toff ? 0u : block_prefix(W.tcount, t0, sh);
  if (threadIdx.x < 64) {
    const uint32_t i = threadIdx.x;
    const uint32_t c = i < m ? W.tcount[t0 + i] : 0u;
    uint32_t x = c;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if ((int)i >= o) x += y;
    }
    if (i < m) {
      cnt[i] = c;
      off[i] = toff ? toff[t0 + i] : before + x - c;
    }
    if (!toff && t0 + m == n_tiles && i == 63) *W.total = before + x;
  }
  __syncthreads();
  for (uint32_t i = threadIdx.x >> 6; i < m; i += kBlock / 64) {
    const uint2 tile = tiles[t0 + i];
    const SceneDev& S = scenes[tile.x];
    const PV_GLOBAL uint32_t* src = G(W.tmp) + S.task_base + (size_t)(t0 + i - S.tile_base) * kBlock * S.B;
    PV_GLOBAL uint32_t* dst = G(W.tasks) + off[i];
    for (uint32_t k = lane_id(); k < cnt[i]; k += 64) dst[k] = src[k];
  }
}

// The moved objects of a single scene: boxes, roots of their current
// hierarchies, of their upload-time topologies with object-space boxes
// with the least tmin of a segment that is walked there (longer ones, and those
// of a transform without an inverse, are walked in world space), the inverses of
// their transforms (rows of the inverse 3x3, then the translation), and the
// grids of the object-space forms (what their planes count from, and the step).
struct MovedTab {
  MovedSet M;
  int32_t root[PV_MAX_OBJECTS], oroot[PV_MAX_OBJECTS];
  float tmin[PV_MAX_OBJECTS];
  float inv[PV_MAX_OBJECTS][12];
  float4 grid[PV_MAX_OBJECTS];
};

// Persistent: a lane whose walk has finished takes the wave's next task
// (dealt by deal()) while the other lanes continue.

template <bool kSingle, bool kScaled>
__device__ __forceinline__ void verify_loop(const SceneDev* __restrict__ scenes, const uint32_t* __restrict__ gbase,
                                            int n_scenes, const VerifyWork& W, const MovedTab& T, int min_active,
                                            uint32_t entries, uint32_t spread_waves) {
  extern __shared__ int32_t sstack[];  // traversal stacks, launch-time size
  const StackCol col = (StackCol)(sstack + kBlock + threadIdx.x);  // entry 0 of the column; entry -1 spare
  const StackCol limit = col + (int)(entries - 5) * kBlock;  // top from which a full node would pass the last entry
  const float3 base0 = scene_base<kScaled>(scenes[0]);
  const uint32_t total = *W.total;
  const uint32_t wave = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const uint32_t quota = wave_quota(total, spread_waves);
  if (quota < 64) min_active = max(1, (int)(quota * (uint32_t)min_active / 64u));
  bool fresh = true;  // this wave has not taken its share of a spread list
  Walk w;
  w.cur = kRootNone;
  w.leaf = 0;
  Ray r;
  Slab qb{};  // slab parameters of the walk's boxes
  uint32_t gp = 0, j = 0;
  bool busy = false, drained = false, vis_task = false;
  const SceneDev* S = scenes;
  while (true) {
    // lanes without a task take the next ones; a task whose path already
    // failed at an earlier segment is dropped (the minimum only decreases)
    const bool want = !busy && !drained;
    if (__ballot(want)) {
      uint32_t t;
      if (quota < 64) {
        const uint32_t e = wave * quota + lane_id();
        t = fresh && lane_id() < quota && e < total ? e : kNoEntry;
        fresh = false;
      } else {
        t = deal(W.deal, wave, total, want);
      }
      if (want) {
        if (t == kNoEntry) {
          drained = true;
        } else {
          const uint32_t tk = G(W.tasks)[t];
          gp = tk >> 4;
          j = tk & 15u;
          const bool vis = j == kVisTask;  // segment 0 against the whole scene
          if (vis) j = 0;
          if (j < __hip_atomic_load(&W.first[gp], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
            S = scenes + (kSingle ? 0u : scene_of(gbase, n_scenes, gp));
            const uint32_t q = gp - S->gpath_base;
            const size_t stride = S->stride;
            const PV_GLOBAL float* org = G(S->origin);
            const float3 a = j == 0 ? f3(org[q], org[stride + q], org[2 * stride + q])
                                    : xyz(G(S->pos)[(size_t)(j - 1) * stride + q]);
            const float3 b = xyz(G(S->pos)[(size_t)j * stride + q]);
            float tmax;
            r = segment_ray(a, b, S->eps_end, &tmax);
            const BoxRay br = segment_box_ray(a, b, S->eps_end);
            const float3 c = sub(kSingle ? base0 : plane_base<kScaled>(*S), a);
            qb = world_slab(*S, c, br.inv, r.tmin);
            bool far = walk_far(*S, c);
            int32_t root = G(S->wtop)[1];
            if (kSingle && !vis) {
              // the objects whose boxes the segment reaches, from LDS: one
              // object is walked from its own root (its box is the only one
              // of the moved-object tree the ray enters); several, through
              // the moved-object tree; none, not at all
              uint32_t nh = 0;
              int only = 0;
              for (int i = 0; i < T.M.n; ++i) {
                const float4 lo = T.M.lo[i], hi = T.M.hi[i];
                const bool h = box_entry(lo.x, lo.y, lo.z, hi.x, hi.y, hi.z, br, br.tmax) != __builtin_inff();
                nh += h ? 1u : 0u;
                only = h ? i : only;
              }
              root = nh == 0 ? kRootNone : (nh == 1 ? T.root[only] : root);
              if (nh == 1 && r.tmin >= T.tmin[only]) {
                // a rigid object is walked in its own space: the segment
                // mapped by the inverse transform (same parameter interval)
                // meets the fixed object-space boxes, which are tighter than
                // the world boxes of the rotated nodes; triangles are still
                // tested in world space
                const float* mi = T.inv[only];
                const float3 ta = sub(a, f3(mi[9], mi[10], mi[11])), tb = sub(b, f3(mi[9], mi[10], mi[11]));
                const float3 oa = f3(mi[0] * ta.x + mi[1] * ta.y + mi[2] * ta.z,
                                     mi[3] * ta.x + mi[4] * ta.y + mi[5] * ta.z,
                                     mi[6] * ta.x + mi[7] * ta.y + mi[8] * ta.z);
                const float3 ob = f3(mi[0] * tb.x + mi[1] * tb.y + mi[2] * tb.z,
                                     mi[3] * tb.x + mi[4] * tb.y + mi[5] * tb.z,
                                     mi[6] * tb.x + mi[7] * tb.y + mi[8] * tb.z);
                const float4 og = T.grid[only];
                const float3 oc = sub(xyz(og), oa), binv = rcp3(sub(ob, oa));
                qb = make_slab(binv, f3(oc.x * binv.x, oc.y * binv.y, oc.z * binv.z), og.w, r.tmin);
                root = T.oroot[only];
                far = false;
              }
            }
            if (vis) root = G(S->wtop)[0];
            vis_task = vis;
            walk_start(w, root, tmax, col);
            busy = root != kRootNone;
            if (far) walk_leave(w);
          }
        }
      }
    }
    if (__ballot(busy) == 0) {
      if (__ballot(!drained) == 0) break;
      continue;
    }
    const int yield = yield_below(min_active, __ballot(drained) != 0, (int)__popcll(__ballot(busy)));
    if (busy) {
      walk_scene<false, kScaled>(*S, r, qb, true, col, limit, w, yield);
      if (walk_done(w)) {
        if (w.redo) walk_exact(G(S->nodes), G(S->tris), r, 1.0f - r.tmin, G(S->top)[vis_task ? 0 : 1], true, col, w);
        if (w.rec != kRecNone) atomicMin(&W.first[gp], j);
        busy = false;
      }
    }
  }
  if (quota >= 64) deal_done(W.deal);  // uniform over the grid
}

template <bool kSingle>
__global__ __launch_bounds__(kBlock) void k_verify_trace(const SceneDev* __restrict__ scenes,
                                                         const uint32_t* __restrict__ gbase, int n_scenes,
                                                         VerifyWork W, int min_active, uint32_t entries,
                                                         uint32_t spread_waves) {
  __shared__ MovedTab T;
  const bool scaled = any_scaled<kSingle>(scenes, n_scenes);
  if (kSingle) {
    if (threadIdx.x < 64) {
      const SceneDev& S0 = scenes[0];
      const uint32_t o = threadIdx.x;
      const bool mv = o < S0.n_obj && G(S0.obj_moved)[o] != 0;
      const uint64_t mm = __ballot(mv);
      if (mv) {
        const uint32_t i = (uint32_t)__popcll(mm & lanemask_lt());
        const ObjDev ob = G(S0.objs)[o];
        T.root[i] = ob.wroot;
        // inverse of the 3x3 part by cofactors in FP64
        const PV_GLOBAL float* x = G(S0.obj_xf_cur) + 12 * o;
        const double m0 = x[0], m1 = x[1], m2 = x[2], m4 = x[4], m5 = x[5], m6 = x[6];
        const double m8 = x[8], m9 = x[9], m10 = x[10];
        const double c00 = m5 * m10 - m6 * m9, c01 = m2 * m9 - m1 * m10, c02 = m1 * m6 - m2 * m5;
        const double det = m0 * c00 + m4 * c01 + m8 * c02;
        const bool ok = fabs(det) > 1e-12 && isfinite(det);
        const double id = ok ? 1.0 / det : 0.0;
        T.inv[i][0] = (float)(c00 * id);
        T.inv[i][1] = (float)(c01 * id);
        T.inv[i][2] = (float)(c02 * id);
        T.inv[i][3] = (float)((m6 * m8 - m4 * m10) * id);
        T.inv[i][4] = (float)((m0 * m10 - m2 * m8) * id);
        T.inv[i][5] = (float)((m2 * m4 - m0 * m6) * id);
        T.inv[i][6] = (float)((m4 * m9 - m5 * m8) * id);
        T.inv[i][7] = (float)((m1 * m8 - m0 * m9) * id);
        T.inv[i][8] = (float)((m0 * m5 - m1 * m4) * id);
        T.inv[i][9] = x[3];
        T.inv[i][10] = x[7];
        T.inv[i][11] = x[11];
        T.oroot[i] = ob.oroot;
        // a segment of length L that reaches the object's world box stays within
        // 'norm' (L + the box's extent) of the object's middle in object space
        float norm = 0.0f, side = 0.0f, base = 0.0f;
        for (int k = 0; k < 3; ++k) {
          const PV_GLOBAL float* bb = G(S0.obj_aabb) + 6 * o;
          norm = fmaxf(norm, fabsf(T.inv[i][3 * k]) + fabsf(T.inv[i][3 * k + 1]) + fabsf(T.inv[i][3 * k + 2]));
          side = fmaxf(side, bb[3 + k] - bb[k]);
          base = fmaxf(base, fmaxf(fabsf(ob.centre[k]), fabsf(ob.centre[k] - ob.og[k])));
        }
        const float most = (kObjReach * ob.oinv - base) / norm - side;
        T.tmin[i] = ok && most > 0.0f ? S0.eps_end / most : __builtin_inff();
        const float mid = scaled && S0.wshift ? kOriginMid * ob.oinv : 0.0f;
        T.grid[i] = make_float4(ob.og[0] + mid, ob.og[1] + mid, ob.og[2] + mid, ob.oinv);  // exact
      }
    }
    load_moved(scenes[0], T.M);  // ends with a barrier
  }
  __shared__ uint32_t sgb[kSingle ? 1 : kLdsScenes + 1];
  if (!kSingle) gbase = stage_gbase(gbase, n_scenes, sgb);
  if (scaled)
    verify_loop<kSingle, true>(scenes, gbase, n_scenes, W, T, min_active, entries, spread_waves);
  else
    verify_loop<kSingle, false>(scenes, gbase, n_scenes, W, T, min_active, entries, spread_waves);
}

// The tasks of a path are adjacent in the list: the thread holding a path's
// first task writes its information word.  The statistics are the scan's
// per-tile counts, summed by the first kStatBlocks workgroups, and this
// kernel's own, added with one atomic per counter and workgroup (few and large
// workgroups for that reason: an addition to one line takes about 11 ns).
constexpr uint32_t kFinishBlocks = 256, kStatBlocks = 16;
constexpr int kFinishThreads = 1024;

template <bool kSingle>
__global__ __launch_bounds__(kFinishThreads) void k_verify_finish(const SceneDev* __restrict__ scenes,
                                                          const uint32_t* __restrict__ gbase, int n_scenes,
                                                          VerifyWork W, uint32_t n_tiles, pv_stats* stats) {
  __shared__ uint32_t sred[4][kFinishThreads / 64];
  __shared__ uint32_t sgb[kSingle ? 1 : kLdsScenes + 1];
  if (!kSingle) gbase = stage_gbase(gbase, n_scenes, sgb);
  const uint32_t total = *W.total;
  uint32_t ex = 0, inv = 0;
  // kIlp tasks at a time: their loads (task, then word and first) overlap
  constexpr uint32_t kIlp = 4;
  const uint32_t step = gridDim.x * kFinishThreads;
  for (uint32_t t0 = blockIdx.x * kFinishThreads + threadIdx.x; t0 < total; t0 += kIlp * step) {
    uint32_t gp[kIlp], w[kIlp], k[kIlp];
    PV_GLOBAL uint32_t* word[kIlp];
    bool use[kIlp];
#pragma unroll
    for (uint32_t i = 0; i < kIlp; ++i) {
      const uint32_t t = t0 + i * step;
      use[i] = t < total;
      gp[i] = use[i] ? G(W.tasks)[t] >> 4 : 0u;
      if (use[i] && t > 0) use[i] = (G(W.tasks)[t - 1] >> 4) != gp[i];
    }
#pragma unroll
    for (uint32_t i = 0; i < kIlp; ++i) {
      w[i] = 0;
      k[i] = 0;
      if (!use[i]) continue;
      const SceneDev& S = scenes[kSingle ? 0u : scene_of(gbase, n_scenes, gp[i])];
      word[i] = G(S.info) + (gp[i] - S.gpath_base);
      w[i] = *word[i];  // as written by the scan
      k[i] = G(W.first)[gp[i]];
    }
#pragma unroll
    for (uint32_t i = 0; i < kIlp; ++i) {
      if (!use[i]) continue;
      const uint32_t n = info_nseg(w[i]);
      if (k[i] < n) {
        *word[i] = info_pack(info_cell(w[i]), n, k[i], 1, 1);
        ex += k[i] + 1;
        inv += 1;
      } else {
        ex += n;
      }
    }
  }
  if (!stats) return;
  // counts of one launch fit 32 bits each (at most 15 per path of 2^28)
  uint32_t lost = 0, tasks = 0;
  if (blockIdx.x < kStatBlocks) {
    const uint4* __restrict__ p4 = reinterpret_cast<const uint4*>(W.part);  // one record per tile
#pragma unroll 4
    for (uint32_t b = blockIdx.x * kFinishThreads + threadIdx.x; b < n_tiles; b += min(gridDim.x, kStatBlocks) * kFinishThreads) {
      const uint4 r = p4[b];
      ex += r.x;
      inv += r.y;
      lost += r.z;
      tasks += r.w;
    }
  }
  uint32_t v[4] = {ex, inv, lost, tasks};
  for (int c = 0; c < 4; ++c)
    for (int o = 32; o > 0; o >>= 1) v[c] += __shfl_down(v[c], o, 64);
  if (lane_id() == 0)
    for (int c = 0; c < 4; ++c) sred[c][threadIdx.x >> 6] = v[c];
  __syncthreads();
  if (threadIdx.x < 4) {
    unsigned long long t = 0;
    for (int w = 0; w < kFinishThreads / 64; ++w) t += sred[threadIdx.x][w];
    unsigned long long* to[4] = {&stats->segments_examined, &stats->paths_invalid, &stats->paths_light_lost,
                                 &stats->verify_box_hits};
    unsigned long long* at = to[0];
    for (uint32_t c = 1; c < 4; ++c) at = threadIdx.x == c ? to[c] : at;
    if (t) atomicAdd(at, t);
  }
}

// ---------------------------------------------------------------------------
// exclusive scan of n counts by one block of 1024 threads; total -> *total

__global__ __launch_bounds__(1024) void k_scan(const uint32_t* __restrict__ in, uint32_t* __restrict__ out, uint32_t n,
                                               uint32_t* total) {
  __shared__ uint32_t wsum[16];
  __shared__ uint32_t carry_sh;
  if (threadIdx.x == 0) carry_sh = 0;
  __syncthreads();
  for (uint32_t base = 0; base < n; base += 1024) {
    uint32_t i = base + threadIdx.x;
    uint32_t v = i < n ? in[i] : 0u;
    // inclusive wave scan
    uint32_t x = v;
    for (int o = 1; o < 64; o <<= 1) {
      uint32_t y = __shfl_up(x, o, 64);
      if ((int)lane_id() >= o) x += y;
    }
    if (lane_id() == 63) wsum[threadIdx.x >> 6] = x;
    __syncthreads();
    if (threadIdx.x < 16) {
      uint32_t s = wsum[threadIdx.x];
      for (int o = 1; o < 16; o <<= 1) {
        uint32_t y = __shfl_up(s, o, 64);
        if ((int)threadIdx.x >= o) s += y;
      }
      wsum[threadIdx.x] = s;  // inclusive over waves
    }
    __syncthreads();
    uint32_t wpre = (threadIdx.x >> 6) ? wsum[(threadIdx.x >> 6) - 1] : 0u;
    uint32_t carry = carry_sh;
    if (i < n) out[i] = carry + wpre + x - v;
    __syncthreads();
    if (threadIdx.x == 0) carry_sh = carry + wsum[15];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    *total = carry_sh;
  }
}

// Exclusive scan of count arrays: each block scans a tile of kScanTile
// entries, kScanPer rows of 1024 read and written coalesced (row k of the tile
// is entries k * 1024 .. k * 1024 + 1023).  Every row is scanned within its
// waves, then one pass over the (row, wave) totals in entry order gives each
// wave its offset.  One tile (the per-tile counts of a few million paths) is
// the whole scan in one launch; longer arrays add k_scan over the tile totals
// and k_scan_add.
constexpr uint32_t kScanPer = 16;
constexpr uint32_t kScanTile = 1024 * kScanPer;

// total of the scan tiles before tile 'tiles' (called by whole waves)
__device__ inline uint32_t scan_tile_offset(const uint32_t* __restrict__ sums, uint32_t tiles) {
  uint32_t v = 0;
  for (uint32_t t = lane_id(); t < tiles; t += 64) v += sums[t];
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}

__global__ __launch_bounds__(1024) void k_scan_tiles(const uint32_t* __restrict__ in, uint32_t* __restrict__ out,
                                                     uint32_t n, uint32_t* __restrict__ tile_sums) {
  static_assert(kScanPer * 16 == 256, "four waves scan the (row, wave) totals");
  __shared__ uint32_t part[kScanPer * 16];  // (row, wave) totals, then their exclusive offsets
  __shared__ uint32_t qsum[4];
  const uint32_t tid = threadIdx.x, wave = tid >> 6, lane = lane_id();
  const uint32_t base = blockIdx.x * kScanTile + tid;
  uint32_t v[kScanPer], x[kScanPer];
#pragma unroll
  for (uint32_t k = 0; k < kScanPer; ++k) {
    const uint32_t i = base + k * 1024;
    v[k] = i < n ? in[i] : 0u;
    x[k] = v[k];
  }
  for (int o = 1; o < 64; o <<= 1) {
#pragma unroll
    for (uint32_t k = 0; k < kScanPer; ++k) {
      const uint32_t y = __shfl_up(x[k], o, 64);
      if ((int)lane >= o) x[k] += y;
    }
  }
  if (lane == 63) {
#pragma unroll
    for (uint32_t k = 0; k < kScanPer; ++k) part[k * 16 + wave] = x[k];
  }
  __syncthreads();
  uint32_t a = 0, q = 0;
  if (tid < 256) {
    a = part[tid];
    q = a;
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(q, o, 64);
      if ((int)lane >= o) q += y;
    }
    if (lane == 63) qsum[wave] = q;
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t pre = 0;
    for (uint32_t w = 0; w < wave; ++w) pre += qsum[w];
    part[tid] = pre + q - a;
  }
  if (tid == 0) tile_sums[blockIdx.x] = qsum[0] + qsum[1] + qsum[2] + qsum[3];
  __syncthreads();
#pragma unroll
  for (uint32_t k = 0; k < kScanPer; ++k) {
    const uint32_t i = base + k * 1024;
    if (i < n) out[i] = part[k * 16 + wave] + x[k] - v[k];
  }
}

__global__ __launch_bounds__(256) void k_scan_add(uint32_t* __restrict__ out, uint32_t n,
                                                  const uint32_t* __restrict__ tile_off) {
  uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) out[i] += tile_off[i / kScanTile];
}

// full invalidation: every path replace=1, start=0, reuse_light=0; queue = all
__global__ __launch_bounds__(kBlock) void k_mark_all(const SceneDev* __restrict__ scenes, const uint2* __restrict__ tiles,
                                                     uint32_t* __restrict__ queue, uint32_t* __restrict__ qcount) {
  const uint2 tile = tiles[blockIdx.x];
  const SceneDev& S = scenes[tile.x];
  const uint32_t p = tile.y + threadIdx.x;
  if (blockIdx.x == 0 && threadIdx.x == 0) *qcount = S.n_paths;
  if (p >= S.n_paths) return;
  const uint32_t w = S.info[p];
  S.info[p] = info_pack(info_cell(w), info_nseg(w), 0, 1, 0);
  queue[p] = p;
}

// The work queue: ascending global path ids with the replace bit, and the same
// ids in the order in which the re-trace takes them.  A path's re-trace costs
// up to one ray per segment from its first invalid one on, so the persistent
// re-trace kernel is given the paths by that segment, smallest first (a stable
// counting sort over kOrderBuckets buckets): the refills deal the long paths
// first and the last refills of a launch are short paths, so the waves finish
// closer together.  Two launches over chunks of kChunkTiles path tiles: counts
// per bucket and chunk, then the scatter of both lists.  For up to
// kInlineChunks chunks every workgroup of the scatter sums the counts itself
// (at most 32 KB from L2, less than the 5 us of another launch; twice as many
// chunks made the scatter 5 us longer); else it adds the tiles' totals to the
// offsets of a scan in tiles ('hoff', 'sums').
constexpr int kOrderBuckets = 8;
constexpr uint32_t kChunkTiles = 4;
constexpr uint32_t kInlineChunks = 1024;

__device__ inline uint32_t order_bucket(uint32_t w, uint32_t B) {
  const uint32_t n = min(info_nseg(w), B), k = info_start(w);
  return min(k < n ? k : 0u, (uint32_t)kOrderBuckets - 1u);  // k >= n: a new light sample, a full path
}

// lanes of the wave with the same bucket as this one
__device__ inline uint64_t bucket_peers(bool valid, uint32_t b) {
  static_assert(kOrderBuckets == 8, "three bucket bits");
  uint64_t peers = __ballot(valid);
  for (int bit = 0; bit < 3; ++bit) {
    const bool set = ((b >> bit) & 1u) != 0;
    const uint64_t m = __ballot(valid && set);
    peers &= set ? m : ~m;
  }
  return peers;
}

// counts of one chunk, bucket-major (hist[bucket * stride + chunk])
__global__ __launch_bounds__(kBlock) void k_queue_hist(const SceneDev* __restrict__ scenes,
                                                       const uint2* __restrict__ tiles, uint32_t n_tiles,
                                                       uint32_t* __restrict__ hist, uint32_t stride) {
  __shared__ uint32_t h[kOrderBuckets];
  if (threadIdx.x < kOrderBuckets) h[threadIdx.x] = 0;
  uint32_t w[kChunkTiles], B[kChunkTiles];
#pragma unroll
  for (uint32_t i = 0; i < kChunkTiles; ++i) {
    const uint32_t t = blockIdx.x * kChunkTiles + i;
    w[i] = 0;
    B[i] = 0;
    if (t < n_tiles) {
      const uint2 tile = tiles[t];
      const SceneDev& S = scenes[tile.x];
      const uint32_t p = tile.y + threadIdx.x;
      B[i] = S.B;
      if (p < S.n_paths) w[i] = G(S.info)[p];
    }
  }
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kChunkTiles; ++i) {
    const bool f = info_replace(w[i]) != 0;
    const uint32_t b = order_bucket(w[i], B[i]);
    const uint64_t peers = bucket_peers(f, b);
    if (f && (peers & lanemask_lt()) == 0) atomicAdd(&h[b], (uint32_t)__popcll(peers));
  }
  __syncthreads();
  if (threadIdx.x < kOrderBuckets) hist[threadIdx.x * stride + blockIdx.x] = h[threadIdx.x];
}

__global__ __launch_bounds__(kBlock) void k_queue_scatter(const SceneDev* __restrict__ scenes,
                                                          const uint2* __restrict__ tiles, uint32_t n_tiles,
                                                          const uint32_t* __restrict__ hist,
                                                          const uint32_t* __restrict__ hoff,
                                                          const uint32_t* __restrict__ sums, uint32_t stride,
                                                          uint32_t* __restrict__ queue, uint32_t* __restrict__ ordered,
                                                          uint32_t* __restrict__ qcount) {
  constexpr uint32_t kWaves = kBlock / 64, kCells = kChunkTiles * kWaves;
  __shared__ uint32_t tot[kOrderBuckets], bef[kOrderBuckets];  // entries of a bucket: all, in earlier chunks
  __shared__ uint32_t cell[kCells][kOrderBuckets + 1];         // counts per (tile, wave): buckets, all; then offsets
  const uint32_t tid = threadIdx.x, wv = tid >> 6, chunk = blockIdx.x;
  uint32_t w[kChunkTiles], gp[kChunkTiles], bk[kChunkTiles];
#pragma unroll
  for (uint32_t i = 0; i < kChunkTiles; ++i) {
    const uint32_t t = chunk * kChunkTiles + i;
    w[i] = 0;
    gp[i] = 0;
    bk[i] = 0;
    if (t < n_tiles) {
      const uint2 tile = tiles[t];
      const SceneDev& S = scenes[tile.x];
      const uint32_t p = tile.y + tid;
      gp[i] = S.gpath_base + p;
      bk[i] = S.B;
      if (p < S.n_paths) w[i] = G(S.info)[p];
    }
  }
  // totals and earlier chunks of two buckets per wave
  for (uint32_t b = 2 * wv; b < 2 * wv + 2; ++b) {
    uint32_t all = 0, before = 0;
    if (hoff) {
      // exclusive scan over all buckets: a bucket's entries start at its first
      all = hoff[b * stride] + scan_tile_offset(sums, b * stride / kScanTile);
      before = hoff[b * stride + chunk] + scan_tile_offset(sums, (b * stride + chunk) / kScanTile) - all;
    } else {
      const uint4* h4 = reinterpret_cast<const uint4*>(hist + (size_t)b * stride);
#pragma unroll 4
      for (uint32_t q = lane_id(); q < stride / 4; q += 64) {
        const uint4 v = h4[q];
        all += v.x + v.y + v.z + v.w;
        const uint32_t c = 4 * q;
        before += (c < chunk ? v.x : 0u) + (c + 1 < chunk ? v.y : 0u) + (c + 2 < chunk ? v.z : 0u) +
                  (c + 3 < chunk ? v.w : 0u);
      }
      for (int o = 32; o > 0; o >>= 1) {
        all += __shfl_xor(all, o, 64);
        before += __shfl_xor(before, o, 64);
      }
    }
    if (lane_id() == 0) {
      tot[b] = all;
      bef[b] = before;
    }
  }
  uint32_t rank[kChunkTiles], qrank[kChunkTiles];
  for (uint32_t i = tid; i < kCells * (kOrderBuckets + 1); i += kBlock) (&cell[0][0])[i] = 0;
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kChunkTiles; ++i) {
    const bool f = info_replace(w[i]) != 0;
    bk[i] = order_bucket(w[i], bk[i]);
    const uint64_t peers = bucket_peers(f, bk[i]), all = __ballot(f);
    rank[i] = (uint32_t)__popcll(peers & lanemask_lt());
    qrank[i] = (uint32_t)__popcll(all & lanemask_lt());
    if (f && rank[i] == 0) cell[i * kWaves + wv][bk[i]] = (uint32_t)__popcll(peers);
    if (lane_id() == 0) cell[i * kWaves + wv][kOrderBuckets] = (uint32_t)__popcll(all);
  }
  __syncthreads();
  // offsets of the cells: a thread per bucket, and one for the whole queue
  if (tid <= (uint32_t)kOrderBuckets) {
    uint32_t at = 0;
    if (tid < (uint32_t)kOrderBuckets) {
      at = bef[tid];
      if (hoff)
        at += tot[tid];
      else
        for (uint32_t b = 0; b < tid; ++b) at += tot[b];
    } else {
      for (uint32_t b = 0; b < (uint32_t)kOrderBuckets; ++b) at += bef[b];
    }
    uint32_t v[kCells];
#pragma unroll
    for (uint32_t c = 0; c < kCells; ++c) v[c] = cell[c][tid];
#pragma unroll
    for (uint32_t c = 0; c < kCells; ++c) {
      cell[c][tid] = at;
      at += v[c];
    }
    // the last chunk's end is the length of the queue
    if (tid == (uint32_t)kOrderBuckets && chunk == gridDim.x - 1) *qcount = at;
  }
  __syncthreads();
#pragma unroll
  for (uint32_t i = 0; i < kChunkTiles; ++i) {
    if (!info_replace(w[i])) continue;
    const uint32_t c = i * kWaves + wv;
    queue[cell[c][kOrderBuckets] + qrank[i]] = gp[i];
    ordered[cell[c][bk[i]] + rank[i]] = gp[i];
  }
}

// ---------------------------------------------------------------------------
// re-tracing (Section 3.2 naive, Section 3.3 / Algorithm 1 error-based)

constexpr float kTFar = 16.0f;

__device__ inline float3 tri_vertex(const PV_GLOBAL Tri* t, int i) { return f3(t->v[i][0], t->v[i][1], t->v[i][2]); }

__device__ inline float3 hit_normal(const SceneDev& S, const Hit& h) {
  const PV_GLOBAL Tri* t = G(S.tris) + h.rec;
  const float3 v0 = tri_vertex(t, 0), v1 = tri_vertex(t, 1), v2 = tri_vertex(t, 2);
  float3 n = cross(sub(v1, v0), sub(v2, v0));
  return mul(n, 1.0f / length(n));
}

__device__ inline float3 vertex(const SceneDev& S, uint32_t p, uint32_t j) {
  const size_t stride = S.stride;
  const PV_GLOBAL float* org = G(S.origin);
  if (j == 0) return f3(org[p], org[stride + p], org[2 * stride + p]);
  return xyz(G(S.pos)[(size_t)(j - 1) * stride + p]);
}

__device__ inline uint32_t vertex_hit(const SceneDev& S, uint32_t p, uint32_t j) {
  return __float_as_uint(G(S.pos)[(size_t)(j - 1) * S.stride + p].w);
}

__device__ inline float3 energy_row(const SceneDev& S, uint32_t p, uint32_t row) {
  return xyz(G(S.energy)[(size_t)row * S.stride + p]);
}

__device__ inline void put_photon(const SceneDev& S, uint32_t p, uint32_t row, float3 x, uint32_t gid, float3 e) {
  size_t i = (size_t)row * S.stride + p;
  G(S.pos)[i] = make_float4(x.x, x.y, x.z, __uint_as_float(gid));
  G(S.energy)[i] = make_float4(e.x, e.y, e.z, S.radius);
}

// material of a stored hit id (ids beyond the scene map to material 0)
__device__ inline uint32_t mat_of(const SceneDev& S, uint32_t hit) {
  return hit < S.n_tris_total ? G(S.tri_mat)[hit] : 0u;
}

__device__ inline float3 reflect_energy(const SceneDev& S, float3 e, uint32_t mat) {
  const PV_GLOBAL float* rho = G(S.albedo) + 3 * mat;
  return f3(__fmul_rn(e.x, rho[0]), __fmul_rn(e.y, rho[1]), __fmul_rn(e.z, rho[2]));
}

// a . b with the order of its roundings spelled out, x's or y's product rounded
// first: what Equation 2 compares may lie within a rounding of its threshold,
// where a product contracted another way decides another way
__device__ inline float dot_x(float3 a, float3 b) { return fmaf(a.z, b.z, fmaf(a.y, b.y, a.x * b.x)); }
__device__ inline float dot_y(float3 a, float3 b) { return fmaf(a.z, b.z, fmaf(a.x, b.x, a.y * b.y)); }

__device__ inline bool eq2(float3 en, float3 eo, float T) {
  float d0 = __fsub_rn(en.x, eo.x), d1 = __fsub_rn(en.y, eo.y), d2 = __fsub_rn(en.z, eo.z);
  float t0 = __fmul_rn(T, eo.x), t1 = __fmul_rn(T, eo.y), t2 = __fmul_rn(T, eo.z);
  return (-t0 <= d0 && d0 <= t0) && (-t1 <= d1 && d1 <= t1) && (-t2 <= d2 && d2 <= t2);
}

__device__ inline bool on_moved_obj(const SceneDev& S, uint32_t hit) {
  if (hit == kHitNone || hit < S.n_static) return false;
  for (uint32_t o = 0; o < S.n_obj; ++o) {
    const ObjDev ob = G(S.objs)[o];
    if (hit - ob.gbase < ob.n_tris) return G(S.obj_moved)[o] != 0;
  }
  return false;
}

// Object id ranges, moved flags and light path ranges of the scene of a
// single-scene launch, staged in LDS once per workgroup for the state
// machine's lookups.
struct SceneTab {
  uint32_t obj_lo[PV_MAX_OBJECTS], obj_n[PV_MAX_OBJECTS], obj_mv[PV_MAX_OBJECTS];
  uint32_t light_base[PV_MAX_LIGHTS], light_n[PV_MAX_LIGHTS];
  uint32_t n_obj, n_lights;
};

__device__ inline void load_tab(const SceneDev& S, SceneTab& T) {
  const uint32_t i = threadIdx.x;
  if (i < S.n_obj) {
    const ObjDev ob = G(S.objs)[i];
    T.obj_lo[i] = ob.gbase;
    T.obj_n[i] = ob.n_tris;
    T.obj_mv[i] = G(S.obj_moved)[i];
  }
  if (i < S.n_lights) {
    T.light_base[i] = G(S.lights)[i].path_base;
    T.light_n[i] = G(S.lights)[i].path_count;
  }
  if (i == 0) {
    T.n_obj = S.n_obj;
    T.n_lights = S.n_lights;
  }
  __syncthreads();
}

__device__ inline bool on_moved_obj(const PV_LDS SceneTab& T, uint32_t hit) {
  bool mv = false;  // no early exit: the loop count is uniform
  for (uint32_t o = 0; o < T.n_obj; ++o) mv |= (hit - T.obj_lo[o] < T.obj_n[o]) && T.obj_mv[o] != 0;
  return mv;  // kHitNone and static ids lie in no object range
}

__device__ inline int light_of(const PV_LDS SceneTab& T, uint32_t p) {
  int l = -1;
  for (uint32_t i = 0; i < T.n_lights; ++i) l = (p - T.light_base[i] < T.light_n[i]) ? (int)i : l;
  return l;
}

__device__ inline void clear_rows(const SceneDev& S, uint32_t p, uint32_t from) {
  for (uint32_t r = from; r < S.B; ++r) {
    size_t i = (size_t)r * S.stride + p;
    G(S.pos)[i] = make_float4(0.0f, 0.0f, 0.0f, __uint_as_float(kHitNone));
    G(S.energy)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  }
}

__device__ inline float3 normalize3(float3 v) { return mul(v, 1.0f / length(v)); }


// Bound by vector issue (90% of a full trace's cycles at five waves per SIMD)
// and, as much, by the vector memory path (texture addresser 85% busy, a cycle
// per lane and load, its data return 96%); a 3M-path partial re-trace by the
// latter (77%, 75%, 94%, 39% of the lanes active), a list of 45k paths by neither
// (49%, 39%, 63%): with 11% of its lanes active it waits for its longest paths.
// 96 registers hold five waves without a spill (the batch form spills 6) because
// little outlives a walk (struct Lane); sampling, hit normals, photon writes and path ends are shared
// by the modes that need them, since a wave holds lanes of several modes at
// once and would run each mode's copy in turn.  Measured over the 3M-path,
// 380k-triangle interior, one MI355X: full trace 4.08 ms against 4.85 with a
// copy per mode, all of a path's state kept and four waves, partial re-trace
// 1.63 against 1.98 ms; now 3.39 and 1.45 ms with what the walk gained since.
//
// Re-trace state machine: every iteration each busy lane issues exactly one
// query (closest hit over the scene, or any hit against the moved objects),
// then advances its path; lanes whose path is finished take the next path of
// the work queue (persistent while-while scheme, Aila & Laine 2009).
enum : uint32_t {
  ST_IDLE = 0,   // needs a path
  ST_LIGHT,      // draw a new light sample and trace its ray
  ST_DIR,        // trace from x along w, naive continuation
  ST_TAIL,       // sample a bounce at x and trace it
  ST_WCHECK,     // walk: is segment j (origin unchanged) still valid?
  ST_WTRACE,     // walk: trace segment j
  ST_WSKIP,      // walk: accepted close re-hit; is segment j+1 clear?
  ST_END         // queue exhausted
};

// What a lane keeps while its query is walked: its path, the packed state, and
// four words whose meaning follows from the mode.  Everything else (the
// vertex, its normal, the material) is used up when the next query is set up,
// in the same round of the loop, so that it takes no registers during walks.
struct Lane {
  uint32_t s;  // scene of a batch
  uint32_t p;
  // mode, j (walk: segment), newn (photons the path will have), row1 (photon
  // that the ray of ST_LIGHT, ST_DIR or ST_TAIL writes): 4 bits each
  uint32_t st;
  // ST_DIR and ST_TAIL: energy arriving at x and its material (ST_LIGHT, and
  // ST_DIR from the light: the energy of the first photon); ST_WSKIP: the
  // accepted re-hit and its triangle
  float3 e;
  uint32_t mat;
};

__device__ inline uint32_t lane_mode(uint32_t st) { return st & 15u; }
__device__ inline uint32_t lane_j(uint32_t st) { return (st >> 4) & 15u; }
__device__ inline uint32_t lane_newn(uint32_t st) { return (st >> 8) & 15u; }
__device__ inline uint32_t lane_row1(uint32_t st) { return st >> 12; }
__device__ inline uint32_t lane_state(uint32_t mode, uint32_t j, uint32_t newn, uint32_t row1) {
  return mode | (j << 4) | (newn << 8) | (row1 << 12);
}

// A queued path's first query: its mode, and for ST_DIR the vertex x and the
// direction w.  A path without the replace bit stays idle.
__device__ inline void start_path(const SceneDev& S, Lane& L, float T, const PV_LDS SceneTab* tab, float3* x,
                                  float3* wd) {
  const uint32_t w = G(S.info)[L.p];
  const uint32_t n = min(info_nseg(w), S.B);
  uint32_t k = info_start(w);
  const int l = tab ? light_of(*tab, L.p) : light_of(S, L.p);
  bool reuse = info_reuse(w) != 0;
  if (!info_replace(w) || l < 0) {
    L.st = ST_IDLE;
    return;
  }
  if (k >= n) {
    k = 0;
    reuse = false;
  }
  if (k == 0) {
    const PV_GLOBAL LightDev* lt = G(S.lights) + l;
    L.e = f3(lt->e1[0], lt->e1[1], lt->e1[2]);
  }
  if (k == 0 && !reuse) {
    L.st = lane_state(ST_LIGHT, 0, 0, 0);
  } else if (T < 0.0f) {
    *x = vertex(S, L.p, k);
    *wd = normalize3(sub(vertex(S, L.p, k + 1), *x));
    if (k > 0) {
      L.e = energy_row(S, L.p, k - 1);
      L.mat = mat_of(S, vertex_hit(S, L.p, k));
    }
    L.st = lane_state(ST_DIR, 0, 0, k);
  } else {
    // After the triangle test segment k is known to be blocked.  After the
    // box test it only reached a moved object's box, and Section 3.3 casts no
    // ray for a segment that the box crosses but no triangle: with its origin
    // unchanged the walk first checks it against the moved triangles.
    const bool origin_moved = k == 0 && G(S.light_moved)[l] != 0;
    L.st = lane_state((S.verify_boxes && !origin_moved) ? ST_WCHECK : ST_WTRACE, k, n, 0);
  }
}

// The ray of a sampled vertex: a new light sample (position uniform on the
// rectangle, direction cosine-weighted about the light normal, Philox tag 0)
// or a diffuse bounce about n at x (tag 1).  Both draw here, so that lanes
// starting a path share the draw and the disk map with the lanes that bounce.
// Sets x and the stored origin for a light sample; returns the direction.
__device__ inline float3 sample_ray(const SceneDev& S, const Lane& L, uint64_t seed, uint32_t frame,
                                    const PV_LDS SceneTab* tab, float3* x, float3 n) {
  const bool light = lane_mode(L.st) == ST_LIGHT;
  float u[4];
  draw4(seed, L.p, frame, light ? 0u : lane_row1(L.st), light ? 0u : 1u, u);
  float3 lc = cosine_local(light ? u[2] : u[0], light ? u[3] : u[1]);
  float3 tt, bb, nn = n;
  float3 w = f3(0.0f, 0.0f, 0.0f);
  bool done = false;
  if (light) {
    const int l = tab ? light_of(*tab, L.p) : light_of(S, L.p);
    const PV_GLOBAL float* xf = G(S.light_xf_cur) + 12 * l;
    tt = f3(xf[0], xf[4], xf[8]);
    bb = f3(xf[1], xf[5], xf[9]);
    nn = normalize3(f3(xf[2], xf[6], xf[10]));
    const float3 c = f3(xf[3], xf[7], xf[11]);
    const LightDev ld = G(S.lights)[l];
    float3 x0;
    if (S.dm[0] > 0) {
      // distribution maps: the sample is drawn inside the path's cell
      dm_sample((const float*)xf, ld, S.dm, info_cell(G(S.info)[L.p]), u, &x0, &w);
      done = true;
    } else if (ld.kind == PV_LIGHT_CAMERA) {
      // uniform over the near plane at unit distance
      const float px = (2.0f * u[0] - 1.0f) * ld.param[0], py = (2.0f * u[1] - 1.0f) * ld.param[1];
      x0 = c;
      w = mul(add(add(mul(tt, px), mul(bb, py)), nn), 1.0f / sqrtf(px * px + py * py + 1.0f));
      done = true;
    } else {
      const float a = (2.0f * u[0] - 1.0f) * ld.half[0], b = (2.0f * u[1] - 1.0f) * ld.half[1];
      x0 = add(c, add(mul(tt, a), mul(bb, b)));
      if (ld.kind == PV_LIGHT_SPOT) {
        // the disk point scaled to the cone's radius, then lifted: with the
        // unit disk's height z0, 1 - sr^2 r^2 = cos^2 + sr^2 z0^2 (no
        // cancellation near the cone's rim)
        const float sr = sqrtf((1.0f - ld.param[0]) * (1.0f + ld.param[0]));
        const float z0 = lc.z;
        lc.x *= sr;
        lc.y *= sr;
        lc.z = sqrtf(ld.param[0] * ld.param[0] + (sr * sr) * (z0 * z0));
      }
    }
    const size_t stride = S.stride;
    PV_GLOBAL float* org = G(S.origin);
    org[L.p] = x0.x;
    org[stride + L.p] = x0.y;
    org[2 * stride + L.p] = x0.z;
    *x = x0;
  } else {
    onb(nn, &tt, &bb);
  }
  const float3 q = add(add(mul(tt, lc.x), mul(bb, lc.y)), mul(nn, lc.z));
  return done ? w : q;
}

template <bool kSingle, bool kScaled>
__device__ __forceinline__ void retrace_loop(const SceneDev* __restrict__ scenes, const uint32_t* __restrict__ gbase,
                                             int n_scenes, const uint32_t* __restrict__ queue,
                                             const uint32_t* __restrict__ qcount, float T, uint64_t seed,
                                             uint32_t frame, const PV_LDS SceneTab* tab, uint32_t* scount,
                                             pv_stats* stats, int min_active, uint32_t entries, uint32_t spread_waves,
                                             uint32_t* __restrict__ deal_ctr) {
  extern __shared__ int32_t sstack[];  // traversal stacks, launch-time size
  const StackCol col = (StackCol)(sstack + kBlock + threadIdx.x);  // entry 0 of the column; entry -1 spare
  const StackCol limit = col + (int)(entries - 5) * kBlock;  // top from which a full node would pass the last entry
  uint32_t n_rays = 0, n_photons = 0, n_acc = 0, n_trunc = 0;  // of the wave
  const float3 base0 = scene_base<kScaled>(scenes[0]);
  // the work queue, dealt by deal() from the counters 'deal_ctr'
  const uint32_t count = *qcount;
  const uint32_t wave = blockIdx.x * (kBlock / 64) + (threadIdx.x >> 6);
  const uint32_t quota = wave_quota(count, spread_waves);
  if (quota < 64) min_active = max(1, (int)(quota * (uint32_t)min_active / 64u));
  bool fresh = true;  // this wave has not taken its share of a spread queue
  Lane L;
  L.s = 0;
  L.st = ST_IDLE;
  L.p = 0;
  L.e = f3(0.0f, 0.0f, 0.0f);
  L.mat = 0;
  Ray r;             // the lane's current query
  Walk wk;           // its walk through the hierarchy
  wk.cur = kRootNone;
  wk.leaf = 0;
  bool tracing = false, any = false;
  bool drained = false;  // the wave has asked for work in vain
  while (true) {
    const SceneDev& S = scenes[kSingle ? 0u : L.s];
    // ---- walk; the box-test parameters follow from the ray, a few
    // instructions beside the walk's thousands, and hold no registers outside
    const int yield = yield_below(min_active, drained, (int)__popcll(__ballot(tracing)));
    if (tracing) {
      const float3 c = sub(kSingle ? base0 : plane_base<kScaled>(S), ray_origin(r));
      const Slab q = world_slab(S, c, rcp3(r.d), r.tmin);
      if (walk_far(S, c)) walk_leave(wk);
      walk_scene<true, kScaled>(S, r, q, any, col, limit, wk, yield);
    }
    // ---- lanes whose walk is finished advance their path.  What several
    // modes share is done once for all of them: the new vertex with its
    // normal and material before the switch, the photon written, the start
    // of a tail and the end of a path after it
    float3 x = f3(0.0f, 0.0f, 0.0f), nw = x;  // ST_DIR: vertex, direction; ST_TAIL: vertex, normal
    bool write = false, accepted = false, cut = false;
    if (tracing && walk_done(wk)) {
      tracing = false;
      if (wk.redo && !(any && wk.rec != kRecNone))
        walk_exact(G(S.nodes), G(S.tris), r, any ? 1.0f - r.tmin : kTFar, G(S.top)[any ? 1 : 0], any, col, wk);
      Hit h;
      h.t = wk.tb;
      h.rec = wk.rec;
      const bool hit = h.rec != kRecNone;
      h.gid = kHitNone;
      const float3 qd = r.d, xa = ray_origin(r);
      float3 nh = x, en = x;
      uint32_t mat = 0, row = 0;
      if (hit && !any) {
        x = add(xa, mul(qd, h.t));
        nh = hit_normal(S, h);
        h.gid = G(S.tris)[h.rec].gid;
        mat = G(S.rec_mat)[h.rec];
      }
      uint32_t mode = lane_mode(L.st), j = lane_j(L.st), newn = lane_newn(L.st);
      bool tail = false;  // the photon written is followed by sampled bounces
      bool end = false;   // the path ends with newn photons
      uint32_t hgid = h.gid;
      switch (mode) {
        case ST_LIGHT:
        case ST_DIR:
        case ST_TAIL: {
          row = lane_row1(L.st);
          if (!hit) {
            cut = end = true;
            newn = row;
            break;
          }
          en = row == 0 ? L.e : reflect_energy(S, L.e, L.mat);
          write = tail = true;
          break;
        }
        case ST_WCHECK: {
          if (hit)
            mode = ST_WTRACE;
          else
            end = ++j >= newn;
          break;
        }
        case ST_WTRACE: {
          if (!hit) {
            cut = end = true;
            newn = j;
            break;
          }
          en = energy_row(S, L.p, j);
          row = j;
          write = true;
          if (j == newn - 1) {
            end = true;
            break;
          }
          float3 xc = vertex(S, L.p, j + 2);
          float3 d2 = sub(xc, x);
          float c1 = dot_y(qd, nh), l2 = sqrtf(dot_x(d2, d2));
          float c2 = l2 > 0.0f ? dot_y(d2, nh) / l2 : 0.0f;
          float3 eN = (c1 * c2 < 0.0f) ? reflect_energy(S, en, mat) : f3(0.0f, 0.0f, 0.0f);
          if (S.energy_test == PV_ENERGY_COSINE_RATIO && c1 * c2 < 0.0f) {
            // the kept direction's cosine at the new vertex over the one at the
            // old vertex (its stored triangle, from x_{j+1} to x_{j+2})
            const PV_GLOBAL Tri* to = G(S.tris) + G(S.gid_rec)[vertex_hit(S, L.p, j + 1)];
            const float3 o0 = tri_vertex(to, 0);
            const float3 no = cross(sub(tri_vertex(to, 1), o0), sub(tri_vertex(to, 2), o0));
            const float3 d3 = sub(xc, vertex(S, L.p, j + 1));
            const float den = fabsf(dot_x(d3, no));
            const float num = fabsf(c2) * sqrtf(dot_x(d3, d3)) * sqrtf(dot_y(no, no));
            const float ratio = den > 0.0f ? num / den : 0.0f;
            eN = mul(eN, ratio);
          }
          float3 eo = energy_row(S, L.p, j + 1);
          if (!eq2(eN, eo, T)) {
            // energies differ: keep the new hit and re-sample the rest
            tail = true;
            break;
          }
          accepted = true;
          const float3 step = sub(x, vertex(S, L.p, j + 1));
          float dist = sqrtf(dot_x(step, step));
          auto moved = [&](uint32_t id) { return tab ? on_moved_obj(*tab, id) : on_moved_obj(S, id); };
          if (dist <= S.eps_close && !moved(h.gid) && !moved(vertex_hit(S, L.p, j + 1)) &&
              !moved(vertex_hit(S, L.p, j + 2))) {
            L.e = x;
            L.mat = h.gid;
            mode = ST_WSKIP;  // the next segment must also be clear
            write = false;
            break;
          }
          ++j;
          break;
        }
        case ST_WSKIP: {
          if (!hit) {
            j += 2;
            end = j >= newn;
            mode = ST_WCHECK;
          } else {
            en = energy_row(S, L.p, j);
            row = j;
            x = L.e;
            hgid = L.mat;
            write = true;
            ++j;
            mode = ST_WTRACE;
          }
          break;
        }
        default:
          break;
      }
      if (write) put_photon(S, L.p, row, x, hgid, en);
      if (tail) {
        // continue sampling from photon 'row' on the side the ray came from,
        // or finish
        nw = dot(nh, qd) > 0.0f ? mul(nh, -1.0f) : nh;
        L.mat = mat;
        L.e = en;
        mode = ST_TAIL;
        newn = row + 1;
        end = row + 1 >= S.B;
      }
      L.st = lane_state(mode, j, newn, row + 1);
      if (end) {
        clear_rows(S, L.p, newn);
        G(S.info)[L.p] = info_pack(info_cell(G(S.info)[L.p]), newn, 0, 0, 0);
        L.st = ST_IDLE;
      }
    }
    n_photons += (uint32_t)__popcll(__ballot(write));
    n_acc += (uint32_t)__popcll(__ballot(accepted));
    n_trunc += (uint32_t)__popcll(__ballot(cut));
    // ---- idle lanes take the next paths of the queue
    const bool want = lane_mode(L.st) == ST_IDLE;
    if (__ballot(want)) {
      uint32_t qi;
      if (quota < 64) {
        const uint32_t e = wave * quota + lane_id();
        qi = fresh && lane_id() < quota && e < count ? e : kNoEntry;
        fresh = false;
      } else {
        qi = deal(deal_ctr, wave, count, want);
      }
      if (want) {
        if (qi != kNoEntry) {
          uint32_t gp = G(queue)[qi];
          if (kSingle) {
            L.p = gp;
          } else {
            L.s = scene_of(gbase, n_scenes, gp);
            L.p = gp - gbase[L.s];
          }
          // a path without the replace bit is skipped (stays idle this round)
          start_path(scenes[kSingle ? 0u : L.s], L, T, tab, &x, &nw);
        } else {
          L.st = ST_END;
        }
      }
    }
    const uint32_t mode = lane_mode(L.st);
    drained = __ballot(mode == ST_END) != 0;
    if (__ballot(mode != ST_END && mode != ST_IDLE) == 0) {
      if (__ballot(mode == ST_IDLE) == 0) break;
      continue;
    }
    // ---- lanes with a path and no walk in progress start their next query
    const bool start = !tracing && mode != ST_IDLE && mode != ST_END;
    if (start) {
      const SceneDev& Q = scenes[kSingle ? 0u : L.s];
      any = false;
      float3 qd = nw;  // ST_DIR
      float tmin = Q.eps_end, tmax = kTFar;
      if (mode == ST_LIGHT || mode == ST_TAIL) {
        qd = sample_ray(Q, L, seed, frame, tab, &x, nw);
      } else if (mode != ST_DIR) {
        const uint32_t j = lane_j(L.st), sj = mode == ST_WSKIP ? j + 1 : j;
        x = vertex(Q, L.p, sj);
        const float3 xb = vertex(Q, L.p, sj + 1);
        bool trace = mode == ST_WTRACE;
        if (mode == ST_WCHECK && (tab ? on_moved_obj(*tab, vertex_hit(Q, L.p, sj + 1))
                                      : on_moved_obj(Q, vertex_hit(Q, L.p, sj + 1)))) {
          trace = true;
          L.st = lane_state(ST_WTRACE, j, lane_newn(L.st), 0);
        }
        if (trace) {
          qd = normalize3(sub(xb, x));
        } else {
          // any hit of the segment x -> xb against the moved objects
          any = true;
          qd = sub(xb, x);
          float len = length(qd);
          tmin = len > 0.0f ? Q.eps_end / len : 1.0f;
          tmax = 1.0f - tmin;
        }
      }
      r = make_ray(x, qd, tmin);
      walk_start(wk, G(Q.wtop)[any ? 1 : 0], tmax, col);
      tracing = true;
    }
    n_rays += (uint32_t)__popcll(__ballot(start && !any));
  }
  if (quota >= 64) deal_done(deal_ctr);  // uniform over the grid
  if (stats) {
    if (lane_id() == 0) {
      if (n_rays) atomicAdd(&scount[0], n_rays);
      if (n_photons) atomicAdd(&scount[1], n_photons);
      if (n_acc) atomicAdd(&scount[2], n_acc);
      if (n_trunc) atomicAdd(&scount[3], n_trunc);
    }
    __syncthreads();
    // most workgroups of a short queue have nothing to add, and additions to
    // one line serialise: 2048 workgroups' four cost 90 us of a 123 us launch
    // over 2000 paths, and about 50 us of every frame
    if (threadIdx.x < 4 && scount[threadIdx.x]) {
      unsigned long long* to[4] = {&stats->rays_traced, &stats->photons_written, &stats->reuse_accepted,
                                   &stats->paths_truncated};
      atomicAdd(to[threadIdx.x], (unsigned long long)scount[threadIdx.x]);
    }
  }
}

template <bool kSingle, int kWaves>
__global__ __launch_bounds__(kBlock) __attribute__((amdgpu_waves_per_eu(kWaves))) void k_retrace(const SceneDev* __restrict__ scenes, const uint32_t* __restrict__ gbase,
                                                    int n_scenes, const uint32_t* __restrict__ queue,
                                                    const uint32_t* __restrict__ qcount, float T,
                                                    uint64_t seed, uint32_t frame_arg, const uint32_t* frame_ptr,
                                                    pv_stats* stats, int min_active, uint32_t entries,
                                                    uint32_t spread_waves, uint32_t* __restrict__ deal_ctr) {
  __shared__ uint32_t scount[4];
  __shared__ SceneTab stab;
  __shared__ uint32_t sgb[kSingle ? 1 : kLdsScenes + 1];
  const uint32_t frame = frame_ptr ? *frame_ptr : frame_arg;
  if (threadIdx.x < 4) scount[threadIdx.x] = 0;
  const PV_LDS SceneTab* tab = nullptr;
  if (kSingle) {
    load_tab(scenes[0], stab);
    tab = (const PV_LDS SceneTab*)&stab;
  } else {
    gbase = stage_gbase(gbase, n_scenes, sgb);
  }
  __syncthreads();
  if (any_scaled<kSingle>(scenes, n_scenes))
    retrace_loop<kSingle, true>(scenes, gbase, n_scenes, queue, qcount, T, seed, frame, tab, scount, stats, min_active,
                                entries, spread_waves, deal_ctr);
  else
    retrace_loop<kSingle, false>(scenes, gbase, n_scenes, queue, qcount, T, seed, frame, tab, scount, stats, min_active,
                                 entries, spread_waves, deal_ctr);
}

// ---------------------------------------------------------------------------
// compaction of existing photons: counts per (row, block), scan, scatter

__global__ __launch_bounds__(kBlock) void k_photon_count(const SceneDev* __restrict__ scenes, const uint2* __restrict__ tiles,
                                                         uint32_t* __restrict__ counts) {
  __shared__ uint32_t wc[PV_MAX_BOUNCES][kBlock / 64];
  uint2 tile = tiles[blockIdx.x];
  const SceneDev& S = scenes[tile.x];
  uint32_t p = tile.y + threadIdx.x;
  uint32_t n = p < S.n_paths ? min(info_nseg(S.info[p]), S.B) : 0u;
  for (uint32_t r = 0; r < S.B; ++r) {
    uint64_t bal = __ballot(n > r);
    if (lane_id() == 0) wc[r][threadIdx.x >> 6] = (uint32_t)__popcll(bal);
  }
  __syncthreads();
  if (threadIdx.x < S.B) {
    uint32_t c = 0;
    for (int w = 0; w < kBlock / 64; ++w) c += wc[threadIdx.x][w];
    counts[S.count_base + threadIdx.x * S.n_blocks + tile.y / kBlock] = c;
  }
}

// The photons of one (row, path tile) to their place.  Offsets: up to
// kInlineCounts counts, every workgroup sums the counts before its own (at
// most 24 KB from L2, less than a scan launch takes); else the scan's offset
// within its scan tile and the totals of the scan tiles before it.  The
// workgroup of the last count also writes the number of photons, and the
// first one, for a batch, every scene's first photon.
constexpr uint32_t kInlineCounts = 6144;

struct PhotonOffsets {
  const uint32_t* counts;
  const uint32_t* off;   // null: sum the counts
  const uint32_t* sums;  // totals of the scan tiles
  uint32_t n_counts;
  uint32_t* total;
  uint32_t* base;        // null, or [n_scenes + 1]
  int n_scenes;
};

__global__ __launch_bounds__(kBlock) void k_photon_scatter(const SceneDev* __restrict__ scenes, const uint2* __restrict__ tiles,
                                                           PhotonOffsets O, float* __restrict__ out_pos,
                                                           float* __restrict__ out_e, uint32_t capacity) {
  __shared__ uint32_t wcnt[kBlock / 64];
  __shared__ uint32_t sh[kBlock / 64];
  uint32_t r = blockIdx.y;
  uint2 tile = tiles[blockIdx.x];
  const SceneDev& S = scenes[tile.x];
  if (O.base && blockIdx.x == 0 && r == 0) {
    for (int i = threadIdx.x; i <= O.n_scenes; i += kBlock) {
      // a scene's first count; behind the last scene with paths, all photons
      const uint32_t c = i < O.n_scenes ? scenes[i].count_base : O.n_counts;
      const uint32_t k = min(c, O.n_counts - 1);
      uint32_t v = O.off[k] + (c > k ? O.counts[k] : 0u);
      for (uint32_t t = 0; t < k / kScanTile; ++t) v += O.sums[t];
      O.base[i] = v;
    }
  }
  if (r >= S.B) return;
  uint32_t p = tile.y + threadIdx.x;
  bool flag = p < S.n_paths && min(info_nseg(S.info[p]), S.B) > r;
  const uint32_t c = S.count_base + r * S.n_blocks + tile.y / kBlock;
  const uint32_t first = O.off ? O.off[c] + scan_tile_offset(O.sums, c / kScanTile) : block_prefix(O.counts, c, sh);
  uint64_t bal = __ballot(flag);
  if (lane_id() == 0) wcnt[threadIdx.x >> 6] = (uint32_t)__popcll(bal);
  __syncthreads();
  if (c == O.n_counts - 1 && threadIdx.x == 0) *O.total = first + O.counts[c];
  uint32_t pre = 0;
  for (uint32_t w = 0; w < (threadIdx.x >> 6); ++w) pre += wcnt[w];
  if (!flag) return;
  uint32_t idx = first + pre + (uint32_t)__popcll(bal & lanemask_lt());
  if (idx >= capacity) return;
  size_t i = (size_t)r * S.stride + p;
  float4 x = G(S.pos)[i], e = G(S.energy)[i];
  out_pos[3 * (size_t)idx + 0] = x.x;
  out_pos[3 * (size_t)idx + 1] = x.y;
  out_pos[3 * (size_t)idx + 2] = x.z;
  out_e[3 * (size_t)idx + 0] = e.x;
  out_e[3 * (size_t)idx + 1] = e.y;
  out_e[3 * (size_t)idx + 2] = e.z;
}

// ---------------------------------------------------------------------------
// differentiation form

// Three floats of a [..][3] array as one 12-byte access.
struct F3 {
  float x, y, z;
};

// hit ids of a path's rows but the last, all requested before the first is
// used and without waiting for the path's length: rows past its end are in
// bounds (row min(r, B - 1)) and their values unused
template <int kRows>
__device__ inline void load_hits(const SceneDev& S, uint32_t p, uint32_t* hit) {
  const PV_GLOBAL float4* pos = G(S.pos);
#pragma unroll
  for (int r = 0; r + 1 < kRows; ++r)
    hit[r] = __float_as_uint(pos[(size_t)min((uint32_t)r, S.B - 1) * S.stride + p].w);
}

// Deposited energies, one thread per path.  Bound by memory: 16 B of every
// photon row but the last (a hit id takes its row's whole line) and 12 B
// written per slot.  Measured at 1M paths x 7 rows of a 50k-triangle scene,
// one MI355X: 43 us, 4.2 TB/s of row lines and output
// (45 us with the rows read one after another).
template <int kRows>
__global__ __launch_bounds__(kBlock) void k_energy_fwd(const SceneDev* __restrict__ scenes, const uint2* __restrict__ tiles,
                                                       const float* __restrict__ albedo, const float* __restrict__ power,
                                                       float* __restrict__ E) {
  uint2 tile = tiles[blockIdx.x];
  const SceneDev& S = scenes[tile.x];
  uint32_t p = tile.y + threadIdx.x;
  if (p >= S.n_paths) return;
  uint32_t hit[kRows];
  load_hits<kRows>(S, p, hit);
  uint32_t n = min(info_nseg(G(S.info)[p]), S.B);
  int l = light_of(S, p);
  if (l < 0) return;
  float N = (float)S.lights[l].path_count;
  float3 e = f3(__fdiv_rn(power[3 * l], N), __fdiv_rn(power[3 * l + 1], N), __fdiv_rn(power[3 * l + 2], N));
  const size_t np = S.n_paths;
#pragma unroll
  for (int r = 0; r < kRows; ++r) {
    if ((uint32_t)r >= S.B) break;
    F3 o{0.0f, 0.0f, 0.0f};
    if ((uint32_t)r < n) {
      if (r > 0) {
        const uint32_t m = mat_of(S, hit[r - 1]);
        e = f3(__fmul_rn(e.x, albedo[3 * m]), __fmul_rn(e.y, albedo[3 * m + 1]), __fmul_rn(e.z, albedo[3 * m + 2]));
      }
      o = F3{e.x, e.y, e.z};
    }
    *reinterpret_cast<F3*>(E + 3 * ((size_t)r * np + p)) = o;
  }
}

// Gradients, one thread per path.  With P_j = prod_{i<j} rho_i (photon j has
// energy Phi/N * P_j) and R_i = g_{i+1} + rho_{i+1} R_{i+1} (R_{n-1} = 0,
// photon rows 0..n-1, vertex i = row i), the contribution of vertex i to the
// albedo gradient is Phi/N * P_i * R_i (division free), and the power
// gradient is sum_j g_j P_j / N.
//
// A resident grid of single-wave workgroups walks the paths 64 at a time.
// Every path's rows and upstream gradients are read once into registers; the
// sums are kept in LDS as 'cols' columns of FP32 accumulators per material
// and light, [row][column][channel], a lane adding to the column lane mod
// cols by a plain read, add and write: with 64 columns no two lanes meet,
// with fewer the lanes that share a column take turns.  LDS float atomics on
// one shared set cost about 120 cycles a wave instruction whatever the
// conflicts (one or 64 copies timed the same) and were more than half of the
// kernel.  After 'fold_rounds' rounds the columns are folded into FP64 registers, so
// that an accumulator takes kGradAdds additions at most between two folds
// (grad_fold); each workgroup's FP64 sums go to their own slots, which
// k_energy_sum adds in a fixed order (FP64 atomics of every workgroup on one
// set took about 100 us).  Bound by memory: 16 B of every photon row but the
// last and 12 B of upstream gradient per photon.  Measured at 1M paths x 7
// rows, 32 materials, one MI355X: 68 us and 7 us for
// the sum, 2.6 TB/s of row lines and gradients (143 us and 901 us with LDS
// atomics, three reads of the gradients and one thread per accumulator
// summing 3907 parts).
template <int kRows>
__global__ __launch_bounds__(64) void k_energy_bwd(const SceneDev* __restrict__ scenes, const float* __restrict__ albedo,
                                                   const float* __restrict__ power, const float* __restrict__ gE,
                                                   uint32_t n_mat, uint32_t cols, uint32_t fold_rounds,
                                                   double* __restrict__ part) {
  extern __shared__ float sh[];
  const SceneDev& S = scenes[0];
  const uint32_t rows = n_mat + S.n_lights, width = 3 * rows, lane = threadIdx.x;
  float* rho_s = sh;             // [n_mat][3]
  float* acc = sh + 3 * n_mat;  // [n_mat + n_lights][cols][3]
  // the lights' path ranges and Phi / N, read here once: a global read inside
  // the loop would make it wait for the loads in flight
  __shared__ uint32_t lbase[PV_MAX_LIGHTS], lcount[PV_MAX_LIGHTS];
  __shared__ float lscale[PV_MAX_LIGHTS][3];
  if (lane < S.n_lights) {
    const LightDev lt = G(S.lights)[lane];
    lbase[lane] = lt.path_base;
    lcount[lane] = lt.path_count;
    for (int c = 0; c < 3; ++c) lscale[lane][c] = power[3 * lane + c] / (float)lt.path_count;
  }
  for (uint32_t i = lane; i < 3 * n_mat; i += 64) rho_s[i] = albedo[i];
  const uint32_t turn = lane / cols, col = 3 * (lane & (cols - 1));
  for (uint32_t i = lane; i < width * cols; i += 64) acc[i] = 0.0f;
  constexpr int kOwn = (3 * (kMaxGradMaterials + PV_MAX_LIGHTS) + 63) / 64;
  double own[kOwn];  // accumulators lane, lane + 64, ... of the width
#pragma unroll
  for (int k = 0; k < kOwn; ++k) own[k] = 0.0;
  // lanes of one wave: LDS operations take effect in program order; the
  // fence keeps the compiler from moving one lane's access across another's
  auto sync_wave = [] {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
  auto fold = [&] {
    sync_wave();
#pragma unroll
    for (int k = 0; k < kOwn; ++k) {
      const uint32_t i = lane + (uint32_t)k * 64;
      if (i >= width) break;
      float* a = acc + (size_t)(i / 3) * cols * 3 + i % 3;
      for (uint32_t q = 0; q < cols; ++q) {
        own[k] += (double)a[3 * q];
        a[3 * q] = 0.0f;
      }
    }
    sync_wave();
  };
  auto add = [&](bool on, uint32_t row, float x, float y, float z) {
    for (uint32_t s = 0; s < 64 / cols; ++s) {
      if (on && turn == s) {
        float* a = acc + (size_t)row * cols * 3 + col;
        a[0] += x;
        a[1] += y;
        a[2] += z;
      }
      sync_wave();
    }
  };
  sync_wave();
  const size_t np = S.n_paths;
  // the next round's loads are issued before this round's sums, so that they
  // are in flight during them
  uint32_t info, mat[kRows], ninfo, nhit[kRows];
  F3 g[kRows], ng[kRows];
  auto load = [&](uint32_t base) {
    const uint32_t p = min(base + lane, S.n_paths - 1);
    ninfo = G(S.info)[p];
    load_hits<kRows>(S, p, nhit);
#pragma unroll
    for (int r = 0; r < kRows; ++r)
      ng[r] = *(const PV_GLOBAL F3*)(G(gE) + 3 * ((size_t)min((uint32_t)r, S.B - 1) * np + p));
  };
  uint32_t held = 0;  // rounds since the last fold
  if (blockIdx.x * 64 < S.n_paths) load(blockIdx.x * 64);
  for (uint32_t base = blockIdx.x * 64; base < S.n_paths; base += gridDim.x * 64) {
    if (held == fold_rounds) {
      fold();
      held = 0;
    }
    ++held;
    const uint32_t p = min(base + lane, S.n_paths - 1);
    info = ninfo;
#pragma unroll
    for (int r = 0; r < kRows; ++r) {
      g[r] = ng[r];
      if (r + 1 < kRows) mat[r] = mat_of(S, nhit[r]);
    }
    if (base + gridDim.x * 64 < S.n_paths) load(base + gridDim.x * 64);  // uniform
    int l = -1;
    for (uint32_t i = 0; i < S.n_lights; ++i) l = p - lbase[i] < lcount[i] ? (int)i : l;
    // lanes past the last path, paths without a photon or a light add nothing
    const uint32_t n = base + lane < S.n_paths && l >= 0 ? min(info_nseg(info), S.B) : 0u;
    float rho[kRows][3];
#pragma unroll
    for (int r = 0; r + 1 < kRows; ++r) {
      for (int c = 0; c < 3; ++c) rho[r][c] = rho_s[3 * mat[r] + c];
    }
    const int lc = max(l, 0);
    const float N = (float)max(lcount[lc], 1u);
    float P[kRows][3], gp[3], R[3], scale[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      float pr = 1.0f;
      gp[c] = 0.0f;
#pragma unroll
      for (int r = 0; r < kRows; ++r) {
        if ((uint32_t)r < n) {
          if (r > 0) pr *= rho[r - 1][c];
          gp[c] += (c == 0 ? g[r].x : (c == 1 ? g[r].y : g[r].z)) * pr;
        }
        P[r][c] = pr;
      }
      scale[c] = lscale[lc][c];
      R[c] = 0.0f;
    }
    add(n > 0, n_mat + (uint32_t)lc, gp[0] / N, gp[1] / N, gp[2] / N);
#pragma unroll
    for (int i = kRows - 2; i >= 0; --i) {
      const bool on = (uint32_t)(i + 1) < n;
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        // R_i = g_{i+1} + rho_{i+1} R_{i+1}
        const float g1 = c == 0 ? g[i + 1].x : (c == 1 ? g[i + 1].y : g[i + 1].z);
        const float rho1 = (uint32_t)(i + 2) < n ? rho[i + 1 < kRows - 1 ? i + 1 : 0][c] : 0.0f;
        R[c] = on ? g1 + rho1 * R[c] : 0.0f;
      }
      add(on, mat[i], scale[0] * P[i][0] * R[0], scale[1] * P[i][1] * R[1], scale[2] * P[i][2] * R[2]);
    }
  }
  fold();
#pragma unroll
  for (int k = 0; k < kOwn; ++k) {
    const uint32_t i = lane + (uint32_t)k * 64;
    if (i < width) part[(size_t)blockIdx.x * width + i] = own[k];
  }
}

// sums of the workgroups' parts: 16 accumulators per workgroup, 16 threads
// each (every 16th part, then a fixed-order tree)
__global__ __launch_bounds__(kBlock) void k_energy_sum(const double* __restrict__ part, uint32_t n_parts, uint32_t width,
                                                       float* __restrict__ g_albedo, uint32_t n_mat3,
                                                       float* __restrict__ g_power) {
  __shared__ double sh[16][17];
  const uint32_t e = threadIdx.x & 15u, q = threadIdx.x >> 4, i = blockIdx.x * 16 + e;
  double s = 0.0;
  if (i < width) {
#pragma unroll 8
    for (uint32_t b = q; b < n_parts; b += 16) s += part[(size_t)b * width + i];
  }
  sh[e][q] = s;
  __syncthreads();
  if (q != 0 || i >= width) return;
  for (uint32_t k = 1; k < 16; ++k) s += sh[e][k];
  if (i < n_mat3)
    g_albedo[i] = (float)s;
  else
    g_power[i - n_mat3] = (float)s;
}

// ---------------------------------------------------------------------------
// launch wrappers (host side)

// the stack columns of a block, plus one spare entry below each column (a walk
// whose sentinel was taken points there)
constexpr size_t kLdsPerCu = 160 * 1024, kStaticLds = 3 * 1024;  // the latter: what the re-trace declares besides
static size_t stack_bytes(uint32_t entries) { return (size_t)(entries + 1) * kBlock * sizeof(int32_t); }

hipError_t launch_verify(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, const uint32_t* gbase,
                         int n_scenes, VerifyWork W, pv_stats* stats, uint32_t stack, uint32_t trace_blocks,
                         uint32_t n_cu, int min_active, uint32_t* scan_tmp, hipStream_t s) {
  if (!n_tiles) return hipSuccess;
  if (stack < kMinStack || stack > (uint32_t)kMaxStack || trace_blocks == 0 || min_active < 1 || min_active > 64)
    return hipErrorInvalidValue;
  hipLaunchKernelGGL(k_verify_scan, dim3(n_tiles), dim3(kBlock), 0, s, scenes, tiles, W, stats);
  const uint32_t* toff = nullptr;
  if (n_tiles > kInlineTiles) {
    hipError_t e = launch_scan(W.tcount, W.toff, n_tiles, W.total, scan_tmp, s);
    if (e != hipSuccess) return e;
    toff = W.toff;
  }
  hipLaunchKernelGGL(k_verify_gather, dim3((n_tiles + kGatherTiles - 1) / kGatherTiles), dim3(kBlock), 0, s, scenes,
                     tiles, n_tiles, W, toff);
  const dim3 gt(trace_blocks), gf(std::min(kFinishBlocks, (n_tiles + 3) / 4));
  const uint32_t spread = std::min(4 * trace_blocks, 4 * kSpreadVerify * n_cu);
  if (n_scenes == 1) {
    hipLaunchKernelGGL(k_verify_trace<true>, gt, dim3(kBlock), stack_bytes(stack), s, scenes, gbase, n_scenes, W,
                       min_active, stack, spread);
    hipLaunchKernelGGL(k_verify_finish<true>, gf, dim3(kFinishThreads), 0, s, scenes, gbase, n_scenes, W, n_tiles, stats);
  } else {
    hipLaunchKernelGGL(k_verify_trace<false>, gt, dim3(kBlock), stack_bytes(stack), s, scenes, gbase, n_scenes, W,
                       min_active, stack, spread);
    hipLaunchKernelGGL(k_verify_finish<false>, gf, dim3(kFinishThreads), 0, s, scenes, gbase, n_scenes, W, n_tiles, stats);
  }
  return hipGetLastError();
}

hipError_t launch_scan(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t* total,
                       uint32_t* tile_tmp, hipStream_t s) {
  if (n <= kScanTile) {  // one tile: its total is the scan's
    hipLaunchKernelGGL(k_scan_tiles, dim3(1), dim3(1024), 0, s, in, out, n, total);
    return hipGetLastError();
  }
  // tile_tmp holds 2 * ceil(n / kScanTile) words: tile sums, then their offsets
  const uint32_t tiles = (n + kScanTile - 1) / kScanTile;
  hipLaunchKernelGGL(k_scan_tiles, dim3(tiles), dim3(1024), 0, s, in, out, n, tile_tmp);
  hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, tile_tmp, tile_tmp + tiles, tiles, total);
  hipLaunchKernelGGL(k_scan_add, dim3((n + 255) / 256), dim3(256), 0, s, out, n, tile_tmp + tiles);
  return hipGetLastError();
}

uint32_t scan_tmp_words(uint32_t n) { return 2 * ((n + kScanTile - 1) / kScanTile) + 2; }

uint32_t queue_chunks(uint32_t n_tiles) { return ((n_tiles + kChunkTiles - 1) / kChunkTiles + 3) / 4 * 4; }

hipError_t launch_build_queue(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, const OrderWork& O,
                              uint32_t* queue, uint32_t* qcount, hipStream_t s) {
  if (!n_tiles) return launch_scan(nullptr, nullptr, 0, qcount, nullptr, s);  // length 0
  const uint32_t chunks = (n_tiles + kChunkTiles - 1) / kChunkTiles, stride = queue_chunks(n_tiles);
  // the grid covers the padding of the rows too, whose counts are zero
  hipLaunchKernelGGL(k_queue_hist, dim3(stride), dim3(kBlock), 0, s, scenes, tiles, n_tiles, O.hist, stride);
  const uint32_t* hoff = nullptr;
  if (chunks > kInlineChunks) {
    hipLaunchKernelGGL(k_scan_tiles, dim3((kOrderBuckets * stride + kScanTile - 1) / kScanTile), dim3(1024), 0, s, O.hist,
                       O.hoff, kOrderBuckets * stride, O.scan_tmp);
    hoff = O.hoff;
  }
  hipLaunchKernelGGL(k_queue_scatter, dim3(chunks), dim3(kBlock), 0, s, scenes, tiles, n_tiles, O.hist, hoff, O.scan_tmp,
                     stride, queue, O.queue, qcount);
  return hipGetLastError();
}

hipError_t launch_mark_all(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, uint32_t* queue,
                           uint32_t* qcount, hipStream_t s) {
  if (!n_tiles) return launch_scan(nullptr, nullptr, 0, qcount, nullptr, s);
  hipLaunchKernelGGL(k_mark_all, dim3(n_tiles), dim3(kBlock), 0, s, scenes, tiles, queue, qcount);
  return hipGetLastError();
}

// variant v selects the occupancy target of the re-trace kernel (waves per
// SIMD the compiler must allow): 0 -> 4, 1 -> 5, 2 -> 6, 3 -> 8
template <bool kSingle>
static void retrace_variant(int v, dim3 g, size_t lds, hipStream_t s, const SceneDev* scenes, const uint32_t* gbase, int n_scenes,
                            const uint32_t* queue, const uint32_t* qcount, float T, uint64_t seed,
                            uint32_t frame, const uint32_t* frame_ptr, pv_stats* stats, int min_active,
                            uint32_t entries, uint32_t spread_waves, uint32_t* deal_ctr) {
  switch (v) {
    case 1:
      hipLaunchKernelGGL((k_retrace<kSingle, 5>), g, dim3(kBlock), lds, s, scenes, gbase, n_scenes, queue, qcount,
                         T, seed, frame, frame_ptr, stats, min_active, entries, spread_waves, deal_ctr);
      break;
    case 2:
      hipLaunchKernelGGL((k_retrace<kSingle, 6>), g, dim3(kBlock), lds, s, scenes, gbase, n_scenes, queue, qcount,
                         T, seed, frame, frame_ptr, stats, min_active, entries, spread_waves, deal_ctr);
      break;
    case 3:
      hipLaunchKernelGGL((k_retrace<kSingle, 8>), g, dim3(kBlock), lds, s, scenes, gbase, n_scenes, queue, qcount,
                         T, seed, frame, frame_ptr, stats, min_active, entries, spread_waves, deal_ctr);
      break;
    default:
      hipLaunchKernelGGL((k_retrace<kSingle, 4>), g, dim3(kBlock), lds, s, scenes, gbase, n_scenes, queue, qcount,
                         T, seed, frame, frame_ptr, stats, min_active, entries, spread_waves, deal_ctr);
      break;
  }
}

hipError_t launch_retrace(const SceneDev* scenes, const uint32_t* gbase, int n_scenes, const uint32_t* queue,
                          const uint32_t* qcount, float T, uint64_t seed, uint32_t frame,
                          const uint32_t* frame_ptr, pv_stats* stats, uint32_t n_blocks, uint32_t n_cu, int variant,
                          uint32_t stack, int min_active, uint32_t* deal, hipStream_t s) {
  if (stack < kMinStack || stack > (uint32_t)kMaxStack || min_active < 1 || min_active > 64) return hipErrorInvalidValue;
  const uint32_t fit = (uint32_t)(kLdsPerCu / (stack_bytes(stack) + kStaticLds));  // workgroups beside each other
  const uint32_t spread = std::min(4 * n_blocks, 4 * std::min(kSpreadRetrace, fit) * n_cu);
  if (n_scenes == 1)
    retrace_variant<true>(variant, dim3(n_blocks), stack_bytes(stack), s, scenes, gbase, n_scenes, queue, qcount, T, seed, frame,
                          frame_ptr, stats, min_active, stack, spread, deal);
  else
    retrace_variant<false>(variant, dim3(n_blocks), stack_bytes(stack), s, scenes, gbase, n_scenes, queue, qcount, T, seed, frame,
                           frame_ptr, stats, min_active, stack, spread, deal);
  return hipGetLastError();
}

hipError_t launch_compact(const SceneDev* scenes, int n_scenes, const uint2* tiles, uint32_t n_tiles, uint32_t B,
                          uint32_t n_counts, uint32_t* counts, uint32_t* offsets, uint32_t* scan_tmp, float* out_pos,
                          float* out_e, uint32_t capacity, uint32_t* total, uint32_t* base, hipStream_t s) {
  if (!n_tiles || !n_counts) {
    // no photon: every count and base is zero
    hipError_t e = launch_scan(nullptr, nullptr, 0, total, nullptr, s);
    for (int i = 0; base && e == hipSuccess && i <= n_scenes; ++i) e = launch_scan(nullptr, nullptr, 0, base + i, nullptr, s);
    return e;
  }
  hipLaunchKernelGGL(k_photon_count, dim3(n_tiles), dim3(kBlock), 0, s, scenes, tiles, counts);
  PhotonOffsets O{counts, nullptr, scan_tmp, n_counts, total, base, n_scenes};
  if (n_counts > kInlineCounts || base) {
    hipLaunchKernelGGL(k_scan_tiles, dim3((n_counts + kScanTile - 1) / kScanTile), dim3(1024), 0, s, counts, offsets,
                       n_counts, scan_tmp);
    O.off = offsets;
  }
  hipLaunchKernelGGL(k_photon_scatter, dim3(n_tiles, B), dim3(kBlock), 0, s, scenes, tiles, O, out_pos, out_e, capacity);
  return hipGetLastError();
}

// rows of the per-path register arrays: 8 for the usual bounce limits, else
// all PV_MAX_BOUNCES
constexpr int kFewRows = 8;

hipError_t launch_energy_fwd(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, uint32_t B,
                             const float* albedo, const float* power, float* E, hipStream_t s) {
  if (!n_tiles) return hipSuccess;
  if (B <= (uint32_t)kFewRows)
    hipLaunchKernelGGL(k_energy_fwd<kFewRows>, dim3(n_tiles), dim3(kBlock), 0, s, scenes, tiles, albedo, power, E);
  else
    hipLaunchKernelGGL(k_energy_fwd<PV_MAX_BOUNCES>, dim3(n_tiles), dim3(kBlock), 0, s, scenes, tiles, albedo, power,
                       E);
  return hipGetLastError();
}

// Columns of the gradient accumulators: as many (a power of two, at most one
// per lane) as keep a wave's accumulators near 26 KB, six waves per compute
// unit at 32 materials; at 256 materials eight lanes take turns on a column.
static uint32_t grad_cols(uint32_t rows) {
  uint32_t cols = 64;
  while (cols > 8 && rows * cols * 12 > 27 * 1024) cols >>= 1;
  return cols;
}
// Rounds of 64 paths between two folds: an accumulator serves 64 / cols lanes,
// and up to B - 1 vertices of a path may lie on one material.  With 32 rounds
// whatever the columns, 256 materials of which one takes nearly all hits had
// 3,584 additions in a row at 15 bounces, and the gradient of 1.6M paths an
// error of 4.4e-7 (FP32 accumulators per 256 paths had 6.1e-8; now 3.0e-8).  A
// fold costs about a round: 586 us there instead of 548, 157 and 154 at 60
// materials and 7 bounces, nothing measurable at 32.
constexpr uint32_t kGradAdds = 224;
static uint32_t grad_fold(uint32_t cols, uint32_t B) {
  const uint32_t adds = (64 / cols) * (std::max(B, 2u) - 1);
  return std::min(32u, std::max(1u, kGradAdds / adds));
}
// LDS bytes of a workgroup: the accumulators and the albedos (rows: materials and lights)
static uint32_t grad_lds(uint32_t rows) { return rows * (grad_cols(rows) + 1) * 12; }
// single-wave workgroups per compute unit: what the LDS holds, at most 16
static uint32_t grad_waves_per_cu(uint32_t rows) { return std::min(16u, 160u * 1024 / grad_lds(rows)); }

uint32_t grad_part_words(uint32_t n_cu) {
  uint32_t most = 0;
  for (uint32_t rows = 2; rows <= kMaxGradMaterials + PV_MAX_LIGHTS; ++rows)
    most = std::max(most, grad_waves_per_cu(rows) * 3 * rows);
  return most * n_cu;
}

hipError_t launch_energy_bwd(const SceneDev* scene, uint32_t n_paths, uint32_t B, const float* albedo,
                             const float* power, const float* gE, uint32_t n_mat, uint32_t n_lights, uint32_t n_cu,
                             double* part, float* g_albedo, float* g_power, hipStream_t s) {
  if (n_mat < 1 || n_mat > kMaxGradMaterials || n_lights < 1 || n_lights > PV_MAX_LIGHTS) return hipErrorInvalidValue;
  const uint32_t rows = n_mat + n_lights, width = 3 * rows, cols = grad_cols(rows);
  // an empty store: one workgroup writes zero sums
  const dim3 g(std::max(1u, std::min((n_paths + 63) / 64, n_cu * grad_waves_per_cu(rows))));
  const size_t lds = grad_lds(rows);
  const uint32_t fold = grad_fold(cols, B);
  if (B <= (uint32_t)kFewRows)
    hipLaunchKernelGGL(k_energy_bwd<kFewRows>, g, dim3(64), lds, s, scene, albedo, power, gE, n_mat, cols, fold, part);
  else
    hipLaunchKernelGGL(k_energy_bwd<PV_MAX_BOUNCES>, g, dim3(64), lds, s, scene, albedo, power, gE, n_mat, cols, fold,
                       part);
  hipLaunchKernelGGL(k_energy_sum, dim3((width + 15) / 16), dim3(kBlock), 0, s, part, g.x, width, g_albedo, 3 * n_mat,
                     g_power);
  return hipGetLastError();
}

}  // namespace pv
