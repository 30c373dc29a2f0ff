// Per-frame rebuild of the dynamic objects' hierarchies on the device: a
// linear BVH (Karras, "Maximizing Parallelism in the Construction of BVHs,
// Octrees, and k-d Trees", HPG 2012) over 30-bit Morton codes of the
// triangles' centroids, quantised in each object's centroid box.
//
//   k_lbvh_bounds   one workgroup per object: centroid box of its triangles
//   k_lbvh_keys     one thread per dynamic triangle: key (object << 30 |
//                   Morton code), value (its record)
//   k_lbvh_hist /   stable least-significant-digit radix sort of the keys, 8
//   k_lbvh_scatter  bits per pass: digit counts per tile, then a scatter that
//                   keeps the order of equal digits (wave ballots rank the keys
//                   of one digit inside a wave); the scatter scans the counts
//                   itself when there are few tiles
//   k_lbvh_sort     the four above in one launch, one workgroup per object,
//                   where every object fits a workgroup's memory
//   k_lbvh_leaves / padded triangle boxes in sorted order and a pyramid of
//   k_lbvh_pyramid  their unions over aligned power-of-two blocks
//   k_lbvh_nodes    one thread per internal node of each object's radix tree:
//                   its key range and split (the object's keys are contiguous
//                   after the sort; equal keys are ordered by position), and
//                   its two child boxes as unions over the children's position
//                   ranges, each assembled from O(log n) pyramid entries: no
//                   node waits for another
//   k_lbvh_depth    one thread per leaf counts its ancestors
//   k_lbvh_finish   one thread per object: the rebuilt tree becomes the
//                   object's hierarchy unless it is deeper than the traversal
//                   stacks allow (up to 30 + ceil(log2 n) levels are possible:
//                   the common prefix of a node's keys grows from a node to its
//                   children); the refit upload-time topology serves otherwise
//
// Leaves hold one triangle and name its record directly, so triangles are
// never moved.  The boxes are the same unions of the same padded triangle
// boxes that a bottom-up refit computes.
#include "pv_launch.h"
// The frame's beginning is here too: k_place (moved flags, world triangles,
// low pyramid levels) and k_refit (the moved objects' boxes, current
// transforms, top-level trees).

namespace pv {

namespace {

constexpr int kSortThreads = 256;
constexpr int kSortItems = 8;
constexpr uint32_t kSortTile = kSortThreads * kSortItems;  // keys per sort tile
constexpr int kDigits = 256;
constexpr int kSortPasses = 5;          // 8-bit digits over the 36 key bits (6 object + 30 Morton)
constexpr uint32_t kFusedTiles = 256;   // up to this many tiles the scatter scans the counts itself
constexpr uint32_t kSmallSort = 16384;  // up to this many triangles an object is sorted by one workgroup
constexpr int kLowLevels = 8;           // pyramid levels built inside one 256-entry workgroup
constexpr uint32_t kDepthGuard = 64;    // > 30 + 28: no radix tree here is that deep
static_assert(kSortThreads == kDigits, "one thread per digit in the tile histograms");
static_assert(kBlock == (1 << kLowLevels), "one workgroup of the leaf kernel spans the low pyramid levels");
static_assert(PV_MAX_OBJECTS <= 64, "object ids fit the 6 key bits above the Morton code");

__device__ inline uint32_t lane_of() { return threadIdx.x & 63u; }
__device__ inline uint64_t lanes_below() { return (1ull << lane_of()) - 1ull; }

__device__ inline float pad_lo(float x) { return x - (1e-6f + fabsf(x) * 1e-6f); }
__device__ inline float pad_hi(float x) { return x + (1e-6f + fabsf(x) * 1e-6f); }

// object of a dynamic triangle record: the last object whose first record is
// not after it (records are grouped by object, in object order)
__device__ inline uint32_t object_of_record(const SceneDev& S, uint32_t r) {
  uint32_t lo = 0, hi = S.n_obj;
  while (hi - lo > 1) {
    const uint32_t mid = (lo + hi) >> 1;
    if (S.objs[mid].tri_base <= r)
      lo = mid;
    else
      hi = mid;
  }
  return lo;
}

__device__ inline float3 vertex_of(const Tri& t, int i) { return make_float3(t.v[i][0], t.v[i][1], t.v[i][2]); }

constexpr float kThird = 1.0f / 3.0f;

// three times the centroid
__device__ inline float3 vertex_sum(const Tri& t) {
  const float3 a = vertex_of(t, 0), b = vertex_of(t, 1), c = vertex_of(t, 2);
  return make_float3(a.x + b.x + c.x, a.y + b.y + c.y, a.z + b.z + c.z);
}

__device__ inline float3 centroid(const Tri& t) {
  const float3 v = vertex_sum(t);
  return make_float3(v.x * kThird, v.y * kThird, v.z * kThird);
}

// 10 bits spread to every third bit
__device__ inline uint32_t spread3(uint32_t v) {
  v &= 0x3ffu;
  v = (v | (v << 16)) & 0x030000ffu;
  v = (v | (v << 8)) & 0x0300f00fu;
  v = (v | (v << 4)) & 0x030c30c3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// one axis of a centroid's code (sum: three times the centroid), its roundings
// spelled out: the order of codes is that of pv_check.h's
__device__ inline uint32_t quantise(float sum, float lo, float hi) {
  const float ext = hi - lo;
  const float u = ext > 0.0f ? fmaf(sum, kThird, -lo) / ext : 0.0f;
  return min((uint32_t)fmaxf(u * 1024.0f, 0.0f), 1023u);
}

struct Box {
  float3 lo, hi;
};

__device__ inline Box empty_box() {
  return {make_float3(__builtin_inff(), __builtin_inff(), __builtin_inff()),
          make_float3(-__builtin_inff(), -__builtin_inff(), -__builtin_inff())};
}

__device__ inline Box join(const Box& a, const Box& b) {
  return {make_float3(fminf(a.lo.x, b.lo.x), fminf(a.lo.y, b.lo.y), fminf(a.lo.z, b.lo.z)),
          make_float3(fmaxf(a.hi.x, b.hi.x), fmaxf(a.hi.y, b.hi.y), fmaxf(a.hi.z, b.hi.z))};
}

// a leaf's box: the padded box of its triangle (as the refit computes it)
__device__ inline Box tri_box(const Tri& t) {
  const float3 a = vertex_of(t, 0), b = vertex_of(t, 1), c = vertex_of(t, 2);
  return {make_float3(pad_lo(fminf(fminf(a.x, b.x), c.x)), pad_lo(fminf(fminf(a.y, b.y), c.y)),
                      pad_lo(fminf(fminf(a.z, b.z), c.z))),
          make_float3(pad_hi(fmaxf(fmaxf(a.x, b.x), c.x)), pad_hi(fmaxf(fmaxf(a.y, b.y), c.y)),
                      pad_hi(fmaxf(fmaxf(a.z, b.z), c.z)))};
}

__device__ inline Box pyr_get(const float4* pyr, uint32_t i) {
  const float4 a = pyr[2 * i], b = pyr[2 * i + 1];
  return {make_float3(a.x, a.y, a.z), make_float3(b.x, b.y, b.z)};
}

__device__ inline void pyr_put(float4* pyr, uint32_t i, const Box& v) {
  pyr[2 * i] = make_float4(v.lo.x, v.lo.y, v.lo.z, 0.0f);
  pyr[2 * i + 1] = make_float4(v.hi.x, v.hi.y, v.hi.z, 0.0f);
}

// union of the boxes at sorted positions [a, b) from the pyramid: at each
// level the blocks at the range's ragged ends, then one level up.  The
// entries of four levels are loaded before any of them is joined, so their
// loads are in flight together (min and max: the order of the joins does not
// change the box).
// Without 'full' the pyramid ends at level kLowLevels, whose entries are then
// joined one after the other (at most kLinearTris / 256 of them).
__device__ inline Box range_box(const float4* pyr, uint32_t n, uint32_t a, uint32_t b, bool full = true) {
  static_assert(kLowLevels % 4 == 0, "levels are taken four at a time");
  Box r = empty_box();
  uint32_t off = 0, m = n;
  for (int level = 0; a < b; level += 4) {
    if (!full && level == kLowLevels) {
#pragma unroll 8
      for (uint32_t i = a; i < b; ++i) r = join(r, pyr_get(pyr, off + i));
      break;
    }
    Box e[8];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const bool ta = a < b && (a & 1u) != 0u;
      e[2 * k] = ta ? pyr_get(pyr, off + a) : empty_box();
      a += ta ? 1u : 0u;
      const bool tb = a < b && (b & 1u) != 0u;
      e[2 * k + 1] = tb ? pyr_get(pyr, off + b - 1u) : empty_box();
      b -= tb ? 1u : 0u;
      a >>= 1;
      b >>= 1;
      off += m;
      m = (m + 1) / 2;
    }
#pragma unroll
    for (int k = 0; k < 8; ++k) r = join(r, e[k]);
  }
  return r;
}

// length of the common prefix of the keys at positions i and j of an object's
// sorted range (ties broken by position); -1 outside the range
__device__ inline int prefix(const uint64_t* __restrict__ key, uint32_t start, int n, int i, int j) {
  if (j < 0 || j >= n) return -1;
  const uint64_t a = key[start + (uint32_t)i], b = key[start + (uint32_t)j];
  if (a != b) return __clzll((long long)(a ^ b));
  return 64 + __clz((int)((uint32_t)i ^ (uint32_t)j));
}

}  // namespace

// centroid bounds (lo xyz, hi xyz) of an object's triangles by a workgroup of
// 1024 threads, to all
__device__ inline void object_bounds(const SceneDev& S, const ObjDev& ob, float b[6]) {
  __shared__ float red[6][1024 / 64];
  float lo[3] = {__builtin_inff(), __builtin_inff(), __builtin_inff()};
  float hi[3] = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
  for (uint32_t i = threadIdx.x; i < ob.n_tris; i += 1024) {
    const float3 c = centroid(S.tris[S.n_static + ob.tri_base + i]);
    lo[0] = fminf(lo[0], c.x), lo[1] = fminf(lo[1], c.y), lo[2] = fminf(lo[2], c.z);
    hi[0] = fmaxf(hi[0], c.x), hi[1] = fmaxf(hi[1], c.y), hi[2] = fmaxf(hi[2], c.z);
  }
  for (int off = 32; off > 0; off >>= 1)
    for (int k = 0; k < 3; ++k) {
      lo[k] = fminf(lo[k], __shfl_xor(lo[k], off, 64));
      hi[k] = fmaxf(hi[k], __shfl_xor(hi[k], off, 64));
    }
  const uint32_t w = threadIdx.x >> 6;
  if (lane_of() == 0)
    for (int k = 0; k < 3; ++k) {
      red[k][w] = lo[k];
      red[3 + k][w] = hi[k];
    }
  __syncthreads();
  for (int k = 0; k < 6; ++k) {
    float v = red[k][0];
    for (uint32_t q = 1; q < 1024 / 64; ++q) v = k < 3 ? fminf(v, red[k][q]) : fmaxf(v, red[k][q]);
    b[k] = v;
  }
}

// Morton code of a triangle's centroid in its object's centroid box
__device__ inline uint32_t morton(const Tri& t, const float b[6]) {
  const float3 c = vertex_sum(t);
  return (spread3(quantise(c.x, b[0], b[3])) << 2) | (spread3(quantise(c.y, b[1], b[4])) << 1) |
         spread3(quantise(c.z, b[2], b[5]));
}

__global__ __launch_bounds__(1024) void k_lbvh_bounds(const SceneDev* __restrict__ scenes, LbvhWork W) {
  const SceneDev& S = scenes[0];
  const uint32_t o = blockIdx.x;
  float b[6];
  object_bounds(S, S.objs[o], b);
  if (threadIdx.x == 0) {
    for (int k = 0; k < 6; ++k) W.cbox[6 * o + k] = b[k];
    W.odepth[o] = 0;
  }
}

__global__ __launch_bounds__(kBlock) void k_lbvh_keys(const SceneDev* __restrict__ scenes, LbvhWork W) {
  const SceneDev& S = scenes[0];
  const uint32_t r = blockIdx.x * blockDim.x + threadIdx.x;
  if (r >= W.n_dyn) return;
  const uint32_t o = object_of_record(S, r);
  W.key[0][r] = ((uint64_t)o << 30) | morton(S.tris[S.n_static + r], W.cbox + 6 * o);
  W.val[0][r] = r;
}

// Keys and their sort for an object of at most kSmallSort triangles by one
// workgroup: the same stable order by (object, code) as the passes below, whose
// twelve dependent launches took 85 us for 24 objects of 1,024 triangles.  A
// thread keeps its keys in registers, wave w those of the w-th sixteenth of the
// order, 64 at a time; a pass counts its digits per wave (ballots rank equal
// digits), scans the counts digit by digit, and moves the keys through LDS.
constexpr uint32_t kSortWaves = 1024 / 64;

// The lanes of a wave exchange words in LDS: its operations take effect in
// program order, and the fence keeps the compiler from moving one lane's access
// across another's (a scheduling barrier alone does not say so).
__device__ __forceinline__ void sync_wave() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// kMax: triangles of the largest object, 8,192 or kSmallSort (24 objects of
// 1,024: 14.8 us; eight of 10,000, a frame begin with rebuild 213 to 176 us)
template <uint32_t kMax>
__global__ __launch_bounds__(1024) void k_lbvh_sort(const SceneDev* __restrict__ scenes, LbvhWork W) {
  __shared__ uint32_t skey[kMax];
  __shared__ uint16_t sval[kMax], cnt[kSortWaves][kDigits];
  __shared__ uint32_t wsum[kDigits / 64];
  constexpr uint32_t kSortRounds = kMax / 1024;
  const SceneDev& S = scenes[0];
  const uint32_t o = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = lane_of();
  const ObjDev ob = S.objs[o];
  const uint32_t n = ob.n_tris;
  float b[6];
  object_bounds(S, ob, b);
  const uint32_t rounds = (n + 1023) / 1024, first = wave * rounds * 64 + lane;
  uint32_t key[kSortRounds], val[kSortRounds], pos[kSortRounds];
#pragma unroll
  for (uint32_t i = 0; i < kSortRounds; ++i) {
    const uint32_t r = first + i * 64;
    val[i] = r;
    key[i] = i < rounds && r < n ? morton(S.tris[S.n_static + ob.tri_base + r], b) : 0u;
  }
  for (int shift = 0; shift < 30; shift += 8) {
    for (uint32_t d = lane; d < kDigits; d += 64) cnt[wave][d] = 0;
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kSortRounds; ++i) {
      if (i >= rounds) break;
      const bool have = first + i * 64 < n;
      const uint32_t d = (key[i] >> shift) & (kDigits - 1u);
      uint64_t peers = __ballot(have);
      for (int bit = 0; bit < 8; ++bit) {
        const bool set = ((d >> bit) & 1u) != 0;
        const uint64_t m = __ballot(have && set);
        peers &= set ? m : ~m;
      }
      const uint32_t before = have ? cnt[wave][d] : 0u;
      pos[i] = before + (uint32_t)__popcll(peers & lanes_below());
      sync_wave();  // every lane has read before the last of its peers writes
      if (have && (peers >> lane) == 1ull) cnt[wave][d] = (uint16_t)(pos[i] + 1);
      sync_wave();
    }
    __syncthreads();
    // a thread per digit: exclusive scan over (digit, wave)
    uint32_t total = 0, x = 0;
    if (tid < (uint32_t)kDigits) {
      for (uint32_t w = 0; w < kSortWaves; ++w) total += cnt[w][tid];
      x = total;
      for (int off = 1; off < 64; off <<= 1) {
        const uint32_t y = __shfl_up(x, off, 64);
        if ((int)lane >= off) x += y;
      }
      if (lane == 63) wsum[wave] = x;
    }
    __syncthreads();
    if (tid < (uint32_t)kDigits) {
      uint32_t at = x - total;
      for (uint32_t w = 0; w < wave; ++w) at += wsum[w];
      for (uint32_t w = 0; w < kSortWaves; ++w) {
        const uint32_t c = cnt[w][tid];
        cnt[w][tid] = (uint16_t)at;
        at += c;
      }
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kSortRounds; ++i) {
      if (i >= rounds || first + i * 64 >= n) break;
      const uint32_t q = pos[i] + cnt[wave][(key[i] >> shift) & (kDigits - 1u)];
      skey[q] = key[i];
      sval[q] = (uint16_t)val[i];
    }
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kSortRounds; ++i) {
      if (i >= rounds || first + i * 64 >= n) break;
      key[i] = skey[first + i * 64];
      val[i] = sval[first + i * 64];
    }
  }
#pragma unroll
  for (uint32_t i = 0; i < kSortRounds; ++i) {
    if (i >= rounds || first + i * 64 >= n) break;
    W.key[0][ob.tri_base + first + i * 64] = ((uint64_t)o << 30) | key[i];
    W.val[0][ob.tri_base + first + i * 64] = ob.tri_base + val[i];
  }
  if (tid == 0) W.odepth[o] = 0;
}

// digit counts of one tile, stored digit-major (hist[digit * tiles + tile]),
// so that an exclusive scan gives every (digit, tile) its first output slot
__global__ __launch_bounds__(kSortThreads) void k_lbvh_hist(const uint64_t* __restrict__ key, uint32_t n, int shift,
                                                            uint32_t* __restrict__ hist, uint32_t tiles) {
  __shared__ uint32_t h[kDigits];
  h[threadIdx.x] = 0;
  __syncthreads();
  const uint32_t base = blockIdx.x * kSortTile;
  for (int s = 0; s < kSortItems; ++s) {
    const uint32_t e = base + (uint32_t)s * kSortThreads + threadIdx.x;
    if (e < n) atomicAdd(&h[(uint32_t)(key[e] >> shift) & 255u], 1u);
  }
  __syncthreads();
  hist[threadIdx.x * tiles + blockIdx.x] = h[threadIdx.x];
}

// Stable scatter of one tile: keys are taken in index order, kSortThreads at
// a time; a key's slot is the first slot of its (digit, tile), plus the keys
// of its digit placed by earlier rounds, by lower waves of this round and by
// lower lanes of its wave (lanes of equal digit found by ballots over the
// digit's bits).  hoff == nullptr: the first slots are computed here from the
// raw counts (all digits' totals, scanned, plus this digit's count in the
// earlier tiles).
__global__ __launch_bounds__(kSortThreads) void k_lbvh_scatter(const uint64_t* __restrict__ kin,
                                                               const uint32_t* __restrict__ vin,
                                                               uint64_t* __restrict__ kout, uint32_t* __restrict__ vout,
                                                               uint32_t n, int shift, const uint32_t* __restrict__ hist,
                                                               const uint32_t* __restrict__ hoff, uint32_t tiles) {
  constexpr int kWaves = kSortThreads / 64;
  __shared__ uint32_t run[kDigits];
  __shared__ uint32_t wc[kWaves][kDigits];
  const uint32_t tid = threadIdx.x, w = tid >> 6;
  if (hoff) {
    run[tid] = hoff[tid * tiles + blockIdx.x];
  } else {
    uint32_t tot = 0, mine = 0;
    for (uint32_t t = 0; t < tiles; ++t) {
      const uint32_t c = hist[tid * tiles + t];
      tot += c;
      mine += t < blockIdx.x ? c : 0u;
    }
    uint32_t x = tot;  // inclusive scan of the digit totals: waves, then wave sums
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(x, o, 64);
      if ((int)lane_of() >= o) x += y;
    }
    if (lane_of() == 63) wc[0][w] = x;
    __syncthreads();
    uint32_t before = 0;
    for (uint32_t q = 0; q < w; ++q) before += wc[0][q];
    run[tid] = before + x - tot + mine;
  }
  const uint32_t base = blockIdx.x * kSortTile;
  for (int s = 0; s < kSortItems; ++s) {
    __syncthreads();
    for (int q = 0; q < kWaves; ++q) wc[q][tid] = 0;
    __syncthreads();
    const uint32_t e = base + (uint32_t)s * kSortThreads + tid;
    const bool valid = e < n;
    uint64_t k = 0;
    uint32_t v = 0, d = 0;
    if (valid) {
      k = kin[e];
      v = vin[e];
      d = (uint32_t)(k >> shift) & 255u;
    }
    uint64_t peers = __ballot(valid);
    for (int b = 0; b < 8; ++b) {
      const bool bit = ((d >> b) & 1u) != 0;
      const uint64_t set = __ballot(valid && bit);
      peers &= bit ? set : ~set;
    }
    const uint32_t rank = (uint32_t)__popcll(peers & lanes_below());
    if (valid && rank == 0) wc[w][d] = (uint32_t)__popcll(peers);
    __syncthreads();
    if (valid) {
      uint32_t before = 0;
      for (uint32_t q = 0; q < w; ++q) before += wc[q][d];
      const uint32_t pos = run[d] + before + rank;
      kout[pos] = k;
      vout[pos] = v;
    }
    __syncthreads();
    uint32_t add = 0;
    for (int q = 0; q < kWaves; ++q) add += wc[q][tid];
    run[tid] += add;
  }
}

// level 0 of the pyramid, box b at position block * 256 + thread, and the
// levels 1..kLowLevels of that aligned 256-position block
__device__ inline void pyr_low(float4* pyr, uint32_t n, uint32_t block, Box b) {
  __shared__ float3 slo[kBlock], shi[kBlock];
  const uint32_t g = block * kBlock + threadIdx.x;
  if (g < n) pyr_put(pyr, g, b);
  uint32_t off = 0, m = n;
  for (int l = 1; l <= kLowLevels; ++l) {
    off += m;
    m = (m + 1) / 2;
    slo[threadIdx.x] = b.lo;
    shi[threadIdx.x] = b.hi;
    __syncthreads();
    const uint32_t cnt = (uint32_t)kBlock >> l;
    if (threadIdx.x < cnt) {
      const uint32_t i = 2 * threadIdx.x;
      b = join(Box{slo[i], shi[i]}, Box{slo[i + 1], shi[i + 1]});
      const uint32_t k = (block * kBlock >> l) + threadIdx.x;
      if (k < m) pyr_put(pyr, off + k, b);
    }
    __syncthreads();
  }
}

// the low pyramid levels over the padded triangle boxes in sorted order
__global__ __launch_bounds__(kBlock) void k_lbvh_leaves(const SceneDev* __restrict__ scenes, LbvhWork W,
                                                        const uint32_t* __restrict__ val) {
  const SceneDev& S = scenes[0];
  const uint32_t g = blockIdx.x * kBlock + threadIdx.x;
  Box b = empty_box();
  if (g < W.n_dyn) b = tri_box(S.tris[S.n_static + val[g]]);
  pyr_low(W.pyr, W.n_dyn, blockIdx.x, b);
}

// the pyramid levels above kLowLevels, one workgroup per scene
__global__ __launch_bounds__(1024) void k_lbvh_pyramid(const SceneDev* __restrict__ scenes, uint32_t all) {
  const SceneDev& S = scenes[blockIdx.x];
  if (!all && !S.pyr_full) return;
  const uint32_t n = S.n_dyn;
  float4* pyr = S.pyr;
  uint32_t off = pyr_level(n, kLowLevels), m = (n + (1u << kLowLevels) - 1) >> kLowLevels;
  while (m > 1) {
    const uint32_t up = (m + 1) / 2;
    for (uint32_t k = threadIdx.x; k < up; k += blockDim.x) {
      Box b = pyr_get(pyr, off + 2 * k);
      if (2 * k + 1 < m) b = join(b, pyr_get(pyr, off + 2 * k + 1));
      pyr_put(pyr, off + m + k, b);
    }
    __syncthreads();
    off += m;
    m = up;
  }
}

__global__ __launch_bounds__(kBlock) void k_lbvh_nodes(SceneDev* __restrict__ scenes, LbvhWork W,
                                                       const uint64_t* __restrict__ key,
                                                       const uint32_t* __restrict__ val) {
  SceneDev& S = scenes[0];
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  if (g >= W.n_dyn) return;
  const uint32_t o = (uint32_t)(key[g] >> 30);
  const ObjDev ob = S.objs[o];
  const uint32_t start = ob.tri_base;
  const int n = (int)ob.n_tris;
  const int i = (int)(g - start);
  if (n < 2 || i >= n - 1) return;
  // direction of the node's range and its far end
  const int d = prefix(key, start, n, i, i + 1) > prefix(key, start, n, i, i - 1) ? 1 : -1;
  const int dmin = prefix(key, start, n, i, i - d);
  int lmax = 2;
  while (prefix(key, start, n, i, i + lmax * d) > dmin) lmax *= 2;
  int l = 0;
  for (int t = lmax / 2; t >= 1; t /= 2)
    if (prefix(key, start, n, i, i + (l + t) * d) > dmin) l += t;
  const int j = i + l * d;
  // split: the last position sharing more than the range's common prefix with i
  const int dnode = prefix(key, start, n, i, j);
  int s = 0;
  for (int t = (l + 1) / 2;; t = (t + 1) / 2) {
    if (prefix(key, start, n, i, i + (s + t) * d) > dnode) s += t;
    if (t == 1) break;
  }
  const int split = i + s * d + min(d, 0);
  const int first = min(i, j), last = max(i, j);
  const uint32_t node = ob.lbvh_base + (uint32_t)i;
  int32_t ch[2];
  for (int side = 0; side < 2; ++side) {
    const int c = split + side;
    const bool leaf = side == 0 ? first == c : last == c;
    if (leaf) {
      ch[side] = leaf_code(S.n_static + val[start + (uint32_t)c], 1);
      W.parent_leaf[start + (uint32_t)c] = (int32_t)node;
    } else {
      ch[side] = (int32_t)(ob.lbvh_base + (uint32_t)c);
      W.parent_node[ob.lbvh_base + (uint32_t)c - W.first_node] = (int32_t)node;
    }
  }
  const Box b0 = range_box(W.pyr, W.n_dyn, start + (uint32_t)first, start + (uint32_t)split + 1);
  const Box b1 = range_box(W.pyr, W.n_dyn, start + (uint32_t)split + 1, start + (uint32_t)last + 1);
  Node& nd = S.nodes[node];
  nd.a = make_float4(b0.lo.x, b0.lo.y, b0.lo.z, b0.hi.x);
  nd.b = make_float4(b0.hi.y, b0.hi.z, b1.lo.x, b1.lo.y);
  nd.c = make_float4(b1.lo.z, b1.hi.x, b1.hi.y, b1.hi.z);
  nd.d = make_int4(ch[0], ch[1], -1, 0);
  if (i == 0) W.parent_node[node - W.first_node] = -1;
}

// four-wide form of binary node i of a rebuilt tree: an internal child gives
// way to its own two (every node gets one; a walk meets those of every second
// level)
__device__ inline void collapse_rebuilt(const SceneDev& S, const ObjDev& ob, uint32_t o, uint32_t i) {
  const PlaneWriter wide(S, o, S.obj_xf_cur);
  const PV_GLOBAL Node* nodes = G(S.nodes);
  const Node nd = nodes[ob.lbvh_base + i];
  const uint32_t w = 4 * (ob.lbvh_wbase + i);
  const int32_t ch[2] = {nd.d.x, nd.d.y};
  const float* f = reinterpret_cast<const float*>(&nd);
  auto put = [&](uint32_t slot, const float* b, int32_t code) {
    wide.put(slot, b[0], b[1], b[2], b[3], b[4], b[5]);
    wide.child(slot, wide_code(code < 0 ? code : code - (int32_t)ob.lbvh_base + (int32_t)ob.lbvh_wbase, wide.shift));
  };
  for (uint32_t side = 0; side < 2; ++side) {
    if (ch[side] < 0) {
      put(w + 2 * side, f + 6 * side, ch[side]);
      wide.none(w + 2 * side + 1);
    } else {
      const Node cn = nodes[ch[side]];
      const float* g = reinterpret_cast<const float*>(&cn);
      put(w + 2 * side, g, cn.d.x);
      put(w + 2 * side + 1, g + 6, cn.d.y);
    }
  }
}

// depth of every leaf (its internal ancestors), maximum per object, and the
// rebuilt nodes' four-wide forms
__global__ __launch_bounds__(kBlock) void k_lbvh_depth(const SceneDev* __restrict__ scenes, LbvhWork W,
                                                       const uint64_t* __restrict__ key) {
  const SceneDev& S = scenes[0];
  const uint32_t g = blockIdx.x * blockDim.x + threadIdx.x;
  const bool valid = g < W.n_dyn;
  uint32_t o = 0, depth = 0;
  if (valid) {
    o = (uint32_t)(key[g] >> 30);
    // every non-root node has one parent and the root none, so the climb
    // ends at the root; the step bound (above any radix tree's depth over
    // 2^28 triangles) only keeps a damaged tree from looping
    if (S.objs[o].n_tris > 1)
      for (int32_t p = W.parent_leaf[g]; p >= 0 && depth < kDepthGuard; p = W.parent_node[(uint32_t)p - W.first_node])
        ++depth;
    const ObjDev ob = S.objs[o];
    const uint32_t i = g - ob.tri_base;
    if (i + 1 < ob.n_tris) collapse_rebuilt(S, ob, o, i);
  }
  // one atomic per wave when the wave's leaves share an object
  const uint64_t act = __ballot(valid);
  if (!act) return;
  const uint32_t lead = (uint32_t)__ffsll((long long)act) - 1u;
  const uint32_t o0 = __shfl(o, (int)lead, 64);
  if (__ballot(valid && o != o0) == 0) {
    uint32_t m = valid ? depth : 0u;
    for (int off = 32; off > 0; off >>= 1) m = max(m, (uint32_t)__shfl_xor(m, off, 64));
    if (lane_of() == lead) atomicMax(&W.odepth[o0], m);
  } else if (valid) {
    atomicMax(&W.odepth[o], depth);
  }
}

__global__ void k_lbvh_finish(SceneDev* __restrict__ scenes, LbvhWork W, const uint32_t* __restrict__ val,
                              uint32_t max_depth) {
  SceneDev& S = scenes[0];
  ObjDev* objs = const_cast<ObjDev*>(S.objs);
  const uint32_t o = blockIdx.x * blockDim.x + threadIdx.x;
  if (o >= S.n_obj) return;
  const ObjDev ob = S.objs[o];
  Box b;
  int32_t root, wroot;
  if (ob.n_tris == 1) {
    root = leaf_code(S.n_static + val[ob.tri_base], 1);
    wroot = wide_code(root, S.wshift);
    b = tri_box(S.tris[leaf_first(root)]);
  } else {
    // the rebuilt tree replaces the refit topology only within the depth the
    // traversal stacks were sized for
    if (W.odepth[o] > max_depth) return;
    root = (int32_t)ob.lbvh_base;
    wroot = wide_code((int32_t)ob.lbvh_wbase, S.wshift);
    b = range_box(W.pyr, W.n_dyn, ob.tri_base, ob.tri_base + ob.n_tris);
  }
  S.obj_aabb[6 * o + 0] = b.lo.x;
  S.obj_aabb[6 * o + 1] = b.lo.y;
  S.obj_aabb[6 * o + 2] = b.lo.z;
  S.obj_aabb[6 * o + 3] = b.hi.x;
  S.obj_aabb[6 * o + 4] = b.hi.y;
  S.obj_aabb[6 * o + 5] = b.hi.z;
  objs[o].root = root;
  objs[o].wroot = wroot;
}

// ---------------------------------------------------------------------------
// top-level trees, rebuilt each frame once the object boxes are current: one
// over the static root and every object root, one over the moved objects
// only (the set that verification and the walk's clearance tests query).
// The objects of a tree are split at their median along the widest axis of
// their box centres, recursively; the static hierarchy, whose box spans the
// scene and would widen every node above it, is the root's first child
// (nearly every query enters the static side first).  One wave per tree, one
// lane per position of the item order, one level of the recursion per step:
// every range of the level is stably sorted by rank along its own axis, at
// once.  A range [lo, hi) splits at mid = (lo + hi) / 2, and each split
// position belongs to exactly one range, so node mid - 1 of the tree's block
// holds that range (node n - 1 the root above the static hierarchy).  Sorting
// only permutes a range's own items, so all nodes are written once the order
// is final, lane mid - 1 writing its range's from the range's four quarters:
// the binary node from the halves, and, for the ranges of every second level,
// the four-wide node from the quarters (of the scene's root from the static
// hierarchy and the halves).

constexpr int kTopLevels = kTopDepth - 1;  // median levels over <= PV_MAX_OBJECTS objects

// Whether a frame's walks need nodes with units of their own: an object has
// one, or a light's rays begin beyond what the grid's planes cover.
template <typename M>
__device__ inline bool object_scaled(const SceneDev& S, uint32_t o, M m) {
  return S.wshift && object_grid(S, o, m).e != 0;
}

template <typename M>
__device__ inline bool light_scaled(const SceneDev& S, uint32_t l, M m) {
  const PV_GLOBAL LightDev* lt = G(S.lights) + l;
  float d = 0.0f;
  for (int k = 0; k < 3; ++k)
    d = fmaxf(d, fabsf(m[4 * k + 3] - S.qc[k]) + fabsf(m[4 * k]) * lt->half[0] + fabsf(m[4 * k + 1]) * lt->half[1]);
  return S.wshift && !(d <= kRayReach * S.qinv);
}

// The trees of one scene, by waves 0 and 1 of a workgroup (all its threads
// come here).  scaled (the first wave's): an object, a light or an earlier frame
// asks for units.
__device__ inline void build_top(SceneDev& S, bool scaled) {
  static_assert(PV_MAX_OBJECTS <= 64, "one lane per object");
  static_assert((1 << kTopLevels) >= PV_MAX_OBJECTS, "median levels");
  __shared__ float sbx[2][2][6][64];  // [tree][buffer][box component][position]
  __shared__ int2 scode[2][2][64];    // (binary, four-wide) root codes
  const bool idle = threadIdx.x >= 128;      // a wave without a tree
  const int which = (threadIdx.x >> 6) & 1;  // tree of this wave
  const uint32_t lane = threadIdx.x & 63u;
  PV_GLOBAL Node* nodes = G(S.nodes);
  float sbox[6];
  for (int k = 0; k < 6; ++k) sbox[k] = S.sbox[k];
  // items of the tree in object order (moved objects compacted by ballot)
  const bool have = !idle && lane < S.n_obj;
  const bool take = have && (which == 0 || S.obj_moved[lane] != 0);
  const uint64_t mm = __ballot(take);
  const uint32_t n = (uint32_t)__popcll(mm);
  float ext = 0.0f;  // the objects' largest distance from the grid's middle, in steps
  if (have) {
    float b6[6];
    for (int k = 0; k < 6; ++k) {
      b6[k] = S.obj_aabb[6 * lane + k];
      ext = fmaxf(ext, fabsf((b6[k] - S.qm[k % 3]) * S.qs));
    }
    if (take) {
      const uint32_t i = (uint32_t)__popcll(mm & lanes_below());
      for (int k = 0; k < 6; ++k) sbx[which][0][k][i] = b6[k];
      scode[which][0][i] = make_int2(S.objs[lane].root, S.objs[lane].wroot);
    }
  }
  // unit of the top-level nodes: FP16 planes serve boxes at any distance from
  // their origin alike, up to 65,504 units
  const bool reach = __ballot(!(ext <= 30000.0f)) == 0 && (S.sroot != kRootNone || __ballot(ext >= 1.0f) != 0);
  int unit = 0;
  if (!reach) {
    for (int o = 32; o > 0; o >>= 1) ext = fmaxf(ext, __shfl_xor(ext, o, 64));
    unit = ceil_exp(ext * (1.0f / 128.0f));
  }
  const PlaneWriter wide(S, unit);
  const bool asked = __ballot(scaled) != 0;
  if (which == 0 && lane == 0 && !idle) {
    // once scaled, always: paths may keep vertices from where things were then
    const bool units = S.wshift && (asked || wide.g.e);
    if (units) S.state[1] = 1;
    const float near_ = kRayReach * S.qinv;
    S.wtop[2] = __float_as_int(S.wshift ? (units ? __builtin_inff() : near_) : (reach ? near_ : kReachNone));
  }
  __syncthreads();
  uint32_t lo = 0, hi = n;  // range of this lane's position
  int buf = 0;
  for (int level = 0; level < kTopLevels; ++level) {
    const float(*bx)[64] = sbx[which][buf];
    const bool live = lane < n && hi - lo >= 2;
    uint32_t dst = lane;
    if (live) {
      // widest axis of the range's box centres
      float clo[3] = {__builtin_inff(), __builtin_inff(), __builtin_inff()};
      float chi[3] = {-__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
      for (uint32_t q = lo; q < hi; ++q)
        for (int k = 0; k < 3; ++k) {
          const float c = 0.5f * (bx[k][q] + bx[3 + k][q]);
          clo[k] = fminf(clo[k], c);
          chi[k] = fmaxf(chi[k], c);
        }
      int ax = 0;
      for (int k = 1; k < 3; ++k)
        if (chi[k] - clo[k] > chi[ax] - clo[ax]) ax = k;
      // stable rank along that axis
      const float mine = 0.5f * (bx[ax][lane] + bx[3 + ax][lane]);
      uint32_t rank = 0;
      for (uint32_t q = lo; q < hi; ++q) {
        const float c = 0.5f * (bx[ax][q] + bx[3 + ax][q]);
        rank += (c < mine || (c == mine && q < lane)) ? 1u : 0u;
      }
      dst = lo + rank;
    }
    float mb[6];
    for (int k = 0; k < 6; ++k) mb[k] = bx[k][lane];
    const int2 mc = scode[which][buf][lane];
    if (lane < n) {
      for (int k = 0; k < 6; ++k) sbx[which][buf ^ 1][k][dst] = mb[k];
      scode[which][buf ^ 1][dst] = mc;
    }
    __syncthreads();
    buf ^= 1;
    if (live) {
      const uint32_t mid = (lo + hi) / 2;
      if (lane < mid) hi = mid;
      else lo = mid;
    }
  }
  const float(*bx)[64] = sbx[which][buf];
  const int2* code = scode[which][buf];
  const int32_t sroot = S.sroot, swroot = S.swroot;
  const bool above = which == 0 && sroot != kRootNone;  // the static hierarchy beside the objects
  const uint32_t first = S.top_base + (uint32_t)which * kTopNodes;
  const uint32_t wfirst = S.wtop_base + (uint32_t)which * kTopNodes;
  // root codes of a range of one or more items (its node's index is its split position - 1)
  auto bin = [&](uint32_t a, uint32_t b) { return b - a == 1 ? code[a].x : (int32_t)(first + (a + b) / 2 - 1); };
  auto wid = [&](uint32_t a, uint32_t b) { return b - a == 1 ? code[a].y : wide_code((int32_t)(wfirst + (a + b) / 2 - 1), wide.shift); };
  if (lane + 1 < n) {
    // the range that splits at lane + 1
    uint32_t a = 0, b = n, depth = 0;
    while ((a + b) / 2 != lane + 1) {
      const uint32_t m = (a + b) / 2;
      if (lane + 1 < m) b = m;
      else a = m;
      ++depth;
    }
    const uint32_t mid = lane + 1;
    // quarters (a half of one item is its own first quarter)
    const uint32_t q[5] = {a, mid - a == 1 ? mid : (a + mid) / 2, mid, b - mid == 1 ? b : (mid + b) / 2, b};
    float bb[4][6];
    for (int j = 0; j < 4; ++j) {
      for (int k = 0; k < 3; ++k) {
        bb[j][k] = __builtin_inff();
        bb[j][3 + k] = -__builtin_inff();
      }
      for (uint32_t i = q[j]; i < q[j + 1]; ++i)
        for (int k = 0; k < 3; ++k) {
          bb[j][k] = fminf(bb[j][k], bx[k][i]);
          bb[j][3 + k] = fmaxf(bb[j][3 + k], bx[3 + k][i]);
        }
    }
    float cb[2][6];
    for (int k = 0; k < 3; ++k)
      for (int h = 0; h < 2; ++h) {
        cb[h][k] = fminf(bb[2 * h][k], bb[2 * h + 1][k]);
        cb[h][3 + k] = fmaxf(bb[2 * h][3 + k], bb[2 * h + 1][3 + k]);
      }
    PV_GLOBAL Node& nd = nodes[first + lane];
    nd.a = make_float4(cb[0][0], cb[0][1], cb[0][2], cb[0][3]);
    nd.b = make_float4(cb[0][4], cb[0][5], cb[1][0], cb[1][1]);
    nd.c = make_float4(cb[1][2], cb[1][3], cb[1][4], cb[1][5]);
    nd.d = make_int4(bin(a, mid), bin(mid, b), -1, 0);
    if (((depth + (above ? 1u : 0u)) & 1u) == 0) {
      const uint32_t w = 4 * (wfirst + lane);
      for (int j = 0; j < 4; ++j) {
        if (q[j] < q[j + 1]) {
          wide.put(w + j, bb[j][0], bb[j][1], bb[j][2], bb[j][3], bb[j][4], bb[j][5]);
          wide.child(w + j, wid(q[j], q[j + 1]));
        } else {
          wide.none(w + j);
        }
      }
    }
    if (above && depth == 0) {
      // the scene's root: the static hierarchy and the halves of the objects
      const uint32_t w = 4 * (wfirst + n - 1);
      wide.put(w, sbox[0], sbox[1], sbox[2], sbox[3], sbox[4], sbox[5]);
      wide.child(w, swroot);
      for (int h = 0; h < 2; ++h) wide.put(w + 1 + h, cb[h][0], cb[h][1], cb[h][2], cb[h][3], cb[h][4], cb[h][5]);
      wide.child(w + 1, wid(a, mid));
      wide.child(w + 2, wid(mid, b));
      wide.none(w + 3);
    }
  }
  if (lane != 0 || idle) return;
  // roots: the objects' tree, the single object, or none; the static
  // hierarchy alone or above them
  int32_t root = n == 0 ? kRootNone : bin(0, n), wroot = n == 0 ? kRootNone : wid(0, n);
  if (above && n > 0) {
    float ob[6] = {__builtin_inff(), __builtin_inff(), __builtin_inff(),
                   -__builtin_inff(), -__builtin_inff(), -__builtin_inff()};
    for (uint32_t i = 0; i < n; ++i)
      for (int k = 0; k < 3; ++k) {
        ob[k] = fminf(ob[k], bx[k][i]);
        ob[3 + k] = fmaxf(ob[3 + k], bx[3 + k][i]);
      }
    PV_GLOBAL Node& nd = nodes[first + n - 1];
    nd.a = make_float4(sbox[0], sbox[1], sbox[2], sbox[3]);
    nd.b = make_float4(sbox[4], sbox[5], ob[0], ob[1]);
    nd.c = make_float4(ob[2], ob[3], ob[4], ob[5]);
    nd.d = make_int4(sroot, root, -1, 0);
    root = (int32_t)(first + n - 1);
    if (n == 1) {
      const uint32_t w = 4 * wfirst;
      wide.put(w, sbox[0], sbox[1], sbox[2], sbox[3], sbox[4], sbox[5]);
      wide.child(w, swroot);
      wide.put(w + 1, ob[0], ob[1], ob[2], ob[3], ob[4], ob[5]);
      wide.child(w + 1, wroot);
      wide.none(w + 2);
      wide.none(w + 3);
    }
    wroot = wide_code((int32_t)(wfirst + n - 1), wide.shift);
  } else if (above) {
    root = sroot;
    wroot = swroot;
  }
  S.top[which] = root;
  S.wtop[which] = wroot;
}

// the trees alone (after a rebuild of the objects' hierarchies)
__global__ __launch_bounds__(128) void k_build_top(SceneDev* __restrict__ scenes) {
  SceneDev& S = scenes[blockIdx.x];
  const uint32_t i = threadIdx.x;
  bool scaled = S.state[1] != 0;
  if (i < S.n_obj) scaled |= object_scaled(S, i, S.obj_xf_cur + 12 * i);
  if (i < S.n_lights) scaled |= light_scaled(S, i, S.light_xf_cur + 12 * i);
  build_top(S, scaled);
}

// ---------------------------------------------------------------------------
// The beginning of a frame, two launches (a chain of dependent launches costs
// at least 4.5 us each; the ten of copies, flags, triangles, pyramid levels,
// boxes and trees took 75 us for 80k dynamic triangles and 30 us for a dozen).
//
// k_place: one thread per dynamic triangle record, a workgroup per aligned 256
// of a scene's (tile = scene, first record), so that it also builds the low
// pyramid levels.  An object has moved when its new transform differs from the
// current one, which only k_refit replaces; every workgroup finds the flags by
// itself (at most 64 objects), a scene's first one writes them.

__device__ inline float xform_coord(const float* m, int r, float x, float y, float z) {
  double v = fma((double)m[4 * r + 0], (double)x,
                 fma((double)m[4 * r + 1], (double)y, fma((double)m[4 * r + 2], (double)z, (double)m[4 * r + 3])));
  return (float)v;
}

__global__ __launch_bounds__(kBlock) void k_place(const SceneDev* __restrict__ scenes, const uint2* __restrict__ tiles,
                                                  FrameInput in) {
  __shared__ uint32_t smoved[PV_MAX_OBJECTS], sbase[PV_MAX_OBJECTS];
  const uint2 tile = tiles[blockIdx.x];
  const SceneDev& S = scenes[tile.x];
  const float* xf = in.obj_tab ? in.obj_tab[tile.x] : in.obj;
  const uint32_t n = S.n_dyn, n_obj = S.n_obj;
  for (uint32_t o = threadIdx.x; o < n_obj; o += kBlock) {
    uint32_t moved = S.state[0];
    for (int i = 0; i < 12; ++i)
      moved |= __float_as_uint(S.obj_xf_cur[12 * o + i]) != __float_as_uint(xf[12 * o + i]) ? 1u : 0u;
    smoved[o] = moved;
    sbase[o] = S.objs[o].tri_base;
    if (tile.y == 0) S.obj_moved[o] = moved;
  }
  __syncthreads();
  const uint32_t g = tile.y + threadIdx.x;
  Box b = empty_box();
  if (g < n) {
    uint32_t o = 0, hi = n_obj;  // the last object whose first record is not after g
    while (hi - o > 1) {
      const uint32_t mid = (o + hi) >> 1;
      if (sbase[mid] <= g)
        o = mid;
      else
        hi = mid;
    }
    Tri t;
    if (smoved[o]) {
      const float* m = xf + 12 * o;
      const float* v = S.dlocal + 9 * (size_t)g;
      float w[9];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int r = 0; r < 3; ++r) w[3 * k + r] = xform_coord(m, r, v[3 * k], v[3 * k + 1], v[3 * k + 2]);
      t = make_tri(w, S.dtri_gid[g]);
      S.tris[S.n_static + g] = t;
    } else {
      t = S.tris[S.n_static + g];
    }
    b = tri_box(t);
  }
  pyr_low(S.pyr, n, tile.y / kBlock, b);
}

// k_refit: child boxes of the moved objects' upload-time topologies, one
// thread per node (tile = scene, first object node): each box is the union
// over the leaf-order range of the child's triangles (a subtree is a
// contiguous run of the leaf order), so no node waits for its children.  The
// unions equal those of a level-by-level refit bit for bit: the padding is
// monotone, so the padded box of a union is the union of padded boxes.
//
// One workgroup per scene (tile.y = kSlotNone) meanwhile replaces the current
// transforms, finds the objects' boxes and, with 'top', builds the trees above
// them: it reads none of the nodes that the others write.
__global__ __launch_bounds__(kBlock) void k_refit(SceneDev* __restrict__ scenes, const uint2* __restrict__ tiles,
                                                  FrameInput in, uint32_t top) {
  const uint2 tile = tiles[blockIdx.x];
  SceneDev& S = scenes[tile.x];
  const bool full = S.pyr_full != 0;
  if (tile.y != kSlotNone) {
    const uint32_t i = tile.y + threadIdx.x;
    if (i >= S.n_obj_nodes || !S.obj_moved[S.dspan_obj[i]]) return;
    const uint4 r = S.dspan[i];
    const Box b0 = range_box(S.pyr, S.n_dyn, r.x, r.y, full), b1 = range_box(S.pyr, S.n_dyn, r.z, r.w, full);
    Node& nd = S.nodes[S.obj_node_first + i];
    nd.a = make_float4(b0.lo.x, b0.lo.y, b0.lo.z, b0.hi.x);
    nd.b = make_float4(b0.hi.y, b0.hi.z, b1.lo.x, b1.lo.y);
    nd.c = make_float4(b1.lo.z, b1.hi.x, b1.hi.y, b1.hi.z);
    const uint2 ws = S.wslot[i];
    const PlaneWriter wide(S, S.dspan_obj[i], in.obj_tab ? in.obj_tab[tile.x] : in.obj);
    // slot 0 of a node always holds a child: its writer brings the origin
    if (ws.x != kSlotNone && (ws.x & 3u) == 0) wide.put_origin(ws.x >> 2);
    if (ws.y != kSlotNone && (ws.y & 3u) == 0) wide.put_origin(ws.y >> 2);
    if (ws.x != kSlotNone) wide.put(ws.x, b0.lo.x, b0.lo.y, b0.lo.z, b0.hi.x, b0.hi.y, b0.hi.z);
    if (ws.y != kSlotNone) wide.put(ws.y, b1.lo.x, b1.lo.y, b1.lo.z, b1.hi.x, b1.hi.y, b1.hi.z);
    return;
  }
  const float* oxf = in.obj_tab ? in.obj_tab[tile.x] : in.obj;
  const float* lxf = in.light_tab ? in.light_tab[tile.x] : in.light;
  const uint32_t first = S.state[0];
  static_assert(PV_MAX_OBJECTS <= 64 && PV_MAX_LIGHTS <= 64, "the first wave takes all rows");
  // an object's row by one thread: current transform, the staged copy that later
  // sparse updates start from, box and current hierarchy
  bool scaled = S.state[1] != 0;
  ObjDev* objs = const_cast<ObjDev*>(S.objs);
  for (uint32_t o = threadIdx.x; o < S.n_obj; o += kBlock) {
    float v[12];
    for (int i = 0; i < 12; ++i) v[i] = oxf[12 * o + i];
    if (top) scaled |= object_scaled(S, o, v);
    for (int i = 0; i < 12; ++i) {
      S.obj_xf_cur[12 * o + i] = v[i];
      if (in.obj_staged) in.obj_staged[12 * o + i] = v[i];
    }
    if (!S.obj_moved[o]) continue;
    const Box b = range_box(S.pyr, S.n_dyn, objs[o].tri_base, objs[o].tri_base + objs[o].n_tris, full);
    S.obj_aabb[6 * o + 0] = b.lo.x;
    S.obj_aabb[6 * o + 1] = b.lo.y;
    S.obj_aabb[6 * o + 2] = b.lo.z;
    S.obj_aabb[6 * o + 3] = b.hi.x;
    S.obj_aabb[6 * o + 4] = b.hi.y;
    S.obj_aabb[6 * o + 5] = b.hi.z;
    objs[o].root = objs[o].sah_root;  // the refit topology is the current one
    objs[o].wroot = objs[o].sah_wroot;
  }
  for (uint32_t l = threadIdx.x; l < S.n_lights; l += kBlock) {
    float c[12], v[12];
    uint32_t moved = 0;
    for (int i = 0; i < 12; ++i) {
      c[i] = S.light_xf_cur[12 * l + i];
      v[i] = lxf[12 * l + i];
      moved |= __float_as_uint(c[i]) != __float_as_uint(v[i]) ? 1u : 0u;
    }
    if (top) scaled |= light_scaled(S, l, v);
    for (int i = 0; i < 12; ++i) {
      S.light_xf_cur[12 * l + i] = v[i];
      if (in.light_staged) in.light_staged[12 * l + i] = v[i];
    }
    S.light_moved[l] = first ? 0u : moved;  // a light's first placement does not invalidate anything
  }
  __syncthreads();
  if (threadIdx.x == 0) S.state[0] = 0;
  if (top) build_top(S, scaled);
}

hipError_t launch_frame_begin(SceneDev* scenes, int n_scenes, const uint2* place_tiles, uint32_t n_place,
                              const uint2* refit_tiles, uint32_t n_refit, const FrameInput& in, bool pyramid, bool top,
                              hipStream_t s) {
  if (n_scenes <= 0) return hipSuccess;
  if (n_place) hipLaunchKernelGGL(k_place, dim3(n_place), dim3(kBlock), 0, s, scenes, place_tiles, in);
  if (pyramid) hipLaunchKernelGGL(k_lbvh_pyramid, dim3(n_scenes), dim3(1024), 0, s, scenes, 0u);
  hipLaunchKernelGGL(k_refit, dim3(n_refit), dim3(kBlock), 0, s, scenes, refit_tiles, in, top ? 1u : 0u);
  return hipGetLastError();
}

hipError_t launch_build_top(SceneDev* scenes, int n_scenes, hipStream_t s) {
  if (n_scenes <= 0) return hipSuccess;
  k_build_top<<<n_scenes, 128, 0, s>>>(scenes);
  return hipGetLastError();
}

uint32_t lbvh_sort_tiles(uint32_t n_dyn) { return (n_dyn + kSortTile - 1) / kSortTile; }

// the leaf kernel writes levels 1..kLowLevels even where the pyramid has
// fewer levels (their entries past the top are never read)
uint32_t lbvh_pyramid_entries(uint32_t n_dyn) {
  return std::max(pyr_entries(n_dyn), pyr_level(n_dyn, kLowLevels + 1));
}

hipError_t launch_rebuild_objects(SceneDev* scenes, LbvhWork W, uint32_t n_obj, uint32_t max_tris, uint32_t max_depth,
                                  hipStream_t s) {
  if (!W.n_dyn || !n_obj) return hipSuccess;
  const uint32_t nb = (W.n_dyn + kBlock - 1) / kBlock;
  int src = 0;
  if (max_tris <= kSmallSort) {
    if (max_tris <= kSmallSort / 2)
      hipLaunchKernelGGL(k_lbvh_sort<kSmallSort / 2>, dim3(n_obj), dim3(1024), 0, s, scenes, W);
    else
      hipLaunchKernelGGL(k_lbvh_sort<kSmallSort>, dim3(n_obj), dim3(1024), 0, s, scenes, W);
  } else {
    hipLaunchKernelGGL(k_lbvh_bounds, dim3(n_obj), dim3(1024), 0, s, scenes, W);
    hipLaunchKernelGGL(k_lbvh_keys, dim3(nb), dim3(kBlock), 0, s, scenes, W);
    const uint32_t tiles = lbvh_sort_tiles(W.n_dyn);
    for (int pass = 0; pass < kSortPasses; ++pass) {
      const int shift = 8 * pass;
      hipLaunchKernelGGL(k_lbvh_hist, dim3(tiles), dim3(kSortThreads), 0, s, W.key[src], W.n_dyn, shift, W.hist, tiles);
      const uint32_t* hoff = nullptr;
      if (tiles > kFusedTiles) {
        hipError_t e = launch_scan(W.hist, W.hoff, kDigits * tiles, W.htotal, W.scan_tmp, s);
        if (e != hipSuccess) return e;
        hoff = W.hoff;
      }
      hipLaunchKernelGGL(k_lbvh_scatter, dim3(tiles), dim3(kSortThreads), 0, s, W.key[src], W.val[src], W.key[src ^ 1],
                         W.val[src ^ 1], W.n_dyn, shift, W.hist, hoff, tiles);
      src ^= 1;
    }
  }
  hipLaunchKernelGGL(k_lbvh_leaves, dim3(nb), dim3(kBlock), 0, s, scenes, W, W.val[src]);
  if (W.n_dyn > (1u << kLowLevels)) hipLaunchKernelGGL(k_lbvh_pyramid, dim3(1), dim3(1024), 0, s, scenes, 1u);
  hipLaunchKernelGGL(k_lbvh_nodes, dim3(nb), dim3(kBlock), 0, s, scenes, W, W.key[src], W.val[src]);
  hipLaunchKernelGGL(k_lbvh_depth, dim3(nb), dim3(kBlock), 0, s, scenes, W, W.key[src]);
  hipLaunchKernelGGL(k_lbvh_finish, dim3((n_obj + 63) / 64), dim3(64), 0, s, scenes, W, W.val[src], max_depth);
  return hipGetLastError();
}

}  // namespace pv
