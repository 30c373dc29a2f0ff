// Host-callable launch wrappers of the library's kernels.
#pragma once
#include <hip/hip_runtime.h>

#include "pv_device.h"

namespace pv {

// rows ids[i] of dst (n_rows rows of 12 floats) take m[i] (n <= 64; the last
// entry of a repeated id wins, ids >= n_rows are skipped)
hipError_t launch_scatter_xf(float* dst, uint32_t n_rows, const uint32_t* ids, const float* m, uint32_t n,
                             hipStream_t s);
// A frame's transforms (rows of 12 floats): arrays of one scene, or device
// tables with one array per scene (then not null); the staged copies to bring
// up to date (null: none).
struct FrameInput {
  const float *obj, *light;
  const float* const* obj_tab;
  const float* const* light_tab;
  float *obj_staged, *light_staged;
};
// dynamic triangles of one object up to which its boxes are found without the
// pyramid's upper levels (SceneDev::pyr_full = 0)
constexpr uint32_t kLinearTris = 16384;
// The beginning of a frame: moved flags, current transforms, the moved objects'
// world triangles and boxes, and, with 'top', the top-level trees.
// place_tiles: (scene, first record) per kBlock dynamic triangles;
// refit_tiles: per scene (scene, kSlotNone), and (scene, first object node) per
// kBlock of them; 'pyramid': a scene has pyr_full set.
hipError_t launch_frame_begin(SceneDev* scenes, int n_scenes, const uint2* place_tiles, uint32_t n_place,
                              const uint2* refit_tiles, uint32_t n_refit, const FrameInput& in, bool pyramid, bool top,
                              hipStream_t s);
// every object's hierarchy rebuilt from its current world triangles (one
// scene): linear BVH over Morton codes, into the objects' rebuild regions; an
// object whose tree is deeper than max_depth keeps its current hierarchy;
// max_tris: triangles of the largest object
hipError_t launch_rebuild_objects(SceneDev* scenes, LbvhWork W, uint32_t n_obj, uint32_t max_tris, uint32_t max_depth,
                                  hipStream_t s);
// sort tiles of the rebuild for n_dyn triangles (W.hist holds 256 per tile)
uint32_t lbvh_sort_tiles(uint32_t n_dyn);
// entries of W.pyr (two float4 each) for n_dyn triangles
uint32_t lbvh_pyramid_entries(uint32_t n_dyn);
hipError_t launch_build_top(SceneDev* scenes, int n_scenes, hipStream_t s);
// Verification of every path of the tiles: scan, task list, traversal of the
// box-hit segments, information words of the paths with tasks, statistics.
// 'gbase' / 'n_scenes': scene path ranges (global path ids); 'stack':
// traversal stack entries per lane (stack_entries of the moved objects'
// hierarchy depths, at most kMaxStack); 'trace_blocks': grid of the traversal
// kernel; 'min_active': its walk yield threshold; 'scan_tmp':
// scan_tmp_words(n_tiles) words.
hipError_t launch_verify(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, const uint32_t* gbase,
                         int n_scenes, VerifyWork W, pv_stats* stats, uint32_t stack, uint32_t trace_blocks,
                         uint32_t n_cu, int min_active, uint32_t* scan_tmp, hipStream_t s);
hipError_t launch_scan(const uint32_t* in, uint32_t* out, uint32_t n, uint32_t* total,
                       uint32_t* tile_tmp, hipStream_t s);
uint32_t scan_tmp_words(uint32_t n);
// Scratch of the work queue's order: the ordered queue (as many entries as
// the queue can hold), bucket counts per chunk of path tiles and their scan.
struct OrderWork {
  uint32_t* queue;     // [max entries]
  uint32_t* hist;      // [8 * queue_chunks(tiles)]
  uint32_t* hoff;      // [8 * queue_chunks(tiles)]
  uint32_t* scan_tmp;  // scan_tmp_words(8 * queue_chunks(tiles))
  uint32_t* deal;      // [kDealWords] refill counters of the re-trace, zero between launches
};
uint32_t queue_chunks(uint32_t n_tiles);
// paths with the replace bit in ascending order ('queue', its length
// *qcount), and ordered by their first invalid segment (O.queue)
hipError_t launch_build_queue(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, const OrderWork& O,
                              uint32_t* queue, uint32_t* qcount, hipStream_t s);
// every path of one scene marked and queued
hipError_t launch_mark_all(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, uint32_t* queue,
                           uint32_t* qcount, hipStream_t s);
// queue / qcount: the paths to re-trace, dealt in list order
hipError_t launch_retrace(const SceneDev* scenes, const uint32_t* gbase, int n_scenes, const uint32_t* queue,
                          const uint32_t* qcount, float T, uint64_t seed, uint32_t frame,
                          const uint32_t* frame_ptr, pv_stats* stats, uint32_t n_blocks, uint32_t n_cu, int variant,
                          uint32_t stack, int min_active, uint32_t* deal, hipStream_t s);
// Photons of the tiles' paths in (scene, row, path) order: counts per (row,
// path tile) ('counts', n_counts of them, 16-byte aligned), their offsets (in
// 'offsets' and 'scan_tmp', scan_tmp_words(n_counts) words), the photons (at
// most 'capacity'), their number, and, for a batch, each scene's first photon
// and the number of all (base[n_scenes + 1], else null).
hipError_t launch_compact(const SceneDev* scenes, int n_scenes, const uint2* tiles, uint32_t n_tiles, uint32_t B,
                          uint32_t n_counts, uint32_t* counts, uint32_t* offsets, uint32_t* scan_tmp, float* out_pos,
                          float* out_e, uint32_t capacity, uint32_t* total, uint32_t* base, hipStream_t s);
// Scratch of the distribution-map update (cells: all lights' cells)
struct DmWork {
  uint32_t* dm_c;      // [cells] paths counted per cell (Compute DM_C)
  uint32_t* pruned;    // [cells] paths pruned per cell
  uint32_t* def;       // [cells] deficits
  uint32_t* dex;       // [cells + 1] their exclusive scan, then the total
  uint32_t* tcnt;      // [tiles] re-sampled paths per path tile
  uint32_t* toff;      // [tiles] their exclusive scan
  uint32_t* ttotal;    // [1]
  uint32_t* rank0;     // [PV_MAX_LIGHTS] rank of each light's first path among the re-sampled ones
  uint32_t* scan_tmp;  // scan_tmp_words(cells)
  uint32_t* scan_tmp2; // scan_tmp_words(tiles)
};
// Compute DM_C, prune (Equation 1), fill (Section 3.1) on one scene's store
// (information words updated).  tiles index the descriptor table 'table', and every tile names
// the same scene, 'scene'; the frame number is *frame_ptr when frame_ptr is
// not NULL (graph replays), else 'frame'.
hipError_t launch_dm_update(const SceneDev* table, const SceneDev* scene, const uint2* tiles, uint32_t n_tiles,
                            uint32_t cells, uint32_t n_lights, const DmWork& D, uint64_t seed,
                            uint32_t frame, const uint32_t* frame_ptr, hipStream_t s);
hipError_t launch_energy_fwd(const SceneDev* scenes, const uint2* tiles, uint32_t n_tiles, uint32_t B,
                             const float* albedo, const float* power, float* E, hipStream_t s);
// Gradients over one scene's store.  part: grad_part_words(n_cu) doubles, the
// sums of each workgroup
constexpr uint32_t kMaxGradMaterials = 256;
uint32_t grad_part_words(uint32_t n_cu);
hipError_t launch_energy_bwd(const SceneDev* scene, uint32_t n_paths, uint32_t B, const float* albedo,
                             const float* power, const float* gE, uint32_t n_mat, uint32_t n_lights, uint32_t n_cu,
                             double* part, float* g_albedo, float* g_power, hipStream_t s);

}  // namespace pv
