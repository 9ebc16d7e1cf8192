// Internal declarations shared by the libcvx translation units.
#pragma once

#include <cstdint>
#include <string>
#include <vector>

#include "../../include/cvx.h"

#define CVX_LEAF_BIT 0x80000000u
#define CVX_NONE 0xffffffffu
#define CVX_FREE 0xffffffffu  // record word x of a node that is not in the tree

#define CVX_XLEAF 0x80000000u  // record word x of a leaf, or-ed with its depth

namespace cvx {

#ifdef __HIP__
#define CVX_HD __host__ __device__
#else
#define CVX_HD
#endif
// Record words x (see below): CVX_FREE reads as a leaf too.
CVX_HD inline bool is_leaf(uint32_t x) { return (int32_t)x < 0; }
CVX_HD inline uint32_t leaf_depth(uint32_t x) { return x & 63u; }
CVX_HD inline uint32_t public_x(uint32_t x) {
  return x == CVX_FREE || !is_leaf(x) ? x : 1u | (leaf_depth(x) << 1);
}
CVX_HD inline uint32_t device_x(uint32_t x) {  // the inverse
  return x == CVX_FREE || !(x & 1u) ? x : CVX_XLEAF | (x >> 1);
}

// What a walk of a valid pool finds.
struct PoolPlan {
  uint64_t refined = 0;  // refined nodes reached
  uint32_t depth = 0;    // deepest level present
};

int check_desc(const cvx_canvas_desc* d, std::string& msg);
// the checks of validate_pool that look at no record
int check_pool_args(const cvx_canvas_desc* desc, const cvx_node* nodes, uint64_t n_nodes,
                    const void* leaves, uint64_t n_leaves, std::string& msg);
int validate_pool(const cvx_canvas_desc* desc, const cvx_node* nodes, uint64_t n_nodes,
                  const void* leaves, uint64_t n_leaves, PoolPlan* plan, std::string& msg);
int validate_views(const cvx_view* views, int n_views, const cvx_canvas_desc* const* canvases,
                   int n_canvases, std::string& msg);

// Device node record (16 bytes), one per pool node, indexed like the input:
//   x: leaf -> CVX_XLEAF | depth (the sign bit: one compare tells a leaf, one
//      subtraction gives its width); refined -> index of the first child (a
//      multiple of 8, below 2^31); CVX_FREE for an id not in the tree.  The
//      host mirror and cvx_read_records hold x in its public form, a leaf as
//      1 | depth << 1.
//   y, z, w: outer-face neighbour on the x, y, z axis: the cell of the same
//            depth across the face of the parent that this child touches, or
//            the coarser leaf covering it; CVX_NONE outside the canvas or for roots.
// Payload (indexed by node id): RGBA8 + half kappa (uint2) or 4 doubles.
// A cell on the walk of a brush stroke: node id, integer coordinates at its
// depth (root array at depth 0), depth.
struct StrokeItem {
  uint32_t node, x, y, z, depth, pad0, pad1, pad2;
};

// A leaf waiting for a split, or a cell for a merge: with its payload from
// before the stroke (RGBA8 leaves: the first word).
struct StrokePend {
  StrokeItem item;
  uint64_t pay[4];
};

// One stroke in device-ready form (world units, as the canvas descriptor).
struct StrokeArgs {
  double origin[3];
  double root_edge;
  double rgb[3];
  double sigma, radius, hmin;  // hmin = radius / k_refine
  uint32_t R, max_depth, fmt, n_stamps;
};

// A stroke whose splits are still being applied, one level per step: its
// parameters and stamps, and the leaves waiting for a split with their
// payloads from before the stroke.
struct StrokeState {
  bool active = false;
  bool coarsen = false;  // merge uniform cells once the splits are done
  bool merging = false;  // pending holds cells to merge, not leaves to split
  StrokeArgs args{};
  std::vector<double> stamps;  // 4 per stamp: x, y, z, r
  std::vector<StrokePend> pending;
};

struct DevCanvas {
  bool present = false;
  cvx_canvas_desc desc{};
  uint64_t n_nodes = 0;
  uint32_t depth = 0;     // deepest level present
  void* rec = nullptr;    // uint4 per node
  void* pay = nullptr;    // uint2 or double4 per node
  uint32_t* top = nullptr;  // top-level table: node covering each cell of depth top_depth
  uint32_t top_depth = 0;   // 0: no table
  uint64_t bytes = 0;
  // pool edits: device capacity in nodes, and a host mirror of every record
  // word x (built on the first edit), the freed groups (LIFO) and the leaf
  // count per depth
  uint64_t cap_nodes = 0;
  bool mirror_ready = false;
  bool top_stale = false;  // the top-level table may not be that of the records
  std::vector<uint32_t> mirror;
  std::vector<uint32_t> free_groups;
  std::vector<uint64_t> leaves_at_depth;
  uint64_t n_refined = 0;  // refined nodes in the tree
  // per node: the position of its last paint or the number of the link rebuild
  // that last visited it, both from the running count `epoch`
  uint32_t* mark = nullptr;
  uint64_t mark_cap = 0;
  uint32_t epoch = 0;
  StrokeState stroke;
};

// Numbers of a batch's link rebuild and of its repetitions with larger lists (at
// most one per power of two).
constexpr uint32_t kLinkRuns = 64;
// Whether the running count of a pool's marks starts again from 0 for a batch of
// n_paint payloads: where it would pass 32 bits, and wherever the marks are
// new (and all 0).
inline bool count_again(uint32_t epoch, uint64_t n_paint, bool new_marks) {
  return new_marks || epoch + n_paint + kLinkRuns > 0xffffffffull;
}

// Depth of the top-level table of a canvas: at most 6 levels and 2^18 cells,
// never below the deepest level present; 0 means no table.
inline uint32_t top_table_depth(uint32_t R, uint32_t depth) {
  uint32_t L = depth < 6 ? depth : 6;
  while (L > 0 && ((uint64_t)R << L) * ((uint64_t)R << L) * ((uint64_t)R << L) > (1ull << 18)) --L;
  return L;
}

// Per-view parameters (the host computes them once per render).
struct DViewHost {
  const void* rec;
  const void* pay;
  uint32_t R, fmt, max_depth, tiles_x;
  double o[3];          // eye in root-edge units
  // unnormalised direction of pixel (x, y): fwd + (x + cx) dirx + (y + cy) diry,
  // x + cx and y + cy exact, counted from the image centre
  double fwd[3], dirx[3], diry[3];
  double cx, cy;        // (1 - W) / 2 and (1 - H) / 2
  uint32_t W, H;
  uint64_t out_off;
  uint64_t first_tile;  // prefix sum of tile counts over the views
  float alpha_stop;
  uint32_t max_steps;
  uint32_t n_nodes;     // node ids at or above this are never loaded
  uint32_t top_depth;   // 0: ray starts descend from the root array
  const uint32_t* top;  // (R 2^top_depth)^3 node ids, x fastest
  uint32_t pieces;      // chord pieces per ray (1: unsplit)
  float t_stop;         // 1 - alpha_stop, rounded once: the FP32 caster stops once T <= t_stop
};

// The same in device memory, with what the device adds: the leaf holding the
// eye when every ray of the view starts there (eye inside the canvas, off
// every plane of the deepest grid); start_ok = 0: each ray locates its first
// leaf.
struct DView : DViewHost {
  uint32_t start_ok, start_node, start_dep;
  uint32_t start_c[3];     // the leaf's integer coordinates at start_dep
  double start_up[3], start_dn[3];  // from the eye to its upper and lower planes, in cells of the
                                    // deepest level
};

// Work queues: the work items (tiles or 64-ray chunks) are split into
// CVX_NQ contiguous ranges, one per XCD (a workgroup runs on XCD
// blockIdx.x mod 8), so the tiles one XCD renders are neighbours and share
// its L2.  A wavefront drains its own range first, then the others in turn.
constexpr uint32_t CVX_NQ_LOG = 3;
constexpr uint32_t CVX_NQ = 1u << CVX_NQ_LOG;

struct alignas(128) QueueHead {
  uint32_t next;  // items taken from this range past the fixed ones
  uint32_t pad[31];
};

// Launch-invariant header in device memory, so a captured graph can be
// replayed for any view set of the same launch shape.
struct CastHeader {
  uint64_t total_work;  // tiles (render) or 64-ray chunks (trace)
  uint64_t n_rays;      // trace mode: number of listed rays
  uint32_t n_views;
  uint32_t n_queues;        // 1 or CVX_NQ ranges in use
  uint32_t drained;         // bit q: range q was found exhausted
  uint32_t pad[25];
  QueueHead queue[CVX_NQ];  // reset by a kernel before each cast
};

// Views of a call passed as kernel arguments (at most 4 KB a launch).
constexpr uint32_t CVX_STAGE_VIEWS = 16;
struct StageViews {
  uint64_t total_work, n_rays;  // the call's header
  uint32_t n_views, n_queues;
  uint32_t first, count;        // the views of this launch
  DViewHost v[CVX_STAGE_VIEWS];
};
static_assert(sizeof(StageViews) <= 4000, "kernel arguments are limited to 4 KB");

struct CastArgs {
  const DView* views;
  CastHeader* hdr;
  void* out;
  const cvx_trace* trace_host;  // unused on device
  // trace mode
  const uint64_t* ray_ids;
  uint32_t max_leaves;
  uint32_t* leaf_ids;
  float* local_len;
  double* local_len64;
  uint32_t* n_leaves;
  uint32_t* flags;
  float* trace_rgba;
  double* end_point;
  uint64_t* stats;
  uint32_t tile_w, tile_h;
  uint32_t fixed_wgs;    // the first workgroups of the grid, whose wavefronts have a fixed item
  uint32_t small_pools;  // every pool the views read has at most 2^28 nodes
  uint32_t root_leaves;  // some view's canvas may have leaves of depth 0 (R > 1, or one leaf)
  // FP32 render with lane refill when item_tiles > 1: a work item is up to
  // item_tiles tiles of one view, and waiting lanes take its next rays once
  // refill_min lanes of the wavefront wait
  uint32_t item_tiles;
  uint32_t refill_min;
  // FP32 render or trace of chord pieces when pieces > 1: a view with
  // pieces > 1 splits each ray's chord into that many consecutive pieces,
  // traced as separate work items; render pieces write (colour, T) to
  // split_tmp[pixel * pieces + piece] for the merge
  uint32_t pieces;
  void* split_tmp;
};

// kernel launchers (cvx_upload.hip, cvx_cast.hip); return a hipError_t value
int launch_top_table(void* stream, const void* rec, uint64_t n_nodes, uint32_t R, uint32_t L,
                     uint32_t* top);
// Counts of k_extract_x: leaves per depth, then the refined nodes.
constexpr uint32_t CVX_COUNT_REFINED = 63, CVX_COUNT_WORDS = 64;
static_assert(CVX_MAX_DEPTH < CVX_COUNT_REFINED, "one word per depth");
int launch_extract_x(void* stream, const void* rec, uint64_t n, uint32_t* counts, uint32_t* out);
// A small batch of edits (k_edit_small).  counts: region roots found, then
// nodes per level; state: the level whose links are not done, depth if none is.
struct EditArgs {
  const uint32_t *ids, *xs, *pids;
  const void* src;
  const uint32_t *changed, *changed_depth;
  uint32_t *roots, *root_depth, *counts, *state, *mark, *frontiers;
  void *rec, *pay;
  uint64_t n_nodes;
  uint32_t n_touched, n_paint, n_changed, words, base, epoch, R, first_level, depth, cap;
};
constexpr uint32_t EDIT_LIST = 2048;
int launch_edit_small(void* stream, const EditArgs& a);
int launch_scatter_records(void* stream, const uint32_t* ids, const uint32_t* xs, uint64_t n,
                           void* rec);
int launch_scatter_payloads(void* stream, const uint32_t* ids, const void* src, uint64_t n,
                            uint32_t leaf_bytes, void* pay, uint32_t* mark, uint32_t base);
// the outer links below the region roots, level by level: frontiers holds two
// lists of cap nodes, counts one count per level (zeroed by the caller, the
// counts of levels first_level + 1 .. last_level + 1 are left in it)
int launch_links(void* stream, uint32_t first_level, uint32_t last_level, void* rec, uint32_t R,
                 const uint32_t* roots, const uint32_t* root_depth, const uint32_t* n_roots,
                 uint32_t* frontiers, uint32_t cap, uint32_t* counts, uint64_t n_nodes,
                 uint32_t* mark, uint32_t epoch);
int launch_dirty_roots(void* stream, const uint32_t* changed, const uint32_t* depth, uint64_t n,
                       const void* rec, uint32_t R, uint32_t* out, uint32_t* out_depth,
                       uint32_t* out_count, uint64_t n_nodes, uint32_t* mark, uint32_t base);
// Words of the state of launch_pool_build: refined nodes found per level, then
// a word that is not 0 when the pool is invalid; the list of refined nodes (as
// many as there are child groups) follows at UP_LIST.
constexpr uint32_t UP_BAD = CVX_MAX_DEPTH + 1, UP_LIST = 64;
static_assert(UP_BAD < UP_LIST, "one state word per level");
int launch_pool_build(void* stream, const void* raw_nodes, uint64_t n_nodes, const void* raw_leaves,
                      uint64_t n_leaves, uint32_t fmt, uint32_t R, uint32_t max_depth, void* rec,
                      void* pay, uint32_t* state, uint32_t cap);
int launch_cast(void* stream, uint32_t variant, bool trace, bool stats, bool out_f64,
                const CastArgs& a, uint32_t workgroups, uint32_t wg_size);
// the front-to-back merge of chord pieces into out (views with pieces > 1)
int launch_merge_pieces(void* stream, const DView* views, const CastHeader* hdr, uint32_t n_views,
                        const void* tmp, void* out, uint32_t stride);
// Scratch of the allocation-free render entry point: a CastHeader followed by
// CVX_NOALLOC_MAX_VIEWS view records, in a fixed device array of
// cvx_cast.hip.  scratch_address returns its address on the current device
// (looked up once per device; call with that device current).
constexpr size_t CVX_SCRATCH_BYTES = sizeof(CastHeader) + CVX_NOALLOC_MAX_VIEWS * sizeof(DView);
int scratch_address(int device, void** ptr);
// the shared first leaf of every view whose eye lies inside its canvas
int launch_view_starts(void* stream, DView* views, CastHeader* hdr, uint32_t enable);
// the same for views passed as kernel arguments, which it also writes to the
// device table together with the header
int launch_stage_views(void* stream, const DView* host_views, uint32_t n_views,
                       const CastHeader& host_hdr, DView* views, CastHeader* hdr,
                       uint32_t enable);
// `levels` levels of a stroke's walk (cvx_stroke.hip) from n cells: items, or
// nullptr for the roots.  counts[0] holds n; level l leaves its children's
// count in counts[l + 1] and them in lists + (l & 1) cap (two lists of cap
// cells).  merge = 1: find cells to merge instead of painting and splitting.
int launch_stroke_visit(void* stream, uint32_t levels, const StrokeItem* items, uint32_t n,
                        const StrokeArgs& a, const void* stamps, const void* rec, void* pay,
                        uint64_t n_nodes, StrokeItem* lists, uint32_t cap, uint32_t* counts,
                        StrokePend* pend, uint32_t* pend_count, uint32_t pend_cap,
                        uint32_t merge);

}  // namespace cvx
