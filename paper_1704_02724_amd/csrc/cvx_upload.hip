// Device re-layout of an uploaded pool and the GPU build of the 3-neighbour
// graph G_3 (Sec. 4.1.1 "Neighbor Graph", Sec. 4.1.2: G_3 is derived on the
// GPU from G_p after every update).
//
// Each cell has six face neighbours of the same or smaller depth.  The three
// on the sibling side follow from index arithmetic (the sibling across axis k
// is I xor 2^k inside the group); the three "outer" ones cross the parent's
// boundary and are stored.  They are produced level by level, one thread per
// node, from the parent's neighbours only:
//   child I = first_child(P) + o touches, on axis k, the face of P on side
//   s = bit_k(o).  Let M be P's same-depth-or-coarser neighbour across that
//   face (P's sibling when that face is inner to P's own group, P's stored
//   link otherwise, root-array arithmetic for roots).  If M is refined, the
//   same-depth neighbour of I is M's child o xor 2^k (Sec. 4.1.1: the children
//   of D_1 touching D are C(D_1) and C(D_1)+2 in the quadtree case); else M.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "cvx_internal.h"

namespace cvx {

// (r: P's record)
__device__ __forceinline__ uint32_t neighbour_of_parent(const uint4 r, uint32_t P,
                                                        uint32_t plevel, uint32_t k, uint32_t s,
                                                        uint32_t R) {
  if (plevel == 0) {
    uint32_t c[3] = {P % R, (P / R) % R, P / (R * R)};
    uint32_t stride = k == 0 ? 1u : (k == 1 ? R : R * R);
    if (s) return c[k] + 1 < R ? P + stride : CVX_NONE;
    return c[k] > 0 ? P - stride : CVX_NONE;
  }
  uint32_t oP = P & 7u;
  if (((oP >> k) & 1u) != s) return s ? P + (1u << k) : P - (1u << k);
  return k == 0 ? r.y : (k == 1 ? r.z : r.w);
}

// ---- uploads ----------------------------------------------------------------
// An upload is checked and laid out in one walk from the roots down, a launch
// per level, the refined nodes of a level in a list that the level above has
// written.  Eight lanes take a refined node, one per child: they check the
// child's parent field, its leaf index or child group, write its record and
// payload, and list it if it is refined.  A group is claimed by its first
// reference (its first record word leaves CVX_FREE), so a second one, a shared
// group or a cycle, is found whatever the order, and the lists hold no more
// nodes than there are groups.  A faulty child is laid out as a leaf: nothing
// that was not checked is followed, and the walk ends.  The host then looks for
// the message; it used to make this walk for every pool, one random record
// after the other, and send its breadth-first order along.  An upload of 357,040
// nodes took 1.36 ms and takes 0.44, of 33.4 M nodes 154 ms and 20: the copy of
// the pool from pageable memory bounds it now (of 56.5 M nodes the kernels take
// 2.9 ms of 37).
__device__ __forceinline__ bool bad_payload(const uint2* pay, uint64_t i, uint32_t fmt) {
  if (fmt == CVX_LEAF_RGBA8_F16) {
    const uint32_t h = pay[i].y & 0xffffu;  // negative (but not -0), or not finite
    return h > 0x8000u || (h & 0x7c00u) == 0x7c00u;
  }
  const double4 v = ((const double4*)pay)[i];
  return !(isfinite(v.x) && isfinite(v.y) && isfinite(v.z) && isfinite(v.w) && v.w >= 0.0);
}

__global__ __launch_bounds__(256) void k_check_leaves(const uint2* __restrict__ leaves, uint64_t n,
                                                      uint32_t fmt, uint32_t* __restrict__ state) {
  bool bad = false;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x)
    bad |= bad_payload(leaves, i, fmt);
  if (bad) state[UP_BAD] = 1;
}

struct PoolArgs {
  const uint2* raw;
  const void* raw_leaves;
  uint4* rec;
  void* pay;
  uint32_t* state;
  uint64_t n_nodes, n_leaves;
  uint32_t fmt, R, max_depth, cap;
};

// Record word x of node I of depth `level` from its uploaded form, its payload,
// and its place at `out` in the list.
__device__ __forceinline__ uint32_t lay_out_node(const PoolArgs& a, uint32_t I, uint2 nd,
                                                 uint32_t level, uint32_t out, bool bad) {
  const uint32_t leaf = CVX_XLEAF | level;
  bool refined = false;
  if (nd.x & CVX_LEAF_BIT) {
    const uint32_t li = nd.x & ~CVX_LEAF_BIT;
    if (li >= a.n_leaves)
      bad = true;
    else if (a.fmt == CVX_LEAF_RGBA8_F16)
      ((uint2*)a.pay)[I] = ((const uint2*)a.raw_leaves)[li];
    else
      ((double4*)a.pay)[I] = ((const double4*)a.raw_leaves)[li];
  } else {
    const uint32_t P0 = (a.R * a.R * a.R + 7u) & ~7u;
    bad |= nd.x % 8u != 0 || nd.x < P0 || (uint64_t)nd.x + 8 > a.n_nodes || level >= a.max_depth;
    if (!bad) bad = atomicCAS(&a.rec[nd.x].x, CVX_FREE, I) != CVX_FREE;
    refined = !bad;
  }
  if (bad) a.state[UP_BAD] = 1;
  const uint64_t m = __ballot(refined);
  if (refined) {
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t before = (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
    uint32_t base = 0;
    if (before == 0) base = atomicAdd(&a.state[level], (uint32_t)__popcll(m));
    base = __shfl(base, __ffsll((unsigned long long)m) - 1, 64);
    if (out + base + before < a.cap) a.state[UP_LIST + out + base + before] = I;
  }
  return refined ? nd.x : leaf;
}

__global__ __launch_bounds__(256) void k_pool_roots(PoolArgs a) {
  const uint32_t I = blockIdx.x * blockDim.x + threadIdx.x;
  if (I >= a.R * a.R * a.R) return;
  const uint2 nd = a.raw[I];
  const uint32_t x = lay_out_node(a, I, nd, 0, 0, nd.y != CVX_NONE);
  a.rec[I] = make_uint4(x, CVX_NONE, CVX_NONE, CVX_NONE);
}

// The children of the refined nodes of depth level - 1.
__global__ __launch_bounds__(256) void k_pool_level(PoolArgs a, uint32_t level) {
  uint32_t begin = 0;
  for (uint32_t d = 0; d + 1 < level; ++d) begin += a.state[d];
  uint32_t end = begin + a.state[level - 1];
  if (end > a.cap) end = a.cap;
  const uint32_t o = threadIdx.x & 7u, groups = gridDim.x * (blockDim.x / 8u);
  for (uint32_t i = begin + blockIdx.x * (blockDim.x / 8u) + threadIdx.x / 8u; i < end;
       i += groups) {
    const uint32_t P = a.state[UP_LIST + i];
    const uint4 rp = a.rec[P];
    const uint32_t I = rp.x + o;
    const uint2 nd = a.raw[I];
    uint32_t link[3];
    for (uint32_t k = 0; k < 3; ++k) {
      uint32_t M = neighbour_of_parent(rp, P, level - 1, k, (o >> k) & 1u, a.R);
      if (M != CVX_NONE) {
        const uint32_t mx = a.rec[M].x;
        if (!is_leaf(mx)) M = mx + (o ^ (1u << k));
      }
      link[k] = M;
    }
    const uint32_t x = lay_out_node(a, I, nd, level, end, nd.y != P);
    a.rec[I] = make_uint4(x, link[0], link[1], link[2]);
  }
}

int launch_pool_build(void* stream, const void* raw_nodes, uint64_t n_nodes, const void* raw_leaves,
                      uint64_t n_leaves, uint32_t fmt, uint32_t R, uint32_t max_depth, void* rec,
                      void* pay, uint32_t* state, uint32_t cap) {
  const PoolArgs a = {(const uint2*)raw_nodes, raw_leaves, (uint4*)rec, pay, state,
                      n_nodes, n_leaves, fmt, R, max_depth, cap};
  hipStream_t s = (hipStream_t)stream;
  const uint32_t bs = 256;
  if (n_leaves) {
    const uint64_t blocks = std::min<uint64_t>((n_leaves + bs - 1) / bs, 2048);
    hipLaunchKernelGGL(k_check_leaves, dim3((uint32_t)blocks), dim3(bs), 0, s,
                       (const uint2*)raw_leaves, n_leaves, fmt, state);
  }
  hipLaunchKernelGGL(k_pool_roots, dim3((R * R * R + bs - 1) / bs), dim3(bs), 0, s, a);
  // the levels of a tree are as many as it has groups at most
  const uint32_t blocks = std::min<uint32_t>((cap + bs / 8 - 1) / (bs / 8), 2048);
  for (uint32_t level = 1; level <= max_depth && level <= cap; ++level)
    hipLaunchKernelGGL(k_pool_level, dim3(blocks), dim3(bs), 0, s, a, level);
  return (int)hipGetLastError();
}

// Top-level table (Sec. 4: the canvas is a uniform array of roots): for every
// cell of depth L, x fastest, the node of depth <= L that covers it (a leaf
// above L, or the depth-L node itself).  One thread per cell walks down from
// its root by the bits of its coordinates.
__global__ void k_top_table(const uint4* __restrict__ rec, uint64_t n_nodes, uint32_t R,
                            uint32_t L, uint32_t* __restrict__ top) {
  const uint32_t side = R << L;
  const uint64_t n = (uint64_t)side * side * side;
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t x = (uint32_t)(i % side), y = (uint32_t)((i / side) % side),
                 z = (uint32_t)(i / ((uint64_t)side * side));
  uint32_t I = (x >> L) + R * ((y >> L) + R * (z >> L));
  for (uint32_t lvl = 0; lvl < L; ++lvl) {
    const uint32_t cx = rec[I].x;
    if (is_leaf(cx) || (uint64_t)cx + 8 > n_nodes) break;
    const uint32_t sh = L - 1 - lvl;
    I = cx + (((x >> sh) & 1u) | (((y >> sh) & 1u) << 1) | (((z >> sh) & 1u) << 2));
  }
  top[i] = I;
}

int launch_top_table(void* stream, const void* rec, uint64_t n_nodes, uint32_t R, uint32_t L,
                     uint32_t* top) {
  const uint64_t side = (uint64_t)R << L, n = side * side * side;
  const uint32_t bs = 256;
  hipLaunchKernelGGL(k_top_table, dim3((uint32_t)((n + bs - 1) / bs)), dim3(bs), 0,
                     (hipStream_t)stream, (const uint4*)rec, n_nodes, R, L, top);
  return (int)hipGetLastError();
}

// ---- pool edits -------------------------------------------------------------
// Record words x of nodes [0, n) in their public form, packed (for the host
// mirror), and how many leaves there are per depth and (at CVX_COUNT_REFINED)
// refined nodes.  Bound by the copy of the words to the host.  The host counted
// them before, a chain of increments of mostly one counter: the first edit of a
// pool of 357,040 nodes took 430 us and takes 200.  A wavefront adds up its
// nodes of one kind at a time, nearly always two or three kinds.
__global__ __launch_bounds__(256) void k_extract_x(const uint4* __restrict__ rec, uint64_t n,
                                                   uint32_t* __restrict__ counts,
                                                   uint32_t* __restrict__ out) {
  __shared__ uint32_t sum[CVX_COUNT_WORDS];
  if (threadIdx.x < CVX_COUNT_WORDS) sum[threadIdx.x] = 0;
  __syncthreads();
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (uint64_t)gridDim.x * blockDim.x) {
    const uint32_t dx = rec[i].x;
    out[i] = public_x(dx);
    uint32_t kind = is_leaf(dx) ? leaf_depth(dx) : CVX_COUNT_REFINED;
    bool todo = dx != CVX_FREE;
    while (todo) {
      const uint32_t k = __builtin_amdgcn_readfirstlane(kind);
      const uint64_t m = __ballot(kind == k);
      if (kind == k) {
        todo = false;
        if ((m & ((1ull << (threadIdx.x & 63u)) - 1ull)) == 0)
          atomicAdd(&sum[k], (uint32_t)__popcll(m));
      }
    }
  }
  __syncthreads();
  if (threadIdx.x < CVX_COUNT_WORDS && sum[threadIdx.x])
    atomicAdd(&counts[threadIdx.x], sum[threadIdx.x]);
}

int launch_extract_x(void* stream, const void* rec, uint64_t n, uint32_t* counts, uint32_t* out) {
  if (!n) return hipSuccess;
  const uint32_t bs = 256;
  const uint64_t blocks = std::min<uint64_t>((n + bs - 1) / bs, 2048);
  hipLaunchKernelGGL(k_extract_x, dim3((uint32_t)blocks), dim3(bs), 0, (hipStream_t)stream,
                     (const uint4*)rec, n, counts, out);
  return (int)hipGetLastError();
}

// Record words x of touched nodes (first child, 1 | depth << 1, or CVX_FREE, as
// the host mirror holds them).
// A node that stays in the tree keeps its links (they depend on its parent,
// which did not change); a node leaving the tree gets null links.
__global__ void k_scatter_records(const uint32_t* __restrict__ ids, const uint32_t* __restrict__ xs,
                                  uint64_t n, uint4* __restrict__ rec) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  const uint32_t x = xs[i];
  if (x == CVX_FREE)
    rec[ids[i]] = make_uint4(CVX_FREE, CVX_NONE, CVX_NONE, CVX_NONE);
  else
    ((uint32_t*)&rec[ids[i]])[0] = device_x(x);
}

// Payloads painted by a batch, lb bytes each (8 or 32, so whole uint2 words), in
// the order of the edits: a leaf painted twice keeps its last payload.  The
// first kernel leaves the largest position in the node's mark (base + position,
// above everything an earlier batch left there), the second writes where the
// mark is its own.  (In place of a host sort of the list by node.)
__global__ void k_stamp_payloads(const uint32_t* __restrict__ ids, uint64_t n,
                                 uint32_t* __restrict__ mark, uint32_t base) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) atomicMax(&mark[ids[i]], base + (uint32_t)i);
}
__global__ void k_scatter_payloads(const uint32_t* __restrict__ ids, const uint2* __restrict__ src,
                                   uint64_t n, uint32_t words, uint2* __restrict__ pay,
                                   const uint32_t* __restrict__ mark, uint32_t base) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n * words) return;
  const uint64_t j = i / words, w = i % words;
  const uint32_t id = ids[j];
  if (mark[id] == base + (uint32_t)j) pay[(uint64_t)id * words + w] = src[i];
}

// Links of child o of node P (links final); its id if it is refined, else
// CVX_NONE.
__device__ __forceinline__ uint32_t link_child(uint4* rec, uint32_t P, uint32_t o, uint32_t level,
                                               uint32_t R, uint64_t n_nodes) {
  const uint4 rp = rec[P];
  if (is_leaf(rp.x) || (uint64_t)rp.x + 8 > n_nodes) return CVX_NONE;
  const uint32_t C = rp.x + o;
  const uint32_t cx = rec[C].x;
  uint32_t M[3], mx[3];
  for (uint32_t k = 0; k < 3; ++k) {
    M[k] = neighbour_of_parent(rp, P, level, k, (o >> k) & 1u, R);
    mx[k] = M[k] != CVX_NONE ? rec[M[k]].x : CVX_XLEAF;
  }
  for (uint32_t k = 0; k < 3; ++k)
    if (!is_leaf(mx[k])) M[k] = mx[k] + (o ^ (1u << k));
  uint32_t* w = (uint32_t*)&rec[C];
  w[1] = M[0];
  w[2] = M[1];
  w[3] = M[2];
  return is_leaf(cx) ? CVX_NONE : C;
}

// One level of the G_3 rebuild: for every refined node P of the frontier
// (depth `level`, links already final) and every region root of that depth,
// derive the outer links of its 8 children as at upload and append the refined
// children to the next frontier.  Only the children's y, z, w words are
// written; the x words and the links of level `level` are read.  The counts
// stay on the device, so the levels follow each other without the host, which
// used to launch, read a count back and wait for each (about 40 us a level).
// Latency-bound: eight lanes work on a node, one per child, with its three
// neighbour records in flight together (one thread per node took 14 us for any
// frontier).  A batch of 20,000 paints and 2,000 refinements on a 9 M-node
// canvas, its undo and a 640x360 frame: 5.9 ms before, 1.56 with this, one
// upload block and k_stamp_payloads.
__global__ __launch_bounds__(256) void k_links_level(
    const uint32_t* __restrict__ frontier, const uint32_t* __restrict__ counts,
    const uint32_t* __restrict__ roots, const uint32_t* __restrict__ root_depth,
    const uint32_t* __restrict__ n_roots, uint32_t level, uint4* rec, uint32_t R,
    uint32_t* __restrict__ next, uint32_t* __restrict__ next_count, uint32_t cap, uint64_t n_nodes,
    uint32_t* __restrict__ mark, uint32_t epoch) {
  const uint32_t n_in = counts[level] < cap ? counts[level] : cap, n_r = *n_roots;
  const uint32_t o = threadIdx.x & 7u;
  const uint32_t groups = gridDim.x * (blockDim.x / 8u);
  for (uint32_t i = blockIdx.x * (blockDim.x / 8u) + threadIdx.x / 8u; i < n_in + n_r; i += groups) {
    const bool is_root = i >= n_in;
    if (is_root && root_depth[i - n_in] != level) continue;
    const uint32_t P = is_root ? roots[i - n_in] : frontier[i];
    // a node listed twice (reached from its parent and named as a root of a
    // changed region, or as a root twice) is processed once
    uint32_t seen = 0;
    if (o == 0) seen = atomicExch(&mark[P], epoch) == epoch ? 1u : 0u;
    if (__shfl(seen, (int)(threadIdx.x & 63u & ~7u), 64)) continue;
    const uint32_t C = link_child(rec, P, o, level, R, n_nodes);
    if (C != CVX_NONE) {
      const uint32_t slot = atomicAdd(next_count, 1u);
      if (slot < cap) next[slot] = C;  // the host sees a count above the capacity
    }
  }
}

// Roots of the regions whose links a batch of edits can change.  A node's
// links depend only on its parent's links and on the record words of the
// parent's face neighbours; so after the nodes `changed` (depth `depth`)
// were refined or coarsened, every changed link lies strictly below one of:
// a changed node that is refined (its children are new), or a refined
// same-depth face neighbour of a changed node (a sibling, a same-depth outer
// link, or at depth 0 a neighbouring root).  Outer links to coarser cells
// are leaves and have nothing below them (one that the batch refined is a
// changed node itself, at its own, smaller depth).
// The links are from before the batch.  One may name a node whose group the
// batch has freed and given out again, now at any depth: rebuilt at this one
// and marked, it would be passed over at its own.  Every child that a batch
// creates is painted by it, so it carries a mark of `base` or above; a refined
// neighbour with such a mark is left out, being either below a refined cell
// that is listed or a changed node, listed for itself.
__device__ __forceinline__ void dirty_roots_of(uint32_t X, uint32_t d, const uint4* rec, uint32_t R,
                                               uint32_t* out, uint32_t* out_depth,
                                               uint32_t* out_count, uint64_t n_nodes,
                                               uint32_t* mark, uint32_t base) {
  uint32_t cand[7];
  cand[0] = X;
  if (d == 0) {
    const uint32_t c[3] = {X % R, (X / R) % R, X / (R * R)};
    for (uint32_t k = 0; k < 3; ++k) {
      const uint32_t stride = k == 0 ? 1u : (k == 1 ? R : R * R);
      cand[1 + 2 * k] = c[k] + 1 < R ? X + stride : CVX_NONE;
      cand[2 + 2 * k] = c[k] > 0 ? X - stride : CVX_NONE;
    }
  } else {
    const uint4 r = rec[X];
    for (uint32_t k = 0; k < 3; ++k) cand[1 + k] = X ^ (1u << k);
    cand[4] = r.y;
    cand[5] = r.z;
    cand[6] = r.w;
  }
  for (uint32_t j = 0; j < 7; ++j) {
    const uint32_t N = cand[j];
    if (N == CVX_NONE || (uint64_t)N >= n_nodes) continue;
    const uint32_t x = rec[N].x;
    if (is_leaf(x)) continue;  // or not in the tree (CVX_FREE)
    if (j && __hip_atomic_load(&mark[N], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= base)
      continue;
    const uint32_t slot = atomicAdd(out_count, 1u);
    out[slot] = N;
    out_depth[slot] = d;
  }
}

__global__ void k_dirty_roots(const uint32_t* __restrict__ changed,
                              const uint32_t* __restrict__ depth, uint64_t n,
                              const uint4* __restrict__ rec, uint32_t R,
                              uint32_t* __restrict__ out, uint32_t* __restrict__ out_depth,
                              uint32_t* __restrict__ out_count, uint64_t n_nodes,
                              uint32_t* __restrict__ mark, uint32_t base) {
  const uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  dirty_roots_of(changed[i], depth[i], rec, R, out, out_depth, out_count, n_nodes, mark, base);
}

// A small batch in one launch, by one workgroup: records, payloads, region
// roots and links, as the kernels above, with barriers in place of launches and
// the frontiers in LDS.  A batch is a chain of dependent steps of little work
// each, a launch and its gap (about 10 us a step) against one or two round trips
// to the cache here.  Where a frontier is larger than the LDS list, the launches
// per level go on from there: the frontiers stand in their lists too.  A batch of
// 8 refinements and its undo, in pools of 0.36 and 9 M nodes: 148 and 209 us
// before, 71 and 84 now, most of it the host's side.
__global__ __launch_bounds__(1024) void k_edit_small(EditArgs a) {
  __shared__ uint32_t list[2][EDIT_LIST];
  __shared__ uint32_t count[2];
  __shared__ uint32_t n_roots;
  const uint32_t t = threadIdx.x, nt = blockDim.x;
  uint4* rec = (uint4*)a.rec;
  uint2* pay = (uint2*)a.pay;
  const uint2* src = (const uint2*)a.src;
  if (t == 0) count[0] = count[1] = n_roots = 0;
  for (uint32_t i = t; i < a.n_touched; i += nt) {
    const uint32_t x = a.xs[i];
    if (x == CVX_FREE)
      rec[a.ids[i]] = make_uint4(CVX_FREE, CVX_NONE, CVX_NONE, CVX_NONE);
    else
      ((uint32_t*)&rec[a.ids[i]])[0] = device_x(x);
  }
  for (uint32_t i = t; i < a.n_paint; i += nt) atomicMax(&a.mark[a.pids[i]], a.base + i);
  __syncthreads();
  for (uint32_t i = t; i < a.n_paint * a.words; i += nt) {
    const uint32_t j = i / a.words, w = i % a.words, id = a.pids[j];
    if (__hip_atomic_load(&a.mark[id], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.base + j)
      pay[(uint64_t)id * a.words + w] = src[i];
  }
  for (uint32_t i = t; i < a.n_changed; i += nt)
    dirty_roots_of(a.changed[i], a.changed_depth[i], rec, a.R, a.roots, a.root_depth, &n_roots,
                   a.n_nodes, a.mark, a.base);
  __syncthreads();
  const uint32_t n_r = n_roots, o = t & 7u;
  if (t == 0) a.counts[0] = n_r;
  uint32_t now = 0;
  for (uint32_t level = a.first_level; level < a.depth; ++level) {
    const uint32_t n_children = count[now];
    __syncthreads();
    for (uint32_t i = t; i < n_r; i += nt)
      if (a.root_depth[i] == level) {
        const uint32_t slot = atomicAdd(&count[now], 1u);
        if (slot < EDIT_LIST) list[now][slot] = a.roots[i];
      }
    __syncthreads();
    const uint32_t n = count[now];
    if (n > EDIT_LIST) {  // the whole workgroup
      if (t == 0) {
        a.counts[1 + level] = n_children;
        a.state[0] = level;
      }
      return;
    }
    uint32_t* next = a.frontiers + ((level + 1u) & 1u) * (uint64_t)a.cap;
    for (uint32_t i = t / 8u; i < n; i += nt / 8u) {
      const uint32_t P = list[now][i];
      uint32_t seen = 0;  // a node listed twice is processed once
      if (o == 0) seen = atomicExch(&a.mark[P], a.epoch) == a.epoch ? 1u : 0u;
      if (__shfl(seen, (int)(t & 63u & ~7u), 64)) continue;
      const uint32_t C = link_child(rec, P, o, level, a.R, a.n_nodes);
      if (C != CVX_NONE) {
        const uint32_t slot = atomicAdd(&count[now ^ 1u], 1u);
        if (slot < EDIT_LIST) list[now ^ 1u][slot] = C;
        if (slot < a.cap) next[slot] = C;
      }
    }
    __syncthreads();
    if (t == 0) count[now] = 0;
    now ^= 1u;
    __syncthreads();
  }
  if (t == 0) a.state[0] = a.depth;
}

int launch_edit_small(void* stream, const EditArgs& a) {
  hipLaunchKernelGGL(k_edit_small, dim3(1), dim3(1024), 0, (hipStream_t)stream, a);
  return (int)hipGetLastError();
}

int launch_dirty_roots(void* stream, const uint32_t* changed, const uint32_t* depth, uint64_t n,
                       const void* rec, uint32_t R, uint32_t* out, uint32_t* out_depth,
                       uint32_t* out_count, uint64_t n_nodes, uint32_t* mark, uint32_t base) {
  if (!n) return hipSuccess;
  const uint32_t bs = 256;
  hipLaunchKernelGGL(k_dirty_roots, dim3((uint32_t)((n + bs - 1) / bs)), dim3(bs), 0,
                     (hipStream_t)stream, changed, depth, n, (const uint4*)rec, R, out, out_depth,
                     out_count, n_nodes, mark, base);
  return (int)hipGetLastError();
}

int launch_scatter_records(void* stream, const uint32_t* ids, const uint32_t* xs, uint64_t n,
                           void* rec) {
  if (!n) return hipSuccess;
  const uint32_t bs = 256;
  hipLaunchKernelGGL(k_scatter_records, dim3((uint32_t)((n + bs - 1) / bs)), dim3(bs), 0,
                     (hipStream_t)stream, ids, xs, n, (uint4*)rec);
  return (int)hipGetLastError();
}

int launch_scatter_payloads(void* stream, const uint32_t* ids, const void* src, uint64_t n,
                            uint32_t leaf_bytes, void* pay, uint32_t* mark, uint32_t base) {
  if (!n) return hipSuccess;
  const uint32_t bs = 256, words = leaf_bytes / 8;
  hipLaunchKernelGGL(k_stamp_payloads, dim3((uint32_t)((n + bs - 1) / bs)), dim3(bs), 0,
                     (hipStream_t)stream, ids, n, mark, base);
  hipLaunchKernelGGL(k_scatter_payloads, dim3((uint32_t)((n * words + bs - 1) / bs)), dim3(bs), 0,
                     (hipStream_t)stream, ids, (const uint2*)src, n, words, (uint2*)pay, mark,
                     base);
  return (int)hipGetLastError();
}

int launch_links(void* stream, uint32_t first_level, uint32_t last_level, void* rec, uint32_t R,
                 const uint32_t* roots, const uint32_t* root_depth, const uint32_t* n_roots,
                 uint32_t* frontiers, uint32_t cap, uint32_t* counts, uint64_t n_nodes,
                 uint32_t* mark, uint32_t epoch) {
  for (uint32_t level = first_level; level <= last_level; ++level) {
    hipLaunchKernelGGL(k_links_level, dim3(256), dim3(256), 0, (hipStream_t)stream,
                       frontiers + (level & 1u) * (uint64_t)cap, counts, roots, root_depth, n_roots,
                       level, (uint4*)rec, R, frontiers + ((level + 1u) & 1u) * (uint64_t)cap,
                       counts + level + 1, cap, n_nodes, mark, epoch);
    const int e = (int)hipGetLastError();
    if (e != (int)hipSuccess) return e;
  }
  return (int)hipSuccess;
}

}  // namespace cvx
