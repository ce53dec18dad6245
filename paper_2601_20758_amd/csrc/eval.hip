// ROI evaluation: tile-granular range query over the box hierarchy, a
// device-side work plan (prefix sums, heavy tiles split into chunks of
// leaves), and the persistent work-stealing evaluation kernel.
//
// Paper mapping (Section 3.2): Algorithms 2 and 4 give one thread per grid
// node, a range query of radius max(l) per node (Alg. 2) or a loop over all
// particles (Alg. 4), and a kernel sum per node, gathered (no atomics). Here
// one wavefront owns a tile of tx*ty*tz neighbouring nodes; the tile's
// candidate leaves come from one range query per tile; each lane takes one
// particle of a 64-particle leaf and evaluates it against every node of the
// tile, exploiting the grid's separability (the per-axis squared scaled
// distances are computed once per particle and node row); the per-node sums
// are combined across lanes with a transposing butterfly of wavefront
// shuffles. Heavy tiles are split into chunks of leaves whose partial sums
// are combined in a fixed order, so every grid is bitwise reproducible
// whatever batch it runs in.
#include <type_traits>

#include "sfk_device.h"

namespace sfk {

__device__ __forceinline__ int find_roi(const RoiDev* __restrict__ rois, int n_rois, int64_t t) {
  int lo = 0, hi = n_rois - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (rois[mid].tile_base <= t)
      lo = mid;
    else
      hi = mid - 1;
  }
  return lo;
}

struct TileGeo {
  int r;
  int i0, j0, k0;
  double lo[3], hi[3];
};

template <int TX, int TY, int TZ>
__device__ __forceinline__ TileGeo tile_geo(const RoiDev* __restrict__ rois, int n_rois,
                                            const double* __restrict__ coords, int64_t t) {
  TileGeo g;
  g.r = find_roi(rois, n_rois, t);
  const RoiDev& R = rois[g.r];
  const int64_t lt = t - R.tile_base;
  const int ti = (int)(lt % R.ntile[0]);
  const int tj = (int)((lt / R.ntile[0]) % R.ntile[1]);
  const int tk = (int)(lt / ((int64_t)R.ntile[0] * R.ntile[1]));
  g.i0 = ti * TX;
  g.j0 = tj * TY;
  g.k0 = tk * TZ;
  const int i1 = min(g.i0 + TX, R.res[0]) - 1;
  const int j1 = min(g.j0 + TY, R.res[1]) - 1;
  const int k1 = min(g.k0 + TZ, R.res[2]) - 1;
  const double* cx = coords + R.coord_off;
  const double* cy = cx + R.res[0];
  const double* cz = cy + R.res[1];
  g.lo[0] = cx[g.i0];
  g.hi[0] = cx[i1];
  g.lo[1] = cy[g.j0];
  g.hi[1] = cy[j1];
  g.lo[2] = cz[g.k0];
  g.hi[2] = cz[k1];
  return g;
}

// Box test shared by the count, fill, evaluation and debug walks.
__device__ __forceinline__ bool tile_box_test(const TreeView& tv, const RoiDev& R,
                                              const TileGeo& g, const NodeBox& b, int gidx) {
  float ihx = R.ih[0], ihy = R.ih[1], ihz = R.ih[2];
  if (R.pp_mode != PP_UNIFORM) {
    const float4 m = tv.node_ih[gidx];
    ihx = m.x;
    ihy = m.y;
    ihz = m.z;
  }
  return box_gap_u2(b, g.lo[0], g.lo[1], g.lo[2], g.hi[0], g.hi[1], g.hi[2], ihx, ihy, ihz) <
         (double)R.c2;
}

// ---------------------------------------------------------------------------
// ROI coordinate tables: x_i = lo + (i*(hi-lo))/(res-1) in double.
// ---------------------------------------------------------------------------

__device__ __forceinline__ double node_coord(const RoiDev& R, int k, int i) {
  const double lo = R.lo[k], hi = R.hi[k];
  const double num = __dmul_rn((double)i, __dsub_rn(hi, lo));
  return __dadd_rn(lo, __ddiv_rn(num, (double)(R.res[k] - 1)));
}

__device__ void roi_list_walk(const TreeView& tv, int r, const RoiDev& R, int32_t* stack,
                              int32_t* __restrict__ roi_leaves, int32_t* __restrict__ roi_nl);

// One block per ROI: the coordinate table, then (first wavefront) the ROI's
// leaf list, described below.
__global__ __launch_bounds__(256) void k_roi_coords(TreeView tv, const BatchHdr* __restrict__ hdr,
                                                    const RoiDev* __restrict__ rois,
                                                    double* __restrict__ coords,
                                                    int32_t* __restrict__ roi_leaves,
                                                    int32_t* __restrict__ roi_nl) {
  __shared__ int32_t lds_stack[SFK_STACK];
  if ((int)blockIdx.x >= hdr->n_rois) return;
  const RoiDev& R = rois[blockIdx.x];
  const int tot = R.res[0] + R.res[1] + R.res[2];
  for (int q = threadIdx.x; q < tot; q += blockDim.x) {
    int k = 0, i = q;
    if (i >= R.res[0]) {
      i -= R.res[0];
      k = 1;
      if (i >= R.res[1]) {
        i -= R.res[1];
        k = 2;
      }
    }
    coords[R.coord_off + q] = node_coord(R, k, i);
  }
  if (threadIdx.x < 64) roi_list_walk(tv, (int)blockIdx.x, R, lds_stack, roi_leaves, roi_nl);
}

hipError_t launch_roi_coords(TreeView tv, const BatchHdr* hdr, const RoiDev* rois, int grid_rois,
                             double* coords, int32_t* roi_leaves, int32_t* roi_nl,
                             hipStream_t s) {
  if (grid_rois <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_roi_coords, dim3(grid_rois), dim3(256), 0, s, tv, hdr, rois, coords,
                     roi_leaves, roi_nl);
  return hipGetLastError();
}

// ---------------------------------------------------------------------------
// ROI leaf lists: one wavefront per ROI walks the hierarchy once with the
// box of all the ROI's nodes and keeps the passing leaves, ascending, when
// there are at most kRoiListCap of them (else the count is -1 and every tile
// walks). A tile's box lies inside the ROI's and the test is monotone in the
// box (rounded subtractions, products with non-negative inverse bandwidths
// and sums are monotone), so every leaf a tile's walk yields is in the list;
// a tile then tests the list's leaves directly and yields the same leaves in
// the same order, without descending from the root.
// ---------------------------------------------------------------------------

// The box of the first and last nodes, computed as the coordinate table
// computes them.
__device__ void roi_list_walk(const TreeView& tv, int r, const RoiDev& R, int32_t* stack,
                              int32_t* __restrict__ roi_leaves, int32_t* __restrict__ roi_nl) {
  const int lane = lane_id();
  TileGeo g;
  g.r = r;
  g.i0 = g.j0 = g.k0 = 0;
  for (int k = 0; k < 3; ++k) {
    g.lo[k] = node_coord(R, k, 0);
    g.hi[k] = node_coord(R, k, R.res[k] - 1);
  }
  int32_t* out = roi_leaves + (int64_t)r * kRoiListCap;
  int cnt = 0;
  traverse_until(
      tv, stack,
      [&](const NodeBox& b, int gidx) { return tile_box_test(tv, R, g, b, gidx); },
      [&](int child, bool pass, uint64_t mask) {
        const int pos = cnt + popc64(mask & lanemask_lt());
        if (pass && pos < kRoiListCap) out[pos] = child;
        cnt += popc64(mask);
        return cnt <= kRoiListCap;
      });
  if (lane == 0) roi_nl[r] = cnt <= kRoiListCap ? cnt : -1;
}

// A tile's candidate leaves: from its ROI's list when there is one, else by
// a walk from the root. leaves(child, pass, mask) per group of up to 64, in
// ascending leaf order either way.
template <class LeafF>
__device__ __forceinline__ void tile_leaves(const TreeView& tv, int32_t* stack, const RoiDev& R,
                                            const TileGeo& g,
                                            const int32_t* __restrict__ roi_leaves,
                                            const int32_t* __restrict__ roi_nl, LeafF leaves) {
  const int nl = roi_nl[g.r];
  if (nl >= 0) {
    const int32_t* list = roi_leaves + (int64_t)g.r * kRoiListCap;
    for (int i0 = 0; i0 < nl; i0 += 64) {
      const int i = i0 + lane_id();
      int child = 0;
      bool pass = false;
      if (i < nl) {
        child = list[i];
        const int gi = tv.level_off[0] + child;
        pass = tile_box_test(tv, R, g, tv.nodes[gi], gi);
      }
      leaves(child, pass, ballot(pass));
    }
    return;
  }
  traverse(
      tv, stack, [&](const NodeBox& b, int gidx) { return tile_box_test(tv, R, g, b, gidx); },
      leaves);
}

// ---------------------------------------------------------------------------
// tile range query: count pass and fill pass (one wavefront per tile)
// ---------------------------------------------------------------------------

template <int TX, int TY, int TZ>
__global__ __launch_bounds__(256) void k_tile_count(TreeView tv, const BatchHdr* __restrict__ hdr,
                                                    const RoiDev* __restrict__ rois,
                                                    const double* __restrict__ coords,
                                                    const int32_t* __restrict__ roi_leaves,
                                                    const int32_t* __restrict__ roi_nl,
                                                    int32_t* __restrict__ tile_cnt,
                                                    int32_t* __restrict__ tile_fit,
                                                    int32_t* __restrict__ tile_done,
                                                    int32_t* __restrict__ tile_slots) {
  __shared__ int32_t lds_stack[4][SFK_STACK];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t n_tiles = hdr->n_tiles;
  const int n_rois = hdr->n_rois;
  const int slot_cap = hdr->slot_cap;
  const int poison = hdr->debug_poison;
  for (int64_t t = (int64_t)blockIdx.x * 4 + wave; t < n_tiles; t += (int64_t)gridDim.x * 4) {
    const TileGeo g = tile_geo<TX, TY, TZ>(rois, n_rois, coords, t);
    const RoiDev& R = rois[g.r];
    int cnt = 0;
    int32_t* slot = tile_slots + t * slot_cap;
    tile_leaves(tv, lds_stack[wave], R, g, roi_leaves, roi_nl,
                [&](int child, bool pass, uint64_t mask) {
                  const int pos = cnt + popc64(mask & lanemask_lt());
                  if (pass && pos < slot_cap)
                    slot[pos] = (poison & 1) && pos >= 64 ? tv.n_leaves + child : child;
                  cnt += popc64(mask);
                });
    if (lane == 0) {
      tile_cnt[t] = cnt;
      tile_fit[t] = (R.chunk << kFitChunk) | (R.block_log2 << kFitBlock);
      tile_done[t] = 0;
    }
  }
}

// How a tile is evaluated. Lists: its leaf list and partial slots fit the
// buffers, one work item per chunk (or block) of its list. Listed whole: only
// the list fits, one work item for all of it. Walk per item: only the partial
// slots fit; each work item walks the hierarchy and evaluates its leaves. Walk
// whole tile: one work item walks and evaluates everything. All visit the same
// leaves in the same order, add a chunk's terms in float (each wavefront lane
// its own, then over the lanes), a block's chunks in double and the blocks in
// double, so the sums are bitwise equal.
static constexpr int kModeWalkTile = 0;
static constexpr int kModeLists = 1;
static constexpr int kModeWalkItem = 2;
static constexpr int kModeListTile = 3;
__device__ __forceinline__ bool mode_listed(int mode) {
  return mode == kModeLists || mode == kModeListTile;
}
__device__ __forceinline__ bool mode_whole(int mode) {
  return mode == kModeWalkTile || mode == kModeListTile;
}
// of a tile_fit entry
__device__ __forceinline__ int fit_mode(int fit) { return fit & 3; }
__device__ __forceinline__ int fit_chunk(int fit) {
  return (fit & ((1 << kFitCoarse) - 1)) >> kFitChunk;
}
__device__ __forceinline__ int fit_coarse(int fit) { return (fit >> kFitCoarse) & 1; }
__device__ __forceinline__ int fit_block(int fit) { return fit >> kFitBlock; }
// leaves of a work item
__device__ __forceinline__ int fit_span(int fit) {
  return fit_chunk(fit) << (fit_coarse(fit) ? fit_block(fit) : 0);
}

template <int TX, int TY, int TZ>
__global__ __launch_bounds__(256) void k_tile_fill(
    TreeView tv, const BatchHdr* __restrict__ hdr, const RoiDev* __restrict__ rois,
    const double* __restrict__ coords, const int32_t* __restrict__ roi_leaves,
    const int32_t* __restrict__ roi_nl, const int32_t* __restrict__ tile_slots,
    const int32_t* __restrict__ tile_cnt, const int32_t* __restrict__ tile_fit,
    const int64_t* __restrict__ leaf_off,
    const int64_t* __restrict__ chunk_off, int32_t* __restrict__ leaves,
    int32_t* __restrict__ item_tile, int32_t* __restrict__ claims, double* __restrict__ partials,
    const int64_t* __restrict__ partial_off) {
  __shared__ int32_t lds_stack[4][SFK_STACK];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t n_tiles = hdr->n_tiles;
  const int n_rois = hdr->n_rois;
  const int slot_cap = hdr->slot_cap;
  const int poison = hdr->debug_poison;
  for (int64_t t = (int64_t)blockIdx.x * 4 + wave; t < n_tiles; t += (int64_t)gridDim.x * 4) {
    const int64_t c0 = chunk_off[t], c1 = min(chunk_off[t + 1], hdr->item_cap);
    for (int64_t c = c0 + lane; c < c1; c += 64) item_tile[c] = (int32_t)t;
    const int tc = tile_cnt[t];
    if (tc == 0) {
      // no candidate leaf, hence no work item: the tile's nodes are zero
      constexpr int T = TX * TY * TZ;
      const int r = find_roi(rois, n_rois, t);
      const RoiDev& R = rois[r];
      const int64_t lt = t - R.tile_base;
      const int ti = (int)(lt % R.ntile[0]) * TX, tj = (int)((lt / R.ntile[0]) % R.ntile[1]) * TY;
      const int tk = (int)(lt / ((int64_t)R.ntile[0] * R.ntile[1])) * TZ;
      for (int q = lane; q < T; q += 64) {
        const int gi = ti + q % TX, gj = tj + (q / TX) % TY, gk = tk + q / (TX * TY);
        if (gi < R.res[0] && gj < R.res[1] && gk < R.res[2])
          R.out[(int64_t)gi + (int64_t)R.res[0] * ((int64_t)gj + (int64_t)R.res[1] * gk)] = 0.0f;
      }
      continue;
    }
    const int mode = fit_mode(tile_fit[t]);
    if (hdr->splat && !mode_whole(mode) && chunk_off[t + 1] - c0 > 1) {
      // a brick split over several work items: its integer node sums start at 0
      constexpr int64_t T = (int64_t)TX * TY * TZ;
      unsigned long long* sums = (unsigned long long*)(partials) + partial_off[t] * T;
      for (int64_t i = lane; i < T; i += 64) sums[i] = 0ull;
    }
    if (!mode_listed(mode)) continue;
    int32_t* out = leaves + leaf_off[t];
    if (tc <= slot_cap) {
      // the count pass kept the whole list, in walk order; an entry that is
      // not a leaf of the tree is an internal error: flag it, copy leaf 0
      bool bad = false;
      for (int i = lane; i < tc; i += 64) {
        int v = tile_slots[t * slot_cap + i];
        if ((unsigned)v >= (unsigned)tv.n_leaves) {
          bad = true;
          v = 0;
        }
        out[i] = (poison & 2) && i >= 64 ? tv.n_leaves + v : v;
      }
      if (bad) claims[kErrWord] = 1;
      continue;
    }
    const TileGeo g = tile_geo<TX, TY, TZ>(rois, n_rois, coords, t);
    const RoiDev& R = rois[g.r];
    int cnt = 0;
    tile_leaves(tv, lds_stack[wave], R, g, roi_leaves, roi_nl,
                [&](int child, bool pass, uint64_t mask) {
                  if (pass) out[cnt + popc64(mask & lanemask_lt())] = child;
                  cnt += popc64(mask);
                });
  }
}

// ---------------------------------------------------------------------------
// work plan: per tile, leaf_off (prefix of candidate leaves), partial_off
// (prefix of partial-sum slots of split tiles), tile_fit (the count pass left
// the tile's chunk and block there: how the tile is evaluated, above) and
// chunk_off (prefix of work items). Three launches over blocks of kPlanNT
// consecutive tiles (coalesced; no block waits for another): per-block sums of
// leaves and of the partial slots that chunks and that blocks would need; then
// each block adds the sums of the blocks before it, scans its tiles, decides
// each tile's mode from the prefixes and its number of work items (kept in
// chunk_off) and sums those; then the same for the items.
// The batch's items are chunks if its partial slots last for that and blocks
// otherwise: short chunks need up to eight times the slots, and where these run
// out (a bounded workspace, very many or very heavy tiles) the tiles past the
// last slot would be one item each, the heaviest of them the last to end: a
// 64^3 grid of 20M points in wide supports took 3.3 ms so, 1.1 in blocks.
// Block 0 of the last launch writes the totals. A batch of at most kPlanNT
// tiles takes one launch of one block instead.
// ---------------------------------------------------------------------------

static constexpr int kPlanNT = 1024;

// Work items of a tile that is split where it can be. A tile with no candidate
// leaf has none: the fill pass writes its (zero) nodes.
__device__ __forceinline__ int64_t plan_items(int64_t cnt, int span) {
  return cnt > 0 ? (cnt + span - 1) / span : 0;
}

// Partial slots a tile of n items needs: one per item when it is split (its
// items' sums are combined in order), or one for a split brick (its items add
// integer node sums into that one slot).
__device__ __forceinline__ int64_t plan_partials(int64_t n, int splat) {
  return n > 1 ? (splat ? 1 : n) : 0;
}

// A tile's mode, and the number of its items.
__device__ __forceinline__ int plan_mode(bool fit_list, bool fit_slots, int64_t n, int splat) {
  if (fit_list) return fit_slots ? kModeLists : kModeListTile;
  // bricks never walk per item: their items stay within the list capacity
  return fit_slots && n > 1 && !splat ? kModeWalkItem : kModeWalkTile;
}
__device__ __forceinline__ int64_t plan_count(int64_t cnt, int64_t n, int mode) {
  return cnt > 0 && mode_whole(mode) ? 1 : n;
}

// sum of v over the block (every thread gets it)
__device__ __forceinline__ int64_t block_sum(int64_t v, int64_t* lds) {
  int64_t tot;
  (void)block_excl_scan<kPlanNT>(v, &tot, lds);
  return tot;
}

// sum of bs[kPlanSums * i + k] over the blocks i < nb (each wavefront by itself
// where its lanes hold them all)
__device__ __forceinline__ int64_t sum_before(const int64_t* __restrict__ bs, int k, int64_t nb,
                                              int64_t* lds) {
  if (nb <= 64) return wave_sum(lane_id() < nb ? bs[kPlanSums * lane_id() + k] : (int64_t)0);
  int64_t v = 0;
  for (int64_t i = threadIdx.x; i < nb; i += kPlanNT) v += bs[kPlanSums * i + k];
  return block_sum(v, lds);
}

__global__ __launch_bounds__(kPlanNT) void k_plan_sums(const int32_t* __restrict__ tile_cnt,
                                                       const int32_t* __restrict__ tile_fit,
                                                       const BatchHdr* __restrict__ hdr,
                                                       int64_t* __restrict__ bs) {
  __shared__ int64_t lds[kPlanNT / 64];
  const int64_t n_tiles = hdr->n_tiles;
  const int64_t t = (int64_t)blockIdx.x * kPlanNT + threadIdx.x;
  if ((int64_t)blockIdx.x * kPlanNT >= n_tiles) return;  // whole block past the end
  const int64_t cnt = t < n_tiles ? tile_cnt[t] : 0;
  const int fit = t < n_tiles ? tile_fit[t] : 1 << kFitChunk;
  const int64_t sl = block_sum(cnt, lds);
  const int64_t sf = block_sum(plan_partials(plan_items(cnt, fit_span(fit)), hdr->splat), lds);
  const int64_t sc = block_sum(plan_partials(plan_items(cnt, fit_span(fit | 1 << kFitCoarse)), hdr->splat), lds);
  if (threadIdx.x == 0) {
    bs[kPlanSums * blockIdx.x] = sl;
    bs[kPlanSums * blockIdx.x + 1] = sf;
    bs[kPlanSums * blockIdx.x + 2] = sc;
  }
}

__global__ __launch_bounds__(kPlanNT) void k_plan_modes(const int32_t* __restrict__ tile_cnt,
                                                        const BatchHdr* __restrict__ hdr,
                                                        int64_t* __restrict__ bs,
                                                        int64_t* __restrict__ leaf_off,
                                                        int64_t* __restrict__ partial_off,
                                                        int64_t* __restrict__ chunk_off,
                                                        int32_t* __restrict__ tile_fit) {
  __shared__ int64_t lds[kPlanNT / 64];
  const int64_t n_tiles = hdr->n_tiles;
  const int64_t leaf_cap = hdr->leaf_cap;
  const int64_t partial_cap = hdr->partial_cap;
  if ((int64_t)blockIdx.x * kPlanNT >= n_tiles) return;
  const int64_t nb = (n_tiles + kPlanNT - 1) / kPlanNT;
  const bool coarse = sum_before(bs, 1, nb, lds) > partial_cap;
  const int64_t base_l = sum_before(bs, 0, blockIdx.x, lds);
  const int64_t base_p = sum_before(bs, coarse ? 2 : 1, blockIdx.x, lds);
  const int64_t t = (int64_t)blockIdx.x * kPlanNT + threadIdx.x;
  const bool v = t < n_tiles;
  const int64_t cnt = v ? tile_cnt[t] : 0;
  const int fit = (v ? tile_fit[t] : 1 << kFitChunk) | (coarse ? 1 << kFitCoarse : 0);
  const int64_t n = plan_items(cnt, fit_span(fit));
  const int64_t pneed = plan_partials(n, hdr->splat);
  int64_t tot;
  const int64_t lo = base_l + block_excl_scan<kPlanNT>(cnt, &tot, lds);
  const int64_t po = base_p + block_excl_scan<kPlanNT>(pneed, &tot, lds);
  const int mode = plan_mode(lo + cnt <= leaf_cap, pneed == 0 || po + pneed <= partial_cap, n,
                             hdr->splat);
  const int64_t nit = plan_count(cnt, n, mode);
  if (v) {
    leaf_off[t] = lo;
    partial_off[t] = po;
    chunk_off[t] = nit;
    tile_fit[t] = fit | mode;
  }
  const int64_t si = block_sum(nit, lds);
  if (threadIdx.x == 0) bs[kPlanSums * blockIdx.x + 3] = si;
}

__global__ __launch_bounds__(kPlanNT) void k_plan_items(BatchHdr* __restrict__ hdr,
                                                        int32_t* __restrict__ claims,
                                                        const int64_t* __restrict__ bs,
                                                        int64_t* __restrict__ leaf_off,
                                                        int64_t* __restrict__ partial_off,
                                                        int64_t* __restrict__ chunk_off) {
  __shared__ int64_t lds[kPlanNT / 64];
  const int64_t n_tiles = hdr->n_tiles;
  const int64_t nb = (n_tiles + kPlanNT - 1) / kPlanNT;
  if (blockIdx.x == 0) {
    // totals (block 0 runs even for an empty batch)
    const int64_t partial_cap = hdr->partial_cap;
    const int64_t tl = sum_before(bs, 0, nb, lds);
    const int64_t tf = sum_before(bs, 1, nb, lds);
    const bool coarse = tf > partial_cap;
    const int64_t tp = coarse ? sum_before(bs, 2, nb, lds) : tf;
    const int64_t tc = sum_before(bs, 3, nb, lds);
    // every thread of this block has read the header before thread 0 writes it
    __syncthreads();
    if (threadIdx.x < kClaimSlices) claims[threadIdx.x * kClaimStride] = 0;
    if (threadIdx.x == 0) {
      leaf_off[n_tiles] = tl;
      partial_off[n_tiles] = tp;
      chunk_off[n_tiles] = tc;
      hdr->total_leaves = tl;
      hdr->n_items = tc;
      hdr->total_partials = tp;
      hdr->fine_partials = tf;
      hdr->coarse = coarse ? 1 : 0;
    }
  }
  if ((int64_t)blockIdx.x >= nb) return;
  const int64_t base_c = sum_before(bs, 3, blockIdx.x, lds);
  const int64_t t = (int64_t)blockIdx.x * kPlanNT + threadIdx.x;
  const bool v = t < n_tiles;
  const int64_t nit = v ? chunk_off[t] : 0;
  int64_t tot;
  const int64_t co = base_c + block_excl_scan<kPlanNT>(nit, &tot, lds);
  if (v) chunk_off[t] = co;
}

// ---------------------------------------------------------------------------
// evaluation
// ---------------------------------------------------------------------------

// One split stage of the transposing reduction: lanes with bit OFF keep the
// upper half of the live accumulators, the others the lower half; each adds
// its partner's copy of the half it keeps.
template <int N, int OFF, typename A, int T>
__device__ __forceinline__ void xsplit(A (&acc)[T]) {
  const bool up = (lane_id() & OFF) != 0;
#pragma unroll
  for (int i = 0; i < N / 2; ++i) {
    const A lo = acc[i], hi = acc[i + N / 2];
    const A send = up ? lo : hi;
    const A keep = up ? hi : lo;
    acc[i] = keep + __shfl_xor(send, OFF, 64);
  }
}

template <int OFF, typename A, int T>
__device__ __forceinline__ void xfold(A (&acc)[T]) {
#pragma unroll
  for (int i = 0; i < T; ++i) acc[i] = acc[i] + __shfl_xor(acc[i], OFF, 64);
}

template <int OFF, typename A, int T>
__device__ __forceinline__ void fold_down(A (&acc)[T]) {
  if constexpr (OFF >= T && OFF >= 1) {
    xfold<OFF>(acc);
    fold_down<OFF / 2>(acc);
  }
}

template <int N, typename A, int T>
__device__ __forceinline__ void split_down(A (&acc)[T]) {
  if constexpr (N >= 2) {
    xsplit<N, N / 2>(acc);
    split_down<N / 2>(acc);
  }
}

// Reduce T per-lane accumulators over the 64 lanes. Afterwards lane l holds
// node (l * NPL + m) in acc[m] for m < NPL = max(1, T/64); for T < 64 the
// lanes first fold in halves down to T lanes' worth, so lane l holds node
// l mod T. Fixed order: deterministic.
template <typename A, int T>
__device__ __forceinline__ void reduce_nodes(A (&acc)[T]) {
  if constexpr (T >= 64) {
    xsplit<T, 32>(acc);
    xsplit<T / 2, 16>(acc);
    xsplit<T / 4, 8>(acc);
    xsplit<T / 8, 4>(acc);
    xsplit<T / 16, 2>(acc);
    xsplit<T / 32, 1>(acc);
  } else {
    fold_down<32>(acc);
    split_down<T>(acc);
  }
}

// leaf ids a walking work item holds (two blocks of 64 and a step's 64 more)
constexpr int kWalkRing = 256;

// The hand-over of a split tile's sums from the items that made them to the
// last one, which combines them. Sums are stored and loaded as relaxed atomics
// of agent scope, which go past the L2s of the eight XCDs to the memory they
// share (the memory model of the gfx942 family in LLVM's user guide for the
// AMDGPU backend), and an item waits for its own before it counts itself done.
// An agent release would write back, and an acquire invalidate, the XCD's whole
// L2 for the plain stores and loads that might go with them; there must be
// none: whatever is handed over goes through these functions (or through
// atomicAdd). With a device-wide fence per chunk the 128^3 MBE estimate of 2.1M
// particles in chunks of 64 leaves (three a tile) took 3.63 ms, and 1.93
// without, in chunks of 32 5.57 and 2.06.
template <typename V>
__device__ __forceinline__ void hand_over(V* p, V v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename V>
__device__ __forceinline__ V handed_over(const V* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void agent_writes_done() {
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// -log2(e)/2 in double: exp(-u2/2) = exp2(KG * u2)
#define SFK_KG64 (-0.72134752044448170368)

// The evaluation kernel. Template parameters: tile shape (TX, TY, TZ), kernel
// (Epanechnikov / truncated Gaussian), bandwidth source (uniform, per-particle
// isotropic, per-particle anisotropic) and counting mode. Membership and the
// Epanechnikov value 1 - u2 are double (same rate as unpacked float32 on
// gfx950), each term then rounded once to float32 where the sums are; the
// Gaussian factors are float32 exp2 of the double exponents.
//
// Bound by VALU issue, two thirds busy, half of it culling (a 4x4x4 tile whose
// supports span 11 nodes tests four particles for each that reaches it) and
// half evaluation, about 200 instructions for 64 particles and 64 nodes. Three
// wavefronts a SIMD (at most 168 registers): with two, and double sums of
// 4x4x4 tiles, the 128^3 pilot grid of 2.1M particles took 8% longer, with
// four the sums spill. That grid takes 1.0 ms (1.37 with the cull in double,
// a maximum per term, a queue moved to the front after each batch and ids read
// from LDS), the 101x87x93 per-point grid of 1M points 0.18 ms (0.39).
// (The order of the arguments keeps the compiler from loading and spilling them
// eight registers at a time, with scratch memory for it.)
template <int TX, int TY, int TZ, int KK, int PP, bool CNT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void k_eval(
    TreeView tv, const RoiDev* __restrict__ rois, const double* __restrict__ coords,
    const BatchHdr* __restrict__ hdr, int32_t* __restrict__ claims,
    const int64_t* __restrict__ leaf_off, const int64_t* __restrict__ chunk_off,
    const int64_t* __restrict__ partial_off, const int32_t* __restrict__ tile_cnt,
    const int32_t* __restrict__ tile_fit, const int32_t* __restrict__ leaves,
    const int32_t* __restrict__ item_tile, double* __restrict__ partials,
    int32_t* __restrict__ tile_done) {
  constexpr int T = TX * TY * TZ;
  constexpr int NPL = T >= 64 ? T / 64 : 1;
  // Per-lane node accumulators are float32: a lane adds one term per drained
  // batch of 64 particles (at most one per leaf of a chunk), the 64 lanes are
  // combined by a 6-level tree and the chunks of a tile in double.
  // Epanechnikov tiles of at most 16 nodes accumulate in double (registers
  // allow it), which also saves the per-pair conversion.
  constexpr bool kDoubleAcc = T <= 16 && KK == KK_EPAN && !CNT;
  using Acc = std::conditional_t<kDoubleAcc, double, float>;
  // particle buffers of the leaf pipeline (four were no faster and spilled);
  // the queue is a ring that takes two leaves on top of a remainder below 64
  constexpr int NB = 2;
  constexpr int QCAP = 256;
  __shared__ int32_t lds_stack[4][SFK_STACK];
  __shared__ int32_t lds_walk[4][kWalkRing];
  __shared__ float4 lds_qpts[4][QCAP];
  __shared__ float4 lds_qprm[4][PP == PP_ANISO ? QCAP : 1];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t n_items = min(hdr->n_items, hdr->item_cap);  // equal by construction
  const int n_rois = hdr->n_rois;
  // XCD-aware work stealing. Workgroups are dispatched round-robin over the
  // 8 XCDs, each with its own L2. The item list is cut into kClaimSlices
  // contiguous (hence spatially coherent) slices, 8 per XCD, each with its own
  // counter on its own cache line: device-scope atomics serialize per line,
  // so spreading them is what lets many light items be claimed quickly. A
  // wave claims single items from its home slice (one of its XCD's eight);
  // when that slice is exhausted, the 64 lanes read all 64 counters at once
  // (plain loads) and the wave moves to the first slice with items left in
  // its order: its XCD's other slices, then the other XCDs'. Which wave takes
  // an item never changes what the item computes.
  const int xcd = blockIdx.x & 7;
  const int sub = (int)(((blockIdx.x >> 3) * 4 + wave) & 7);
  auto slice_at = [&](int pos) { return ((xcd + (pos >> 3)) & 7) * 8 + ((sub + pos) & 7); };
  auto slice_begin = [&](int sl) { return n_items * sl / kClaimSlices; };
  int cur = slice_at(0);
  while (true) {
    int64_t item = -1;
    while (true) {
      const int64_t b = slice_begin(cur), e = slice_begin(cur + 1);
      int idx = 0;
      if (b < e && lane == 0) idx = atomicAdd(&claims[cur * kClaimStride], 1);
      idx = __shfl(idx, 0, 64);
      if (b + idx < e) {
        item = b + idx;
        break;
      }
      const int my = slice_at(lane);
      const int64_t mb = slice_begin(my), me = slice_begin(my + 1);
      const int seen =
          __hip_atomic_load(&claims[my * kClaimStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const uint64_t open = __ballot(mb + seen < me);
      if (open == 0) break;
      cur = slice_at(__ffsll((unsigned long long)open) - 1);
    }
    if (item < 0) break;
    const int t = wave_uniform(item_tile[item]);
    const TileGeo g = tile_geo<TX, TY, TZ>(rois, n_rois, coords, t);
    const RoiDev& R = rois[g.r];
    const double* cx = coords + R.coord_off;
    const double* cy = cx + R.res[0];
    const double* cz = cy + R.res[1];
    double nx[TX], ny[TY], nz[TZ];
#pragma unroll
    for (int i = 0; i < TX; ++i) nx[i] = cx[min(g.i0 + i, R.res[0] - 1)];
#pragma unroll
    for (int j = 0; j < TY; ++j) ny[j] = cy[min(g.j0 + j, R.res[1] - 1)];
#pragma unroll
    for (int k = 0; k < TZ; ++k) nz[k] = cz[min(g.k0 + k, R.res[2] - 1)];
    const float uih0 = R.ih[0], uih1 = R.ih[1], uih2 = R.ih[2];
    const double c2 = R.c2;
    // the tile box for the particle cull (keep_of): centre, half widths and
    // the squared reach, for a uniform bandwidth in units of the reach
    constexpr double kWide = 1.0 + 0x1p-20;
    const double reach = 1.0 / (sqrt(c2) * kWide);
    float bc[3], bh[3], us[3], uh[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      bc[k] = (float)(0.5 * (g.lo[k] + g.hi[k]));
      const double h = fmax(g.hi[k] - (double)bc[k], (double)bc[k] - g.lo[k]) * kWide;
      const double sc = (double)R.ih[k] * reach;
      bh[k] = (float)h;
      us[k] = (float)sc;
      uh[k] = (float)(h * sc);
    }
    const float cc = (float)(c2 * (kWide * kWide));
    const int cnt = tile_cnt[t];  // > 0: tiles with no candidate leaf have no work item
    const int fit = wave_uniform(tile_fit[t]), mode = fit_mode(fit);
    const int chunk = fit_chunk(fit), span = fit_span(fit);
    const int nit = (cnt + span - 1) / span;

    Acc acc[T];

    // Per-wave queue of particles whose support reaches the tile box. Each
    // leaf is loaded one particle per lane and culled against the tile (in
    // float32 with a margin, keep_of: a culled particle reaches no node);
    // survivors are appended in leaf-then-lane order and evaluated 64 at a
    // time, so lanes stay busy with particles that can matter. The order is
    // fixed, hence so are the sums.
    float4* qp = lds_qpts[wave];
    float4* qa = lds_qprm[wave];
    int qn = 0, qh = 0;  // particles queued, place of the first

    auto eval_point = [&](const float4 p, const float4 prm) __attribute__((always_inline)) {
      float ihx, ihy, ihz;
      double w = 1.0;
      if constexpr (PP == PP_UNIFORM) {
        ihx = uih0;
        ihy = uih1;
        ihz = uih2;
      } else if constexpr (PP == PP_ISO) {
        ihx = ihy = ihz = p.w;
        const double ih = (double)p.w;
        w = (ih * ih) * ih;
      } else {
        ihx = prm.x;
        ihy = prm.y;
        ihz = prm.z;
        w = (double)prm.w;
      }
      const double px = p.x, py = p.y, pz = p.z;
      double sx[TX], sy[TY], sz[TZ];
#pragma unroll
      for (int i = 0; i < TX; ++i) {
        const double u = (nx[i] - px) * (double)ihx;
        sx[i] = u * u;
      }
#pragma unroll
      for (int j = 0; j < TY; ++j) {
        const double u = (ny[j] - py) * (double)ihy;
        sy[j] = u * u;
      }
#pragma unroll
      for (int k = 0; k < TZ; ++k) {
        const double u = (nz[k] - pz) * (double)ihz;
        sz[k] = u * u;
      }
      // A row (i, j) of nodes where no lane's particle reaches (sx + sy >= c2
      // for all 64; u2 only grows with sz) adds exact zeros: skipped.
      if constexpr (CNT) {
#pragma unroll
        for (int j = 0; j < TY; ++j)
#pragma unroll
          for (int i = 0; i < TX; ++i) {
            const double tt = sx[i] + sy[j];
            if (!ballot(tt < c2)) continue;
#pragma unroll
            for (int k = 0; k < TZ; ++k) {
              const double u2 = tt + sz[k];
              acc[i + TX * (j + TY * k)] += (u2 < c2) ? 1.0f : 0.0f;
            }
          }
      } else if constexpr (KK == KK_EPAN) {
        // 1 - u2 = ((1 - sx) - sy) - sz in double, clamped to [0, 1] (it never
        // exceeds 1; the clamp is an output modifier of the subtraction, a
        // maximum would be an instruction), then added, or multiplied and
        // added: in double for tiles of at most 16 nodes, two instructions a
        // node, after a conversion to float32 for larger ones. The rounding
        // differs from 1 - ((sx + sy) + sz) by at most an ulp of double or
        // two; a term at the support's edge is then up to 1e-16, not 0.
        double ox[TX];
#pragma unroll
        for (int i = 0; i < TX; ++i) ox[i] = 1.0 - sx[i];
#pragma unroll
        for (int j = 0; j < TY; ++j)
#pragma unroll
          for (int i = 0; i < TX; ++i) {
            const double om = ox[i] - sy[j];
            if (!ballot(om > 0.0)) continue;
#pragma unroll
            for (int k = 0; k < TZ; ++k) {
              const double v = fmin(fmax(om - sz[k], 0.0), 1.0);
              Acc& a = acc[i + TX * (j + TY * k)];
              if constexpr (PP == PP_UNIFORM)
                a = a + (Acc)v;
              else
                a = fma((Acc)w, (Acc)v, a);
            }
          }
      } else {
        float ex[TX], ey[TY], ez[TZ];
        const float wf = (float)w;
#pragma unroll
        for (int i = 0; i < TX; ++i) {
          ex[i] = __builtin_amdgcn_exp2f((float)(SFK_KG64 * sx[i]));
          if constexpr (PP != PP_UNIFORM) ex[i] = ex[i] * wf;
        }
#pragma unroll
        for (int j = 0; j < TY; ++j) ey[j] = __builtin_amdgcn_exp2f((float)(SFK_KG64 * sy[j]));
#pragma unroll
        for (int k = 0; k < TZ; ++k) ez[k] = __builtin_amdgcn_exp2f((float)(SFK_KG64 * sz[k]));
#pragma unroll
        for (int j = 0; j < TY; ++j)
#pragma unroll
          for (int i = 0; i < TX; ++i) {
            const double tt = sx[i] + sy[j];
            if (!ballot(tt < c2)) continue;
            const float exy = ex[i] * ey[j];
#pragma unroll
            for (int k = 0; k < TZ; ++k) {
              const double u2 = tt + sz[k];
              const float e = exy * ez[k];
              Acc& a = acc[i + TX * (j + TY * k)];
              a = a + ((u2 < c2) ? e : 0.0f);
            }
          }
      }
    };

    // evaluate the queue's first 64
    auto drain64 = [&]() __attribute__((always_inline)) {
      const int at = (qh + lane) & (QCAP - 1);
      const float4 p = qp[at];
      float4 prm = make_float4(0.f, 0.f, 0.f, 0.f);
      if constexpr (PP == PP_ANISO) prm = qa[at];
      qn -= 64;
      qh += 64;
      wave_sync();
      eval_point(p, prm);
    };
    // fill up the queue's last 64 with far dummy particles
    auto pad64 = [&]() __attribute__((always_inline)) {
      const int r = qn & 63;
      if (r == 0) return;
      if (lane >= r) {
        const int at = (qh + qn - r + lane) & (QCAP - 1);
        qp[at] = make_float4(SFK_SENTINEL, SFK_SENTINEL, SFK_SENTINEL, 1.0f);
        if constexpr (PP == PP_ANISO) qa[at] = make_float4(1.f, 1.f, 1.f, 0.f);
      }
      qn += 64 - r;
      wave_sync();
    };

    // particle (and, anisotropic, its parameters) of lane `lane` of leaf lid
    auto fetch = [&](int lid, float4& p, float4& prm) {
      const int64_t slot = (int64_t)lid * SFK_LEAF + lane;
      p = tv.pts[slot];
      if constexpr (PP == PP_ANISO) prm = tv.pparam[slot];
    };
    // Can the particle's support reach the tile box? Float32 with a margin:
    // d is the distance from the box's centre (as a float), rounded once, the
    // half width is taken 2^-20 larger and the support 2^-20 wider, while all
    // roundings together stay below 2^-22. A particle that reaches a node is
    // always kept; one kept in vain adds zeros (up to 1e-16 at the edge).
    // 10 to 16 instructions; in double, with its conversions and maxima, the
    // test took about 30.
    auto keep_of = [&](const float4 p, const float4 prm) __attribute__((always_inline)) {
      const float dx = fabsf(p.x - bc[0]), dy = fabsf(p.y - bc[1]), dz = fabsf(p.z - bc[2]);
      float ux, uy, uz;
      if constexpr (PP == PP_UNIFORM) {
        // clamped to [0, 1] (an output modifier): 1 on any axis is out
        ux = fminf(fmaxf(fmaf(dx, us[0], -uh[0]), 0.0f), 1.0f);
        uy = fminf(fmaxf(fmaf(dy, us[1], -uh[1]), 0.0f), 1.0f);
        uz = fminf(fmaxf(fmaf(dz, us[2], -uh[2]), 0.0f), 1.0f);
      } else {  // not clamped after the product: infinite ih must give a NaN, out
        const float gx = fmaxf(dx - bh[0], 0.0f), gy = fmaxf(dy - bh[1], 0.0f),
                    gz = fmaxf(dz - bh[2], 0.0f);
        ux = gx * (PP == PP_ISO ? p.w : prm.x);
        uy = gy * (PP == PP_ISO ? p.w : prm.y);
        uz = gz * (PP == PP_ISO ? p.w : prm.z);
      }
      const float u2 = fmaf(ux, ux, fmaf(uy, uy, uz * uz));
      return u2 < (PP == PP_UNIFORM ? 1.0f : cc);
    };
    // append the kept particles of one leaf (lane order) to the queue; the
    // caller makes the writes visible (wave_sync) before the queue is read
    auto push = [&](const float4 p, const float4 prm, bool keep) {
      const uint64_t m = ballot(keep);
      if (keep) {
        const int pos = (qh + qn + popc64(m & lanemask_lt())) & (QCAP - 1);
        qp[pos] = p;
        if constexpr (PP == PP_ANISO) qa[pos] = prm;
      }
      qn += popc64(m);
    };
    auto node_out = [&](int node, double v) {
      const int i = node % TX, j = (node / TX) % TY, k = node / (TX * TY);
      const int gi = g.i0 + i, gj = g.j0 + j, gk = g.k0 + k;
      if (gi < R.res[0] && gj < R.res[1] && gk < R.res[2])
        R.out[(int64_t)gi + (int64_t)R.res[0] * ((int64_t)gj + (int64_t)R.res[1] * gk)] = (float)v;
    };
    auto lane_node = [&](int m) { return T >= 64 ? lane * NPL + m : (lane & (T - 1)); };
    const bool lane_writes = T >= 64 || lane < T;

    const int c = (int)(item - chunk_off[t]);
    const bool whole = mode_whole(mode);
    // A block's chunks are added in double, and the blocks; so an item's sums
    // combine to the same bits whether it is a chunk, a block or the tile.
    const int block_mask = (1 << fit_block(fit)) - 1;
    double dacc[NPL], bacc[NPL];  // the item's sums, its open block's
#pragma unroll
    for (int m = 0; m < NPL; ++m) dacc[m] = bacc[m] = 0.0;
    // the item's per-node sums: the grid values when it is all of the tile,
    // else a partial slot, the last item to finish combining all of them in
    // order
    auto finish_item = [&]() __attribute__((always_inline)) {
      if (whole || nit == 1) {
        if (lane_writes) {
#pragma unroll
          for (int m = 0; m < NPL; ++m) node_out(lane_node(m), dacc[m] * R.scale);
        }
      } else {
        const int64_t pbase = (partial_off[t] + c) * T;
        if (lane_writes) {
#pragma unroll
          for (int m = 0; m < NPL; ++m) hand_over(&partials[pbase + lane_node(m)], dacc[m]);
        }
        agent_writes_done();
        int prev = 0;
        if (lane == 0) prev = atomicAdd(&tile_done[t], 1);
        prev = __shfl(prev, 0, 64);
        if (prev == nit - 1) {
          agent_writes_done();
          if (lane_writes) {
            const int64_t p0 = partial_off[t] * T;
            const int ends = fit_coarse(fit) ? 0 : block_mask;
#pragma unroll
            for (int m = 0; m < NPL; ++m) {
              const int node = lane_node(m);
              double s = 0.0, b = 0.0;
              for (int q = 0; q < nit; ++q) {
                b += handed_over(&partials[p0 + (int64_t)q * T + node]);
                if (((q + 1) & ends) == 0 || q == nit - 1) {
                  s += b;
                  b = 0.0;
                }
              }
              node_out(node, s * R.scale);
            }
          }
        }
      }
    };
    // Where the ids of a tile's leaves come from: its list, or, when the list
    // did not fit, the hierarchy, walked in list order. The walk is a
    // generator, a step of which tests one node's up to 64 children and puts
    // the leaves among them into a ring; so both feed the same loop, and the
    // kernel holds one copy of the evaluation (three took more registers than
    // three wavefronts a SIMD leave).
    const bool listed = mode_listed(mode);
    const int64_t list0 = listed ? leaf_off[t] : 0;
    int32_t* ring = lds_walk[wave];
    int walked = 0, sp = 0, level = tv.n_levels - 1, first = 0, width = tv.level_cnt[level];
    auto walk_step = [&]() __attribute__((always_inline)) {
      const int child = first + lane;
      bool pass = false;
      // the tile's geometry is looked up again: kept, it would take registers
      // from the evaluation, which runs far more often
      int tt = t;
      asm volatile("" : "+s"(tt));
      const TileGeo gw = tile_geo<TX, TY, TZ>(rois, n_rois, coords, tt);
      if (lane < width) {
        const int gi = tv.level_off[level] + child;
        pass = tile_box_test(tv, rois[gw.r], gw, tv.nodes[gi], gi);
      }
      const uint64_t m = ballot(pass);
      const int np = popc64(m), r = popc64(m & lanemask_lt());
      const bool leaf = level == 0;
      if (pass) {
        if (leaf)
          ring[(walked + r) & (kWalkRing - 1)] = child;
        else
          lds_stack[wave][sp + np - 1 - r] = ((level - 1) << 27) | child;
      }
      walked += leaf ? np : 0;
      sp += leaf ? 0 : np;
      wave_sync();
      if (sp == 0) {
        walked = cnt;  // the end (all cnt leaves were met)
        return;
      }
      const int e = wave_uniform(lds_stack[wave][--sp]);
      level = e >> 27;
      first = (e & ((1 << 27) - 1)) * SFK_FANOUT;
      width = min(SFK_FANOUT, tv.level_cnt[level] - first);
    };
    // The work item's leaves, a chunk at a time.
    const int i0 = whole ? 0 : c * span, i1 = whole ? cnt : min(i0 + span, cnt);
    int left = block_mask;  // chunks to the block's end
    for (int lb = i0; lb < i1; lb += chunk, left = (left - 1) & block_mask) {
      const int le = min(lb + chunk, cnt);
#pragma unroll
      for (int q = 0; q < T; ++q) acc[q] = (Acc)0;
      // Ids of leaves [i, i + 64) of the tile, one a lane; past the chunk's
      // end its last leaf stands, culled as empty. A list entry that is not a
      // leaf of the tree is an internal error: flag it and read leaf 0
      // instead (never out of bounds).
      auto load_ids = [&](int i) __attribute__((always_inline)) {
        const int at = min(i + lane, le - 1);
        if (!listed) {
          while (walked < min(i + 64, le)) walk_step();
          return ring[at & (kWalkRing - 1)];
        }
        const int v = leaves[list0 + at];
        const bool bad = (unsigned)v >= (unsigned)tv.n_leaves;
        if (bad) claims[kErrWord] = 1;
        return bad ? 0 : v;
      };
      // Software pipeline over NB particle buffers: a buffer is refilled
      // with the leaf NB places ahead as soon as it has been culled, so
      // NB - 1 leaves are in flight during each cull; the loop is unrolled
      // over the buffers so that no register is copied while its load is
      // pending. The next 64 ids are loaded while 64 are worked on, so
      // reading an id never waits.
      float4 pb[NB], ab[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) pb[u] = ab[u] = make_float4(0.f, 0.f, 0.f, 0.f);
      int next = 0;
      for (int b0 = lb - 64; b0 < le; b0 += 64) {
        const int ids = next;
        next = load_ids(b0 + 64);
        if (b0 < lb) {  // nothing held yet: start the pipeline
#pragma unroll
          for (int u = 0; u < NB; ++u) {
            fetch(__builtin_amdgcn_readlane(next, u), pb[u], ab[u]);
            // keep buffer order = issue order (the oldest load is consumed first)
            __builtin_amdgcn_sched_barrier(0);
          }
          continue;
        }
        const int m = min(64, le - b0);
        for (int i = 0; i < m; i += NB) {
          // the last round's refills are the next 64's first
          const int src = i + NB < 64 ? ids : next;
          const int at = (i + NB) & 63;
#pragma unroll
          for (int u = 0; u < NB; u += 2) {
            // appends only need to be visible to the drain: one visibility
            // point for two leaves lets the compiler overlap their culls
#pragma unroll
            for (int w = u; w < u + 2; ++w) {
              push(pb[w], ab[w], i + w < m && keep_of(pb[w], ab[w]));
              fetch(__builtin_amdgcn_readlane(src, at + w), pb[w], ab[w]);
            }
            wave_sync();
            if (u + 2 == NB && b0 + i + NB >= le) pad64();  // the chunk's end
            while (qn >= 64) drain64();
          }
        }
      }
      reduce_nodes(acc);
#pragma unroll
      for (int m = 0; m < NPL; ++m) {
        bacc[m] += (double)acc[m];
        if (left == 0 || le == i1) {
          dacc[m] += bacc[m];
          bacc[m] = 0.0;
        }
      }
    }
    finish_item();
  }
}

// ---------------------------------------------------------------------------
// Brick evaluation by scattering (uniform bandwidths). A workgroup owns a
// brick of kBrick^3 nodes and keeps one 64-bit integer sum per node in LDS.
// Each lane takes one particle of a candidate leaf, computes on each axis the
// range of brick nodes whose distance can be inside the support (rounded
// outwards by a relative 1e-9, so the range never misses a member), and
// visits those nodes only. An Epanechnikov term is ((1 - ux^2) - uy^2) - uz^2,
// its parts in double and counted in fixed point (epan_sq_units), added with
// an LDS atomic; the support counts and the truncated Gaussian decide
// membership by the canonical u2 = (ux^2 + uy^2) + uz^2 < c2 as the
// definition does (the Gaussian's term is exp(-u2/2) in float). The
// per-particle cost follows the support (about (2h/s)^3 nodes, twice the
// members) instead of a whole tile, and integer sums are exact, so the grid
// is the same whatever the order of particles, chunks or workgroups (alone,
// in any batch, in any evaluation mode). The brick's chunks add their sums
// into one 64-bit slot per node with global atomics; the last chunk to
// finish writes the nodes: sum * unit * scale, rounded once to float. Per
// term the fixed point adds at most 0.75 * 2^-31 (2^-32 for the Gaussian, in
// units of the kernel's peak) to a node sum.
// ---------------------------------------------------------------------------

// Fixed-point units of a truncated Gaussian's term e in [0, 1], rounded to the
// nearest: the scaling is exact, and a float of 2^23 units or more is whole
// (through double, two conversions more a term, 10M points at 128^3 in a
// 3-node sweep took 184 us for 173).
__device__ __forceinline__ unsigned int gauss_units(float e) {
  return (unsigned int)rintf(e * (float)kSplatUnit);
}

// The Epanechnikov term ((1 - ux^2) - uy^2) - uz^2 in fixed point, 2^32 - 1
// units to 1, from the units of its three parts, each rounded to the nearest
// and saturated at 1: a term is 1 - ux^2's less uy^2's less uz^2's, 0 when
// that is not positive (saturating subtractions; a pair outside the support
// counts 0 up to a unit and a half at its edge). A part belongs to a node
// coordinate, so a row of nodes takes one integer subtraction. The clamps are
// output modifiers.
constexpr double kEpanUnit = 4294967295.0;
__device__ __forceinline__ double clamp01(double v) { return fmin(fmax(v, 0.0), 1.0); }
__device__ __forceinline__ unsigned int epan_sq_units(double sq) {
  return (unsigned int)fma(clamp01(sq), kEpanUnit, 0.5);
}
__device__ __forceinline__ unsigned int epan_x_units(double sx) {
  return (unsigned int)fma(clamp01(1.0 - sx), kEpanUnit, 0.5);
}
// units of a node sum
template <int KK, bool CNT>
constexpr double kSumUnit = CNT ? 1.0 : KK == KK_EPAN ? 1.0 / kEpanUnit : 1.0 / kSplatUnit;
__device__ __forceinline__ unsigned int epan_units(unsigned int row, unsigned int z) {
  return row > z ? row - z : 0u;
}

// One wave claims the next work item (XCD-aware slices as in k_eval); -1
// when every slice is exhausted. `cur` carries the wave's current slice.
__device__ __forceinline__ int64_t claim_item(int32_t* __restrict__ claims, int64_t n_items,
                                              int xcd, int sub, int& cur) {
  const int lane = lane_id();
  auto slice_at = [&](int pos) { return ((xcd + (pos >> 3)) & 7) * 8 + ((sub + pos) & 7); };
  auto slice_begin = [&](int sl) { return n_items * sl / kClaimSlices; };
  while (true) {
    const int64_t b = slice_begin(cur), e = slice_begin(cur + 1);
    int idx = 0;
    if (b < e && lane == 0) idx = atomicAdd(&claims[cur * kClaimStride], 1);
    idx = __shfl(idx, 0, 64);
    if (b + idx < e) return b + idx;
    const int my = slice_at(lane);
    const int64_t mb = slice_begin(my), me = slice_begin(my + 1);
    const int seen =
        __hip_atomic_load(&claims[my * kClaimStride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    const uint64_t open = __ballot(mb + seen < me);
    if (open == 0) return -1;
    cur = slice_at(__ffsll((unsigned long long)open) - 1);
  }
}

// -log2(e)/2 (exp(-u2/2) = exp2(KG * u2)), as in k_eval
#define SFK_KG64S (-0.72134752044448170368)

template <int KK, bool CNT>
__global__ __launch_bounds__(256) void k_splat(
    TreeView tv, const RoiDev* __restrict__ rois, const double* __restrict__ coords,
    const BatchHdr* __restrict__ hdr, int32_t* __restrict__ claims,
    const int64_t* __restrict__ leaf_off, const int64_t* __restrict__ chunk_off,
    const int64_t* __restrict__ partial_off, const int32_t* __restrict__ tile_cnt,
    const int32_t* __restrict__ tile_fit, const int32_t* __restrict__ leaves,
    const int32_t* __restrict__ item_tile, double* __restrict__ partials,
    int32_t* __restrict__ tile_done) {
  constexpr int B = kBrick;
  constexpr int T = B * B * B;
  __shared__ unsigned long long sums[T];
  __shared__ double lds_c[3][B];
  __shared__ int32_t lds_stack[4][SFK_STACK];
  __shared__ int64_t lds_item;
  __shared__ int32_t lds_last;
  unsigned long long* gsum = (unsigned long long*)partials;
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const int64_t n_items = min(hdr->n_items, hdr->item_cap);
  const int n_rois = hdr->n_rois;
  const int xcd = blockIdx.x & 7;
  const int sub = (int)((blockIdx.x >> 3) & 7);
  int cur = ((xcd + 0) & 7) * 8 + (sub & 7);
  while (true) {
    if (wave == 0) {
      const int64_t it = claim_item(claims, n_items, xcd, sub, cur);
      if (lane == 0) lds_item = it;
    }
    __syncthreads();
    const int64_t item = lds_item;
    if (item < 0) break;
    const int t = wave_uniform(item_tile[item]);
    const TileGeo g = tile_geo<B, B, B>(rois, n_rois, coords, t);
    const RoiDev& R = rois[g.r];
    const int n_here[3] = {min(B, R.res[0] - g.i0), min(B, R.res[1] - g.j0),
                           min(B, R.res[2] - g.k0)};
    if (threadIdx.x < 3 * B) {
      const int k = threadIdx.x / B, i = threadIdx.x % B;
      const int o = k == 0 ? g.i0 : k == 1 ? g.j0 : g.k0;
      const int off = R.coord_off + (k > 0 ? R.res[0] : 0) + (k > 1 ? R.res[1] : 0);
      lds_c[k][i] = coords[off + min(o + i, R.res[k] - 1)];
    }
    for (int i = threadIdx.x; i < T; i += 256) sums[i] = 0ull;
    __syncthreads();
    const double c2 = R.c2;
    const double lo[3] = {R.lo[0], R.lo[1], R.lo[2]};
    double inv_s[3], half[3];
    const int org[3] = {g.i0, g.j0, g.k0};
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      inv_s[k] = (double)(R.res[k] - 1) / (R.hi[k] - R.lo[k]);
      // support half-width in node steps, rounded outwards
      half[k] = sqrt(c2) * inv_s[k] / (double)R.ih[k];
      half[k] = half[k] * (1.0 + 1e-9) + 1e-9;
    }
    const double ih[3] = {(double)R.ih[0], (double)R.ih[1], (double)R.ih[2]};

    // Supports that span at most kSpan nodes in x keep the x nodes' parts in
    // registers: a row then takes a subtraction, a test and an add per node,
    // where each node of the general loop reads and converts its coordinate
    // again. 4096 bricks of a 256^3 zoom into 100M points, 6 nodes an axis:
    // whole call 171 us, 298 without (with the y nodes kept as well 200 for the
    // 199 it had then, at three wavefronts a SIMD, at which batches lost 1%).
    // Registers for n nodes are worked through by supports of fewer nodes too:
    // 8M uniform points at 200^3 take, with 1 to 8 nodes an axis, 286 417 737
    // 1359 2452 4023 6280 9193 us in the general loop, 304 420 609 891 1313
    // 1897 6285 9181 with 6 kept, 298 386 548 1368 2467 4036 with 3 and 308 446
    // 670 1007 1508 2142 2926 3990 with 8. By default a brick's supports have 4
    // nodes at most, but for regions of under 1/8 particle a node.
    constexpr int kSpan = 6;
    const bool short_span = floor(2.0 * half[0]) + 1.0 <= (double)kSpan;

    // scatter one particle (lane's own) into the brick's node sums
    auto splat = [&](const float4 p) {
      const double pp[3] = {(double)p.x, (double)p.y, (double)p.z};
      int a[3], b[3];
      bool empty = false;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double ic = (pp[k] - lo[k]) * inv_s[k] - (double)org[k];
        const double fa = fmax(ceil(ic - half[k]), 0.0);
        const double fb = fmin(floor(ic + half[k]), (double)(n_here[k] - 1));
        empty |= !(fa <= fb);
        a[k] = empty ? 0 : (int)fa;
        b[k] = empty ? -1 : (int)fb;
      }
      if (empty) return;
      if constexpr (KK == KK_EPAN && !CNT) {
        if (short_span) {
          // (past the range 0 units: no term)
          unsigned int xq[kSpan], xmax = 0u;
#pragma unroll
          for (int m = 0; m < kSpan; ++m) {
            const double ux = (lds_c[0][min(a[0] + m, B - 1)] - pp[0]) * ih[0];
            xq[m] = a[0] + m <= b[0] ? epan_x_units(ux * ux) : 0u;
            xmax = max(xmax, xq[m]);
          }
          const int ny = b[1] - a[1] + 1, nz = b[2] - a[2] + 1;
          const int ry = (lane >> 2) % ny, rz = (lane >> 4) % nz;
          for (int dz = 0; dz < nz; ++dz) {
            int kz = a[2] + dz + rz;
            kz = kz > b[2] ? kz - nz : kz;
            const double uz = (lds_c[2][kz] - pp[2]) * ih[2];
            const unsigned int zq = epan_sq_units(uz * uz);
            for (int dy = 0; dy < ny; ++dy) {
              int jy = a[1] + dy + ry;
              jy = jy > b[1] ? jy - ny : jy;
              const double uy = (lds_c[1][jy] - pp[1]) * ih[1];
              const unsigned int yq = epan_sq_units(uy * uy);
              if (epan_units(xmax, yq) <= zq) continue;
              // byte offsets of the row and of its first node's swizzled slot,
              // made here: the compiler made them again in each node's branch
              // of one of the copies of this code, whose share of a 256^3 zoom
              // was 142 us for 129
              int row = 8 * B * (jy + B * kz), at = 8 * (a[0] + 3 * jy + 5 * kz);
              asm volatile("" : "+v"(row), "+v"(at));
#pragma unroll
              for (int m = 0; m < kSpan; ++m) {
                const unsigned int q = epan_units(epan_units(xq[m], yq), zq);
                if (q != 0u)
                  atomicAdd((unsigned long long*)((char*)sums + (row + ((at + 8 * m) & (8 * (B - 1))))),
                            (unsigned long long)q);
              }
            }
          }
          return;
        }
      }
      // Lanes of a leaf often share their range: each lane starts its walk
      // over the range at its own rotation (lane mod the range size per
      // axis), so the atomics of one instruction spread over the range's
      // nodes instead of queueing on one.
      const int nx = b[0] - a[0] + 1, ny = b[1] - a[1] + 1, nz = b[2] - a[2] + 1;
      const int rx = lane % nx, ry = (lane >> 2) % ny, rz = (lane >> 4) % nz;
      for (int dz = 0; dz < nz; ++dz) {
        int kz = a[2] + dz + rz;
        kz = kz > b[2] ? kz - nz : kz;
        const double uz = (lds_c[2][kz] - pp[2]) * ih[2];
        const double sz = uz * uz;
        const unsigned int zq = epan_sq_units(sz);
        for (int dy = 0; dy < ny; ++dy) {
          int jy = a[1] + dy + ry;
          jy = jy > b[1] ? jy - ny : jy;
          const double uy = (lds_c[1][jy] - pp[1]) * ih[1];
          const double sy = uy * uy;
          const unsigned int yq = epan_sq_units(sy);
          const int row = B * (jy + B * kz);
          const int sw = (3 * jy + 5 * kz) & (B - 1);  // bank swizzle of the row
          for (int dx = 0; dx < nx; ++dx) {
            int ix = a[0] + dx + rx;
            ix = ix > b[0] ? ix - nx : ix;
            const double ux = (lds_c[0][ix] - pp[0]) * ih[0];
            if constexpr (KK == KK_EPAN && !CNT) {
              const unsigned int q = epan_units(epan_units(epan_x_units(ux * ux), yq), zq);
              if (q != 0u) atomicAdd(&sums[row + ((ix + sw) & (B - 1))], (unsigned long long)q);
            } else {
              const double u2 = (ux * ux + sy) + sz;
              if (u2 < c2) {
                unsigned int q;
                if constexpr (CNT) {
                  q = 1u;
                } else {
                  const float e = __builtin_amdgcn_exp2f((float)(SFK_KG64S * u2));
                  q = gauss_units(e);
                }
                atomicAdd(&sums[row + ((ix + sw) & (B - 1))], (unsigned long long)q);
              }
            }
          }
        }
      }
    };
    // Listed leaves: a leaf's particles that reach the brick (the same
    // outward-rounded ranges as splat) are queued and scattered 64 at a time,
    // so every lane has a particle. In the leaves of sparse and deep ROIs
    // most particles reach no node of the brick, and a lane per leaf
    // particle left most lanes idle. The order of the integer adds does not
    // change the sums. The queue (particle indices, at most 127) lives in the
    // wave's traversal stack, which listed leaves do not use.
    uint32_t* qi = reinterpret_cast<uint32_t*>(lds_stack[wave]);
    static_assert(SFK_STACK >= 2 * SFK_LEAF, "the queue shares the traversal stack");
    int qn = 0;
    auto reaches = [&](const float4 p) {
      const double pp[3] = {(double)p.x, (double)p.y, (double)p.z};
      bool ok = true;
#pragma unroll
      for (int k = 0; k < 3; ++k) {
        const double ic = (pp[k] - lo[k]) * inv_s[k] - (double)org[k];
        ok &= fmax(ceil(ic - half[k]), 0.0) <= fmin(floor(ic + half[k]), (double)(n_here[k] - 1));
      }
      return ok;
    };
    auto offer = [&](const float4 p, int64_t idx) {
      const bool ok = reaches(p);
      const uint64_t m = ballot(ok);
      if (ok) qi[qn + popc64(m & lanemask_lt())] = (uint32_t)idx;
      qn += popc64(m);
      wave_sync();
      if (qn >= 64) {
        const uint32_t mine = qi[lane];
        for (int e = lane; e + 64 < qn; e += 64) qi[e] = qi[e + 64];
        qn -= 64;
        wave_sync();
        splat(tv.pts[mine]);
      }
    };
    auto drain_rest = [&]() {
      if (qn == 0) return;
      const bool have = lane < qn;
      const uint32_t mine = have ? qi[lane] : 0u;
      qn = 0;
      wave_sync();
      if (have) splat(tv.pts[mine]);
    };
    auto do_leaf = [&](int lid) {
      const float4 p = tv.pts[(int64_t)lid * SFK_LEAF + lane];
      splat(p);
    };

    const int cnt = tile_cnt[t];
    const int fit = tile_fit[t], mode = fit_mode(fit), span = fit_span(fit);
    const int nit = (cnt + span - 1) / span;
    const bool whole = mode_whole(mode);
    const int c = (int)(item - chunk_off[t]);
    if (mode_listed(mode)) {
      // the item's leaves, every fourth to each wave; ids outside the tree
      // are an internal error (flagged, leaf 0 read instead)
      const int64_t lb = leaf_off[t] + (whole ? 0 : (int64_t)c * span);
      const int64_t le = whole ? lb + cnt : min(lb + span, leaf_off[t] + cnt);
      auto leaf_at = [&](int64_t q) {
        int lid = leaves[q];
        if ((unsigned)lid >= (unsigned)tv.n_leaves) {
          if (lane == 0) claims[kErrWord] = 1;
          lid = 0;
        }
        return __builtin_amdgcn_readfirstlane(lid);
      };
      // the next leaf's particle is in flight while this one is offered
      if (lb + wave < le) {
        int64_t idx = (int64_t)leaf_at(lb + wave) * SFK_LEAF + lane;
        float4 p = tv.pts[idx];
        for (int64_t q = lb + wave; q < le; q += 4) {
          float4 pn = p;
          int64_t nidx = idx;
          if (q + 4 < le) {
            nidx = (int64_t)leaf_at(q + 4) * SFK_LEAF + lane;
            pn = tv.pts[nidx];
          }
          offer(p, idx);
          p = pn;
          idx = nidx;
        }
      }
      drain_rest();
    } else {
      // the whole tile without a list: every wave walks the hierarchy (same
      // order) and takes every fourth leaf
      int done = 0;
      traverse(
          tv, lds_stack[wave],
          [&](const NodeBox& b, int gidx) { return tile_box_test(tv, R, g, b, gidx); },
          [&](int child, bool pass, uint64_t mask) {
            (void)pass;
            uint64_t mm = mask;
            while (mm) {
              const int bl = __ffsll((unsigned long long)mm) - 1;
              mm &= mm - 1;
              if ((done & 3) == wave) do_leaf(__shfl(child, bl, 64));
              ++done;
            }
          });
    }
    __syncthreads();
    const double unit = kSumUnit<KK, CNT>;
    // LDS slot n holds node (ix, jy, kz) with n = B (jy + B kz) + ((ix + sw) mod B)
    auto write_node = [&](int n, unsigned long long v) {
      const int jy = (n / B) % B, kz = n / (B * B);
      const int ix = ((n % B) - ((3 * jy + 5 * kz) & (B - 1))) & (B - 1);
      if (ix < n_here[0] && jy < n_here[1] && kz < n_here[2]) {
        const int64_t gi = g.i0 + ix, gj = g.j0 + jy, gk = g.k0 + kz;
        R.out[gi + (int64_t)R.res[0] * (gj + (int64_t)R.res[1] * gk)] =
            (float)(((double)v * unit) * R.scale);
      }
    };
    if (whole || nit == 1) {
      for (int n = threadIdx.x; n < T; n += 256) write_node(n, sums[n]);
    } else {
      unsigned long long* slot = gsum + partial_off[t] * (int64_t)T;
      for (int n = threadIdx.x; n < T; n += 256)
        if (sums[n]) atomicAdd(&slot[n], sums[n]);
      agent_writes_done();
      __syncthreads();
      if (threadIdx.x == 0) lds_last = atomicAdd(&tile_done[t], 1) == nit - 1 ? 1 : 0;
      __syncthreads();
      if (lds_last) {
        agent_writes_done();
        for (int n = threadIdx.x; n < T; n += 256)
          write_node(n, handed_over(&slot[n]));
      }
    }
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------
// Particle sweep (uniform bandwidths, dense ROIs). Where a ROI holds many
// particles per node, a tile re-reads each particle in every tile whose
// support-widened box holds it (about (t + 2h/s)^3 / t^3 tiles for a tile
// of t^3 nodes) and tests it against all the tile's nodes, and each tile
// pays a range query. The sweep reads every particle of the ROI's support
// once. A work item is a (ROI, box) pair, the box taken from the
// hierarchy's first interior level (64 leaves, 4096 particles, compact in
// curve order); the workgroup scatters the box's particles into an LDS
// window of the ROI's nodes that the box's support can reach, with the
// brick's terms and fixed point (the same operations in the same order)
// and LDS atomics into private copies of the window (lane l adds to copy
// l mod ncp), then adds the window's nonzero sums into the batch's 64-bit
// node sums with global atomics. The Epanechnikov term takes two saturating
// subtractions of fixed-point units, one per node row (those of 1 - ux^2 less
// those of uy^2) and one per node (less those of uz^2), with no membership
// branch. Bound by VALU issue and the LDS atomics together (3-node spans: both
// three quarters busy; their share of 256 zooms into 100M points takes 5.2
// ms, 5.9 when each row converted 1 - (ux^2 + uy^2) and rows without a term
// were added).
// Integer sums make the grid independent of the order of items, particles
// and workgroups, and equal to the brick's grid bit for bit. For spans of 3
// nodes or more the lanes of a wavefront take particles of different leaves
// of the box, so one instruction's atomics spread over the window instead
// of queueing on the few nodes one leaf reaches; spans of 1 and 2 nodes add
// few terms and take one leaf per wavefront, for coalesced loads. Windows
// wider than W nodes on some axis (W = kSweepWin, half that for 1-node
// spans) are swept in blocks of W^3 nodes, each reading the box again.
// ---------------------------------------------------------------------------

// A squared offset past any support (c^2 <= 9): the sweep gives the nodes
// past a particle's z range this value, so their terms are 0.
constexpr double kSweepFar = 1e300;

// Level of the hierarchy whose boxes are the sweep's work items: the first
// interior level (64 leaves a box) when the tree has one, else the leaves.
__device__ __forceinline__ int sweep_level(const TreeView& tv) { return tv.n_levels >= 2 ? 1 : 0; }

// Support half-width of a ROI in node steps on axis k, rounded outwards so
// that a particle's node range never misses a member (as the brick's).
__device__ __forceinline__ double sweep_half(const RoiDev& R, int k, double* inv_s) {
  *inv_s = (double)(R.res[k] - 1) / (R.hi[k] - R.lo[k]);
  const double h = sqrt((double)R.c2) * *inv_s / (double)R.ih[k];
  return h * (1.0 + 1e-9) + 1e-9;
}

// Block 0 zeroes the claim counters (never the error word), every block a
// stride of the node sums of the header's tiles.
__global__ __launch_bounds__(256) void k_sweep_zero(const BatchHdr* __restrict__ hdr,
                                                    unsigned long long* __restrict__ acc,
                                                    int32_t* __restrict__ claims) {
  if (blockIdx.x == 0)
    for (int i = threadIdx.x; i < kClaimSlices * kClaimStride; i += blockDim.x) claims[i] = 0;
  constexpr int T = kSweep * kSweep * kSweep;
  const int64_t n = hdr->n_tiles * T;
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n;
       i += (int64_t)gridDim.x * blockDim.x)
    acc[i] = 0ull;
}

// One wavefront per (ROI, group of 64 item boxes): the group's parent box
// first (when the level above exists), then one box per lane, with the
// tiles' box test against the box of all the ROI's nodes; passing boxes are
// appended as (ROI << 32 | box).
__global__ __launch_bounds__(256) void k_sweep_list(TreeView tv, BatchHdr* __restrict__ hdr,
                                                    const RoiDev* __restrict__ rois,
                                                    const double* __restrict__ coords,
                                                    int64_t* __restrict__ items,
                                                    int32_t* __restrict__ claims) {
  const int lane = lane_id();
  const int L = sweep_level(tv);
  const int nb = tv.level_cnt[L];
  const int ng = (nb + 63) >> 6;
  const int64_t w = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (ng == 0 || w >= (int64_t)hdr->n_rois * ng) return;
  const int r = (int)(w / ng), grp = (int)(w % ng);
  const RoiDev& R = rois[r];
  TileGeo g;
  g.r = r;
  g.i0 = g.j0 = g.k0 = 0;
  {
    const double* cx = coords + R.coord_off;
    const double* cy = cx + R.res[0];
    const double* cz = cy + R.res[1];
    g.lo[0] = cx[0];
    g.hi[0] = cx[R.res[0] - 1];
    g.lo[1] = cy[0];
    g.hi[1] = cy[R.res[1] - 1];
    g.lo[2] = cz[0];
    g.hi[2] = cz[R.res[2] - 1];
  }
  if (L + 1 < tv.n_levels) {
    const int gp = tv.level_off[L + 1] + grp;
    if (!tile_box_test(tv, R, g, tv.nodes[gp], gp)) return;
  }
  const int b = grp * 64 + lane;
  bool pass = false;
  if (b < nb) {
    const int gi = tv.level_off[L] + b;
    pass = tv.nodes[gi].count > 0 && tile_box_test(tv, R, g, tv.nodes[gi], gi);
  }
  const uint64_t m = ballot(pass);
  if (m == 0) return;
  unsigned long long base = 0;
  if (lane == 0) base = atomicAdd((unsigned long long*)&hdr->n_items, (unsigned long long)popc64(m));
  base = __shfl(base, 0, 64);
  const int64_t pos = (int64_t)base + popc64(m & lanemask_lt());
  if (pass) {
    if (pos < hdr->item_cap)
      items[pos] = ((int64_t)r << 32) | (int64_t)(uint32_t)b;
    else
      claims[kErrWord] = 1;
  }
}

// (1-node spans ask for 6 waves per SIMD, their register bound without
// spills; more waves spilled and were slower)
template <int KK, bool CNT, int NM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(NM == 1 ? 6 : 1)))
void k_sweep(TreeView tv, const BatchHdr* __restrict__ hdr, const RoiDev* __restrict__ rois,
             const int64_t* __restrict__ items, unsigned long long* __restrict__ acc,
             int32_t* __restrict__ claims) {
  // Windows of 1-node spans are blocked at 8^3 nodes: their boxes' windows
  // seldom exceed that, and the smaller LDS array lets 6 blocks share a CU
  // (the register bound) to hide more of the memory latency these light
  // particles wait on (2-node spans lost more to re-read blocks than they
  // gained).
  constexpr int W = NM == 1 ? kSweepWin / 2 : kSweepWin;
  constexpr int S = kSweep;
  // rows tested by their Epanechnikov units (the other modes' ranges, with
  // their ends, leave fewer pairs to decide one by one)
  constexpr bool kRowTest = NM > 1 && KK == KK_EPAN && !CNT;
  // the window's node sums, z fastest, with an odd x stride (W^2 + 1 at
  // most) so that threads reading consecutive x fall in different banks
  constexpr int WN = W * (W * W + 1);
  // (the Epanechnikov adds of spans up to 3 nodes are unmasked: a
  // particle's nodes past its z range add 0 up to kSweepMaxNM - 1 words past
  // a copy, hence the padding, which is never read)
  __shared__ unsigned long long sums[WN + kSweepMaxNM];
  // node coordinates of a block, with kSweepMaxNM more past its end so the
  // unrolled per-particle loops read them without clamping
  constexpr int WC = W + kSweepMaxNM;
  __shared__ double lds_c[3][WC];
  __shared__ int64_t lds_item;
  __shared__ int32_t lds_surv[SFK_FANOUT];
  __shared__ int32_t lds_nsurv;
  const int lane = lane_id();
  const int tid = threadIdx.x;
  const int64_t n_items = min((int64_t)hdr->n_items, hdr->item_cap);
  const int L = sweep_level(tv);
  const int xcd = blockIdx.x & 7;
  const int sub = (int)((blockIdx.x >> 3) & 7);
  int cur = ((xcd + 0) & 7) * 8 + (sub & 7);
  bool bad = false;
  while (true) {
    if (tid < 64) {
      const int64_t it = claim_item(claims, n_items, xcd, sub, cur);
      if (lane == 0) lds_item = it;
    }
    __syncthreads();
    const int64_t pos = lds_item;
    __syncthreads();  // lds_item is rewritten by the next claim
    if (pos < 0) break;
    const int64_t item = items[pos];
    const int r = (int)(item >> 32);
    const int b = (int)(item & 0xffffffff);
    // an item outside the batch or the tree is an internal error (flagged,
    // skipped: nothing is read out of bounds)
    if ((unsigned)r >= (unsigned)hdr->n_rois || (unsigned)b >= (unsigned)tv.level_cnt[L]) {
      bad = true;
      continue;
    }
    const RoiDev& R = rois[r];
    const NodeBox box = tv.nodes[tv.level_off[L] + b];
    const int l0 = L == 1 ? b * SFK_FANOUT : b;
    const int nl = L == 1 ? min(SFK_FANOUT, tv.n_leaves - l0) : 1;
    double inv_s[3], half[3], lo[3], ih[3];
    int w0[3], w1[3];
    bool empty = false;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      half[k] = sweep_half(R, k, &inv_s[k]);
      lo[k] = R.lo[k];
      ih[k] = (double)R.ih[k];
      const double fa = fmax(ceil(((double)box.lo[k] - lo[k]) * inv_s[k] - half[k]), 0.0);
      const double fb =
          fmin(floor(((double)box.hi[k] - lo[k]) * inv_s[k] + half[k]), (double)(R.res[k] - 1));
      empty |= !(fa <= fb);
      w0[k] = empty ? 0 : (int)fa;
      w1[k] = empty ? -1 : (int)fb;
      // a support wider than the NM nodes a particle visits: internal error
      if (!(floor(2.0 * half[k]) + 1.0 <= (double)NM)) bad = empty = true;
    }
    if (empty) continue;
    const double c2 = (double)R.c2;
    const float4* pts = tv.pts + (int64_t)l0 * SFK_LEAF;
    for (int bz = w0[2]; bz <= w1[2]; bz += W)
      for (int by = w0[1]; by <= w1[1]; by += W)
        for (int bx = w0[0]; bx <= w1[0]; bx += W) {
          const int blk0[3] = {bx, by, bz};
          const int nbk[3] = {min(W, w1[0] - bx + 1), min(W, w1[1] - by + 1),
                              min(W, w1[2] - bz + 1)};
          const int nyz = (nbk[1] * nbk[2]) | 1, nw = nbk[0] * nyz;
          // ncp private copies of the window's sums (odd stride, so the
          // copies of one node fall in different banks): lane l adds to copy
          // l mod ncp, so lanes whose particles reach the same node seldom
          // add to the same word
          int ncp = 16;
          while (ncp > 1 && ncp * (nw | 1) > WN) ncp >>= 1;
          const int cs = ncp > 1 ? (nw | 1) : nw;
          const int my_copy = (lane % ncp) * cs;
          if (tid < 3 * WC) {
            const int k = tid / WC, i = tid % WC;
            lds_c[k][i] = node_coord(R, k, blk0[k] + i);
          }
          for (int i = tid; i < ncp * cs; i += 256) sums[i] = 0ull;
          // the box's leaves whose box can reach the block (a particle's node
          // range lies inside its leaf's, so the others add nothing here)
          if (tid < 64) {
            bool reach = false;
            if (lane < nl) {
              const NodeBox lb = tv.nodes[tv.level_off[0] + l0 + lane];
              reach = lb.count > 0;
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                const double fa = fmax(ceil(((double)lb.lo[k] - lo[k]) * inv_s[k] - half[k]),
                                       (double)blk0[k]);
                const double fb = fmin(floor(((double)lb.hi[k] - lo[k]) * inv_s[k] + half[k]),
                                       (double)(blk0[k] + nbk[k] - 1));
                reach &= fa <= fb;
              }
            }
            const uint64_t m = ballot(reach);
            if (reach) lds_surv[popc64(m & lanemask_lt())] = lane;
            if (lane == 0) lds_nsurv = popc64(m);
          }
          __syncthreads();
          const int ns = lds_nsurv;
          auto splat = [&](const float4 p) {
            const double pp[3] = {(double)p.x, (double)p.y, (double)p.z};
            int a[3], n[3];
            bool ok = true;
            if constexpr (NM == 1) {
              // a support under half a spacing reaches at most the nearest
              // node: per axis the node rint(ic), if within the half-width
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                const double ic = (pp[k] - lo[k]) * inv_s[k];
                const double r = rint(ic);
                ok &= fabs(ic - r) <= half[k] && r >= (double)blk0[k] &&
                      r <= (double)(blk0[k] + nbk[k] - 1);
                a[k] = ok ? (int)r - blk0[k] : 0;
                n[k] = 1;
              }
              if (!ok) return;
            } else if constexpr (kRowTest && NM <= 3) {
              // The first node of the range on each axis, one exit, and the
              // nodes from there to the block's end. The range's own end
              // needs no test: past it a square is at least 1 and the terms
              // are 0 (15 instructions of 250; 3-node supports 5.45 -> 5.20 ms
              // of a batch of 256 zooms).
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                const double ic = (pp[k] - lo[k]) * inv_s[k];
                const double f = fmax(ceil(ic - half[k]), (double)blk0[k]);
                ok &= f <= (double)(blk0[k] + nbk[k] - 1);
                a[k] = (int)f - blk0[k];
                n[k] = nbk[k] - a[k];
              }
              if (!ok) return;
            } else {
              // the ranges of all three axes first, one exit, then the
              // conversions (no lane mask per axis): wider supports are swept
              // in more blocks, and a particle that only lies before a block
              // would visit NM^2 rows for nothing (6 nodes: 5.49 ms, 5.97
              // without the ranges' ends)
              double fa[3], fb[3];
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                const double ic = (pp[k] - lo[k]) * inv_s[k];
                fa[k] = fmax(ceil(ic - half[k]), (double)blk0[k]);
                fb[k] = fmin(floor(ic + half[k]), (double)(blk0[k] + nbk[k] - 1));
                ok &= fa[k] <= fb[k];
              }
              if (!ok) return;
#pragma unroll
              for (int k = 0; k < 3; ++k) {
                a[k] = (int)fa[k] - blk0[k];
                n[k] = (int)(fb[k] - fa[k]) + 1;
              }
            }
            // the particle's first node in this lane's copy of the window
            // (stored z fastest, x stride nyz); a node (mx, my, mz) past it
            // is base + mz + nbk2 my + nyz mx, so a row's adds differ only
            // in the immediate offset
            const int base = my_copy + a[2] + nbk[2] * a[1] + nyz * a[0];
            double sx[NM], sy[NM], sz[NM];
#pragma unroll
            for (int m = 0; m < NM; ++m) {
              const double ux = (lds_c[0][a[0] + m] - pp[0]) * ih[0];
              const double uy = (lds_c[1][a[1] + m] - pp[1]) * ih[1];
              const double uz = (lds_c[2][a[2] + m] - pp[2]) * ih[2];
              // past the range a huge square makes every term 0 (no add), so
              // the inner loop needs no range test, nor a row its own
              sx[m] = !kRowTest || m < n[0] ? ux * ux : kSweepFar;
              sy[m] = !kRowTest || m < n[1] ? uy * uy : kSweepFar;
              sz[m] = NM == 1 || m < n[2] ? uz * uz : kSweepFar;
            }
            unsigned int xq[NM], yq[NM], zq[NM], zmin = 0xffffffffu;
            if constexpr (KK == KK_EPAN && !CNT) {
#pragma unroll
              for (int m = 0; m < NM; ++m) {
                xq[m] = epan_x_units(sx[m]);
                yq[m] = epan_sq_units(sy[m]);
                zq[m] = epan_sq_units(sz[m]);
                zmin = min(zmin, zq[m]);
              }
            }
#pragma unroll
            for (int my = 0; my < NM; ++my) {
#pragma unroll
              for (int mx = 0; mx < NM; ++mx) {
                const int row = base + nbk[2] * my + nyz * mx;
                if constexpr (KK == KK_EPAN && !CNT) {
                  const unsigned int aq = epan_units(xq[mx], yq[my]);
                  // Lanes whose row has no nonzero term take no part: fewer
                  // lanes add to LDS, and the ranges' far ends need no tests
                  // of their own. Within a row of up to 3 nodes every
                  // lane adds, a zero where its term is 0 (a mask per node
                  // made 3-node supports 5% slower); wider spans add only
                  // nonzero terms: with 216 or more pairs per particle the
                  // unmasked adds made the LDS the bound (6 nodes: 5.9 -> 10
                  // ms on a full 100M-point box at 256^3).
                  if (!kRowTest || aq > zmin) {
#pragma unroll
                    for (int mz = 0; mz < NM; ++mz) {
                      const unsigned int q = epan_units(aq, zq[mz]);
                      if (NM <= 3 || q != 0u) atomicAdd(&sums[row + mz], (unsigned long long)q);
                    }
                  }
                } else {
                  const double sxy = sx[mx] + sy[my];
                  if (mx < n[0] && my < n[1]) {
#pragma unroll
                    for (int mz = 0; mz < NM; ++mz) {
                      const double u2 = sxy + sz[mz];
                      if (u2 < c2) {
                        unsigned int q;
                        if constexpr (CNT) {
                          q = 1u;
                        } else {
                          const float e = __builtin_amdgcn_exp2f((float)(SFK_KG64S * u2));
                          q = gauss_units(e);
                        }
                        atomicAdd(&sums[row + mz], (unsigned long long)q);
                      }
                    }
                  }
                }
              }
            }
          };
          // thread tid takes particles q = tid + 256 i of the surviving
          // leaves, in one of two orders
          if (ns > 0 && NM <= 2) {
            // Spans of 1 and 2 nodes add few terms per particle, so the LDS
            // atomics of one leaf's particles seldom meet (16 private copies
            // for their small windows): consecutive lanes take consecutive
            // particles of one leaf, and a wavefront's load is one 1 KB run
            // instead of 64 cache lines (3-node spans lost more to meeting
            // atomics than they gained)
            const bool all = ns == nl;
            const int total = ns * SFK_LEAF;
            int q = tid;
            if (q < total) {
              float4 p = pts[(int64_t)(all ? q >> 6 : lds_surv[q >> 6]) * SFK_LEAF + (q & 63)];
              while (true) {
                const int qn = q + 256;
                const bool more = qn < total;
                float4 pn = p;
                if (more) pn = pts[(int64_t)(all ? qn >> 6 : lds_surv[qn >> 6]) * SFK_LEAF + (qn & 63)];
                splat(p);
                if (!more) break;
                p = pn;
                q = qn;
              }
            }
          } else if (ns > 0) {
            // wider spans: "leaf q mod ns, slot q / ns", so the lanes of a
            // wavefront take particles of different leaves and one
            // instruction's atomics spread over the window
            const int step_slot = 256 / ns, step_leaf = 256 % ns;
            const bool all = ns == nl;  // every leaf reaches: no indirection
            auto leaf_id = [&](int q) { return all ? q : lds_surv[q]; };
            int leaf = tid % ns, slot = tid / ns;
            if (slot < SFK_LEAF) {
              float4 p = pts[(int64_t)leaf_id(leaf) * SFK_LEAF + slot];
              while (true) {
                int nleaf = leaf + step_leaf, nslot = slot + step_slot;
                if (nleaf >= ns) {
                  nleaf -= ns;
                  ++nslot;
                }
                const bool more = nslot < SFK_LEAF;
                float4 pn = p;
                if (more) pn = pts[(int64_t)leaf_id(nleaf) * SFK_LEAF + nslot];
                splat(p);
                if (!more) break;
                p = pn;
                leaf = nleaf;
                slot = nslot;
              }
            }
          }
          __syncthreads();
          // the window's nonzero sums into the batch's node sums: thread t
          // takes x = t mod W of the x rows t / W, t / W + 256 / W, ...
          // (consecutive threads add to consecutive nodes; the row's (y, z)
          // advances without divisions)
          if ((tid & (W - 1)) < nbk[0]) {
            constexpr int RS = 256 / W;
            const int li = tid & (W - 1);
            int lj = tid / W, lk = 0;
            while (lj >= nbk[1]) {
              lj -= nbk[1];
              ++lk;
            }
            while (lk < nbk[2]) {
              const int w = lk + nbk[2] * lj + nyz * li;
              unsigned long long v = 0ull;
              for (int c = 0; c < ncp; ++c) v += sums[c * cs + w];
              if (v != 0ull) {
                const int gi = blk0[0] + li, gj = blk0[1] + lj, gk = blk0[2] + lk;
                const int64_t t = R.tile_base + (gi / S) +
                                  (int64_t)R.ntile[0] * ((gj / S) + (int64_t)R.ntile[1] * (gk / S));
                atomicAdd(&acc[t * (S * S * S) + (gi % S) + S * ((gj % S) + S * (gk % S))], v);
              }
              lj += RS;
              while (lj >= nbk[1]) {
                lj -= nbk[1];
                ++lk;
              }
            }
          }
          __syncthreads();
        }
  }
  if (bad) claims[kErrWord] = 1;
}

// One block per tile of kSweep^3 nodes: sum * unit * scale, rounded once to
// float (the brick's conversion).
template <int KK, bool CNT>
__global__ __launch_bounds__(256) void k_sweep_write(const BatchHdr* __restrict__ hdr,
                                                     const RoiDev* __restrict__ rois,
                                                     const unsigned long long* __restrict__ acc) {
  constexpr int S = kSweep;
  const int64_t n_tiles = hdr->n_tiles;
  const int n_rois = hdr->n_rois;
  const double unit = kSumUnit<KK, CNT>;
  for (int64_t t = blockIdx.x; t < n_tiles; t += gridDim.x) {
    const int r = find_roi(rois, n_rois, t);
    const RoiDev& R = rois[r];
    const int64_t lt = t - R.tile_base;
    const int i0 = (int)(lt % R.ntile[0]) * S;
    const int j0 = (int)((lt / R.ntile[0]) % R.ntile[1]) * S;
    const int k0 = (int)(lt / ((int64_t)R.ntile[0] * R.ntile[1])) * S;
    for (int n = threadIdx.x; n < S * S * S; n += 256) {
      const int gi = i0 + n % S, gj = j0 + (n / S) % S, gk = k0 + n / (S * S);
      if (gi < R.res[0] && gj < R.res[1] && gk < R.res[2])
        R.out[gi + (int64_t)R.res[0] * (gj + (int64_t)R.res[1] * gk)] =
            (float)(((double)acc[t * (S * S * S) + n] * unit) * R.scale);
    }
  }
}

// ---------------------------------------------------------------------------
// debug: support sets of single nodes (one wavefront per node)
// ---------------------------------------------------------------------------

template <int TX, int TY, int TZ>
__global__ __launch_bounds__(256) void k_debug_candidates(TreeView tv, const int32_t* __restrict__ perm,
                                                          const RoiDev* __restrict__ rois,
                                                          const double* __restrict__ coords,
                                                          int64_t node_begin, int64_t node_end,
                                                          int64_t* __restrict__ cnt_out,
                                                          const int64_t* __restrict__ off,
                                                          int32_t* __restrict__ idx_out) {
  __shared__ int32_t lds_stack[4][SFK_STACK];
  const int lane = lane_id(), wave = threadIdx.x >> 6;
  const RoiDev& R = rois[0];
  const double* cx = coords + R.coord_off;
  const double* cy = cx + R.res[0];
  const double* cz = cy + R.res[1];
  for (int64_t nd = node_begin + (int64_t)blockIdx.x * 4 + wave; nd < node_end;
       nd += (int64_t)gridDim.x * 4) {
    const int ix = (int)(nd % R.res[0]);
    const int iy = (int)((nd / R.res[0]) % R.res[1]);
    const int iz = (int)(nd / ((int64_t)R.res[0] * R.res[1]));
    const int64_t t = (int64_t)(ix / TX) +
                      (int64_t)R.ntile[0] * ((int64_t)(iy / TY) + (int64_t)R.ntile[1] * (iz / TZ));
    const TileGeo g = tile_geo<TX, TY, TZ>(rois, 1, coords, t);
    const double xn = cx[ix], yn = cy[iy], zn = cz[iz];
    int64_t c = 0;
    int32_t* out = off ? idx_out + off[nd - node_begin] : nullptr;
    traverse(
        tv, lds_stack[wave],
        [&](const NodeBox& b, int gidx) { return tile_box_test(tv, R, g, b, gidx); },
        [&](int child, bool pass, uint64_t mask) {
          (void)pass;
          uint64_t mm = mask;
          while (mm) {
            const int b = __ffsll((unsigned long long)mm) - 1;
            mm &= mm - 1;
            const int lid = __shfl(child, b, 64);
            const int64_t slot = (int64_t)lid * SFK_LEAF + lane;
            const float4 p = tv.pts[slot];
            float ihx = R.ih[0], ihy = R.ih[1], ihz = R.ih[2];
            if (R.pp_mode == PP_ISO) {
              ihx = ihy = ihz = p.w;
            } else if (R.pp_mode == PP_ANISO) {
              const float4 q = tv.pparam[slot];
              ihx = q.x;
              ihy = q.y;
              ihz = q.z;
            }
            const bool mem =
                slot < tv.n && canon_u2(xn, yn, zn, p.x, p.y, p.z, ihx, ihy, ihz) < (double)R.c2;
            const uint64_t mb = ballot(mem);
            if (out && mem) out[c + popc64(mb & lanemask_lt())] = perm[slot];
            c += popc64(mb);
          }
        });
    if (!off && lane == 0) cnt_out[nd - node_begin] = c;
  }
}

// ---------------------------------------------------------------------------
// launch wrappers
// ---------------------------------------------------------------------------

bool tile_shape_supported(TileShape ts) {
  return (ts.tx == 4 && ts.ty == 4 && (ts.tz == 4 || ts.tz == 2)) ||
         (ts.tx == 4 && ts.ty == 2 && ts.tz == 2) || (ts.tx == 2 && ts.ty == 2 && ts.tz == 2) ||
         (ts.tx == 1 && ts.ty == 1 && ts.tz == 1) || is_brick(ts) || is_sweep(ts);
}

bool is_brick(TileShape ts) { return ts.tx == kBrick && ts.ty == kBrick && ts.tz == kBrick; }
bool is_sweep(TileShape ts) { return ts.tx == kSweep && ts.ty == kSweep && ts.tz == kSweep; }

hipError_t launch_sweep_list(TreeView tv, BatchHdr* hdr, const RoiDev* rois,
                             const double* coords, int64_t* items, unsigned long long* acc,
                             int32_t* claims, int max_rois, int64_t max_tiles, hipStream_t s) {
  constexpr int64_t T = kSweep * kSweep * kSweep;
  const int zb = (int)std::max<int64_t>(1, std::min<int64_t>((max_tiles * T + 255) / 256, 8192));
  hipLaunchKernelGGL(k_sweep_zero, dim3(zb), dim3(256), 0, s, hdr, acc, claims);
  const int L = tv.n_levels >= 2 ? 1 : 0;
  const int64_t ng = ((int64_t)tv.level_cnt[L] + 63) / 64;
  const int64_t waves = ng * std::max(1, max_rois);
  if (waves > 0)
    hipLaunchKernelGGL(k_sweep_list, dim3((unsigned)((waves + 3) / 4)), dim3(256), 0, s, tv, hdr,
                       rois, coords, items, claims);
  return hipGetLastError();
}

hipError_t launch_sweep_eval(TreeView tv, const BatchHdr* hdr, const RoiDev* rois,
                             const double* coords, int kk, bool cnt, int nm,
                             const int64_t* items, unsigned long long* acc, int32_t* claims,
                             int grid_blocks, int n_cu, int64_t max_tiles, hipStream_t s) {
  (void)coords;
  if (nm < 1 || nm > kSweepMaxNM) return hipErrorInvalidValue;
#define SFK_W(KK, C, NM)                                                                      \
  do {                                                                                        \
    static int occ_ = 0;                                                                      \
    if (occ_ == 0) {                                                                          \
      int b_ = 0;                                                                             \
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b_, k_sweep<KK, C, NM>, 256, 0) !=    \
              hipSuccess ||                                                                   \
          b_ < 1)                                                                             \
        b_ = 1;                                                                               \
      occ_ = b_;                                                                              \
    }                                                                                         \
    const int g_ = grid_blocks > 0 ? grid_blocks : n_cu * occ_;                               \
    hipLaunchKernelGGL((k_sweep<KK, C, NM>), dim3(g_), dim3(256), 0, s, tv, hdr, rois, items, \
                       acc, claims);                                                          \
  } while (0)
#define SFK_W_NM(KK, C)        \
  switch (nm) {                \
    case 1: SFK_W(KK, C, 1); break; \
    case 2: SFK_W(KK, C, 2); break; \
    case 3: SFK_W(KK, C, 3); break; \
    case 4: SFK_W(KK, C, 4); break; \
    case 5: SFK_W(KK, C, 5); break; \
    case 6: SFK_W(KK, C, 6); break; \
    case 7: SFK_W(KK, C, 7); break; \
    default: SFK_W(KK, C, 8); break; \
  }
  if (cnt) {
    SFK_W_NM(KK_EPAN, true);
  } else if (kk == KK_EPAN) {
    SFK_W_NM(KK_EPAN, false);
  } else {
    SFK_W_NM(KK_GAUSS, false);
  }
#undef SFK_W_NM
#undef SFK_W
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int wb = (int)std::max<int64_t>(1, std::min<int64_t>(max_tiles, 16384));
  if (cnt)
    hipLaunchKernelGGL((k_sweep_write<KK_EPAN, true>), dim3(wb), dim3(256), 0, s, hdr, rois, acc);
  else if (kk == KK_EPAN)
    hipLaunchKernelGGL((k_sweep_write<KK_EPAN, false>), dim3(wb), dim3(256), 0, s, hdr, rois, acc);
  else
    hipLaunchKernelGGL((k_sweep_write<KK_GAUSS, false>), dim3(wb), dim3(256), 0, s, hdr, rois, acc);
  return hipGetLastError();
}

// every shape of the range query (wavefront tiles and bricks)
#define SFK_SHAPE_SWITCH(ts, MACRO)                                  \
  do {                                                               \
    if ((ts).tx == kBrick && (ts).ty == kBrick && (ts).tz == kBrick) { \
      MACRO(kBrick, kBrick, kBrick);                                 \
    } else if ((ts).tx == 4 && (ts).ty == 4 && (ts).tz == 4) {       \
      MACRO(4, 4, 4);                                                \
    } else if ((ts).tx == 4 && (ts).ty == 4 && (ts).tz == 2) {       \
      MACRO(4, 4, 2);                                                \
    } else if ((ts).tx == 4 && (ts).ty == 2 && (ts).tz == 2) {       \
      MACRO(4, 2, 2);                                                \
    } else if ((ts).tx == 2 && (ts).ty == 2 && (ts).tz == 2) {       \
      MACRO(2, 2, 2);                                                \
    } else if ((ts).tx == 1 && (ts).ty == 1 && (ts).tz == 1) {       \
      MACRO(1, 1, 1);                                                \
    } else {                                                         \
      return hipErrorInvalidValue;                                   \
    }                                                                \
  } while (0)

static int grid_for(int64_t waves) {
  const int64_t b = (waves + 3) / 4;
  return (int)std::max<int64_t>(1, std::min<int64_t>(b, 65536));
}

int tile_grid_blocks(int64_t n_tiles) { return grid_for(n_tiles); }

hipError_t launch_tile_count(TreeView tv, const BatchHdr* hdr, const RoiDev* rois,
                             const double* coords, const int32_t* roi_leaves,
                             const int32_t* roi_nl, TileShape ts, int grid_blocks,
                             int32_t* tile_cnt, int32_t* tile_fit, int32_t* tile_done,
                             int32_t* tile_slots, hipStream_t s) {
  const int nb = std::max(1, grid_blocks);
#define SFK_L(X, Y, Z)                                                                      \
  hipLaunchKernelGGL((k_tile_count<X, Y, Z>), dim3(nb), dim3(256), 0, s, tv, hdr, rois,  \
                     coords, roi_leaves, roi_nl, tile_cnt, tile_fit, tile_done, tile_slots)
  SFK_SHAPE_SWITCH(ts, SFK_L);
#undef SFK_L
  return hipGetLastError();
}

// The whole plan in one block, for batches of at most kPlanNT tiles.
__global__ __launch_bounds__(kPlanNT) void k_plan_one(const int32_t* __restrict__ tile_cnt,
                                                      BatchHdr* __restrict__ hdr,
                                                      int32_t* __restrict__ claims,
                                                      int64_t* __restrict__ leaf_off,
                                                      int64_t* __restrict__ partial_off,
                                                      int64_t* __restrict__ chunk_off,
                                                      int32_t* __restrict__ tile_fit) {
  __shared__ int64_t lds[kPlanNT / 64];
  const int64_t n_tiles = hdr->n_tiles;
  const int64_t leaf_cap = hdr->leaf_cap, partial_cap = hdr->partial_cap;
  const int64_t t = threadIdx.x;
  const bool v = t < n_tiles;
  const int64_t cnt = v ? tile_cnt[t] : 0;
  int fit = v ? tile_fit[t] : 1 << kFitChunk;
  int64_t n = plan_items(cnt, fit_span(fit));
  int64_t pneed = plan_partials(n, hdr->splat);
  int64_t tl, tp, tc;
  const int64_t lo = block_excl_scan<kPlanNT>(cnt, &tl, lds);
  int64_t po = block_excl_scan<kPlanNT>(pneed, &tp, lds);
  const int64_t tf = tp;
  const bool coarse = tf > partial_cap;
  if (coarse) {
    fit |= 1 << kFitCoarse;
    n = plan_items(cnt, fit_span(fit));
    pneed = plan_partials(n, hdr->splat);
    po = block_excl_scan<kPlanNT>(pneed, &tp, lds);
  }
  const int mode = plan_mode(lo + cnt <= leaf_cap, pneed == 0 || po + pneed <= partial_cap, n,
                             hdr->splat);
  const int64_t nit = plan_count(cnt, n, mode);
  const int64_t co = block_excl_scan<kPlanNT>(nit, &tc, lds);
  if (v) {
    leaf_off[t] = lo;
    partial_off[t] = po;
    chunk_off[t] = co;
    tile_fit[t] = fit | mode;
  }
  // every thread has read the header above before thread 0 writes it
  __syncthreads();
  if (threadIdx.x < kClaimSlices) claims[threadIdx.x * kClaimStride] = 0;
  if (threadIdx.x == 0) {
    leaf_off[n_tiles] = tl;
    partial_off[n_tiles] = tp;
    chunk_off[n_tiles] = tc;
    hdr->total_leaves = tl;
    hdr->n_items = tc;
    hdr->total_partials = tp;
    hdr->fine_partials = tf;
    hdr->coarse = coarse ? 1 : 0;
  }
}

int plan_blocks(int64_t max_tiles) {
  return (int)std::max<int64_t>(1, (max_tiles + kPlanNT - 1) / kPlanNT);
}

hipError_t launch_plan(const int32_t* tile_cnt, BatchHdr* hdr, int32_t* claims, int64_t* leaf_off,
                       int64_t* partial_off, int64_t* chunk_off, int32_t* tile_fit,
                       int64_t* plan_tmp, int64_t max_tiles, hipStream_t s) {
  const int nb = plan_blocks(max_tiles);
  if (nb == 1) {
    hipLaunchKernelGGL(k_plan_one, dim3(1), dim3(kPlanNT), 0, s, tile_cnt, hdr, claims,
                       leaf_off, partial_off, chunk_off, tile_fit);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(k_plan_sums, dim3(nb), dim3(kPlanNT), 0, s, tile_cnt, tile_fit, hdr,
                     plan_tmp);
  hipLaunchKernelGGL(k_plan_modes, dim3(nb), dim3(kPlanNT), 0, s, tile_cnt, hdr, plan_tmp,
                     leaf_off, partial_off, chunk_off, tile_fit);
  hipLaunchKernelGGL(k_plan_items, dim3(nb), dim3(kPlanNT), 0, s, hdr, claims, plan_tmp,
                     leaf_off, partial_off, chunk_off);
  return hipGetLastError();
}

hipError_t launch_tile_fill(TreeView tv, const BatchHdr* hdr, const RoiDev* rois,
                            const double* coords, const int32_t* roi_leaves,
                            const int32_t* roi_nl, const int32_t* tile_slots, TileShape ts,
                            int grid_blocks, const int32_t* tile_cnt, const int32_t* tile_fit,
                            const int64_t* leaf_off, const int64_t* chunk_off, int32_t* leaves,
                            int32_t* item_tile, int32_t* claims, double* partials,
                            const int64_t* partial_off, hipStream_t s) {
  const int nb = std::max(1, grid_blocks);
#define SFK_L(X, Y, Z)                                                                     \
  hipLaunchKernelGGL((k_tile_fill<X, Y, Z>), dim3(nb), dim3(256), 0, s, tv, hdr, rois,  \
                     coords, roi_leaves, roi_nl, tile_slots, tile_cnt, tile_fit, leaf_off,  \
                     chunk_off, leaves, item_tile, claims, partials, partial_off)
  SFK_SHAPE_SWITCH(ts, SFK_L);
#undef SFK_L
  return hipGetLastError();
}

template <int X, int Y, int Z>
static hipError_t launch_eval_shape(int kk, int pp, bool cnt, int grid, int n_cu, int max_blocks,
                                    hipStream_t s,
                                    TreeView tv, const RoiDev* rois, const double* coords,
                                    const int64_t* leaf_off, const int64_t* chunk_off,
                                    const int64_t* partial_off,
                                    const int32_t* tile_cnt, const int32_t* tile_fit,
                                    const int32_t* leaves, const int32_t* item_tile,
                                    double* partials, int32_t* tile_done, BatchHdr* hdr,
                                    int32_t* claims) {
#define SFK_E(KK, PP, C)                                                                       \
  do {                                                                                         \
    static int occ_ = 0;                                                                       \
    if (occ_ == 0) {                                                                           \
      int b_ = 0;                                                                              \
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b_, k_eval<X, Y, Z, KK, PP, C>, 256,   \
                                                       0) != hipSuccess || b_ < 1)             \
        b_ = 1;                                                                                \
      occ_ = b_;                                                                               \
    }                                                                                          \
    const int g_ = grid > 0 ? grid : std::max(1, std::min(n_cu * occ_, max_blocks));          \
    hipLaunchKernelGGL((k_eval<X, Y, Z, KK, PP, C>), dim3(g_), dim3(256), 0, s, tv, rois,      \
                       coords, hdr, claims, leaf_off, chunk_off, partial_off, tile_cnt,        \
                       tile_fit, leaves, item_tile, partials, tile_done);                      \
  } while (0)
  if (cnt) {
    if (pp == PP_UNIFORM) SFK_E(KK_EPAN, PP_UNIFORM, true);
    else if (pp == PP_ISO) SFK_E(KK_EPAN, PP_ISO, true);
    else SFK_E(KK_EPAN, PP_ANISO, true);
  } else if (kk == KK_EPAN) {
    if (pp == PP_UNIFORM) SFK_E(KK_EPAN, PP_UNIFORM, false);
    else if (pp == PP_ISO) SFK_E(KK_EPAN, PP_ISO, false);
    else SFK_E(KK_EPAN, PP_ANISO, false);
  } else {
    if (pp == PP_UNIFORM) SFK_E(KK_GAUSS, PP_UNIFORM, false);
    else if (pp == PP_ISO) SFK_E(KK_GAUSS, PP_ISO, false);
    else SFK_E(KK_GAUSS, PP_ANISO, false);
  }
#undef SFK_E
  return hipGetLastError();
}

hipError_t launch_eval(TreeView tv, const BatchHdr* hdr_c, const RoiDev* rois,
                       const double* coords, TileShape ts, int kk, int pp, bool cnt,
                       const int64_t* leaf_off, const int64_t* chunk_off,
                       const int64_t* partial_off, const int32_t* tile_cnt,
                       const int32_t* tile_fit, const int32_t* leaves, const int32_t* item_tile,
                       double* partials, int32_t* tile_done, BatchHdr* hdr, int32_t* claims,
                       int grid_blocks, int n_cu, int max_blocks, hipStream_t s) {
  (void)hdr_c;
  if (is_brick(ts)) {
    if (pp != PP_UNIFORM) return hipErrorInvalidValue;
#define SFK_S(KK, C)                                                                          \
  do {                                                                                        \
    static int occ_ = 0;                                                                      \
    if (occ_ == 0) {                                                                          \
      int b_ = 0;                                                                             \
      if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b_, k_splat<KK, C>, 256, 0) !=        \
              hipSuccess ||                                                                   \
          b_ < 1)                                                                             \
        b_ = 1;                                                                               \
      occ_ = b_;                                                                              \
    }                                                                                         \
    const int g_ = grid_blocks > 0 ? grid_blocks : std::max(1, std::min(n_cu * occ_, max_blocks)); \
    hipLaunchKernelGGL((k_splat<KK, C>), dim3(g_), dim3(256), 0, s, tv, rois, coords,         \
                       hdr, claims, leaf_off, chunk_off, partial_off, tile_cnt, tile_fit,     \
                       leaves, item_tile, partials, tile_done);                               \
  } while (0)
    if (cnt)
      SFK_S(KK_EPAN, true);
    else if (kk == KK_EPAN)
      SFK_S(KK_EPAN, false);
    else
      SFK_S(KK_GAUSS, false);
#undef SFK_S
    return hipGetLastError();
  }
#define SFK_L(X, Y, Z)                                                                        \
  return launch_eval_shape<X, Y, Z>(kk, pp, cnt, grid_blocks, n_cu, max_blocks, s, tv, rois, \
                                    coords,                                                   \
                                    leaf_off, chunk_off, partial_off, tile_cnt,               \
                                    tile_fit, leaves, item_tile, partials, tile_done, hdr,    \
                                    claims)
  if ((ts).tx == 4 && (ts).ty == 4 && (ts).tz == 4) {
    SFK_L(4, 4, 4);
  } else if ((ts).tx == 4 && (ts).ty == 4 && (ts).tz == 2) {
    SFK_L(4, 4, 2);
  } else if ((ts).tx == 4 && (ts).ty == 2 && (ts).tz == 2) {
    SFK_L(4, 2, 2);
  } else if ((ts).tx == 2 && (ts).ty == 2 && (ts).tz == 2) {
    SFK_L(2, 2, 2);
  } else if ((ts).tx == 1 && (ts).ty == 1 && (ts).tz == 1) {
    SFK_L(1, 1, 1);
  }
#undef SFK_L
  return hipErrorInvalidValue;
}

hipError_t launch_debug_candidates2(TreeView tv, const int32_t* perm, const RoiDev* roi,
                                    const double* coords, TileShape ts, int64_t node_begin,
                                    int64_t node_end, int64_t* cnt, const int64_t* off,
                                    int32_t* idx_out, hipStream_t s) {
  const int64_t nn = node_end - node_begin;
  if (nn <= 0) return hipSuccess;
  const int nb = grid_for(nn);
#define SFK_L(X, Y, Z)                                                                     \
  hipLaunchKernelGGL((k_debug_candidates<X, Y, Z>), dim3(nb), dim3(256), 0, s, tv, perm, \
                     roi, coords, node_begin, node_end, cnt, off, idx_out)
  SFK_SHAPE_SWITCH(ts, SFK_L);
#undef SFK_L
  return hipGetLastError();
}

}  // namespace sfk
