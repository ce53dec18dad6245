// Kernels of the in-box particle set and of the MBE stages (Section 3.1):
// the particles inside a ROI's closed box B are compacted (keeping curve
// order) into a sub-cloud with its own leaves; Eq. 1 takes exact order
// statistics of each axis by radix selection; the adaptive smoothing length
// (Eqs. 5-6) interpolates the pilot grid at every particle, averages with a
// fixed-order two-level reduction (the paper's shared-memory group
// reduction followed by a mean of the group results, Alg. 3) and writes
// per-particle inverse lengths and weights for the final pass (Eq. 7).
#include <cmath>
#include <cstring>
#include <limits>

#include "sfk_device.h"

namespace sfk {

// In-box particles of each leaf, in two passes over the leaves: count, scan
// (by the caller), write. A leaf's count comes from its box alone where the
// box lies inside B or misses it (a particle in B lies in its leaf's box);
// only the leaves whose boxes B's surface cuts read their particles. A wavefront
// takes 16 leaves, so a box of a few thousand leaves still spreads over the
// chip, and asks for the particles of four at once.
//
// The order is the cloud's curve order, leaf by leaf and slot by slot. 1.56M
// leaves and 2.1M particles in the box take 90 us with the scan; flags, 64-bit
// positions and a compaction per candidate slot, with two reads of a total by
// the host instead of one, took 150.
static constexpr int kBoxLeaves = 16;  // leaves per wavefront

struct BoxB {
  double lo[3], hi[3];
  __device__ bool holds(float4 p) const {
    const double x = p.x, y = p.y, z = p.z;
    return p.x < 1.0e29f && x >= lo[0] && x <= hi[0] && y >= lo[1] && y <= hi[1] && z >= lo[2] &&
           z <= hi[2];
  }
};

// An empty leaf's box is inverted and never meets B.
__global__ __launch_bounds__(256) void k_box_count(const NodeBox* __restrict__ leaf_box,
                                                   const float4* __restrict__ pts,
                                                   int32_t n_leaves, BoxB bb,
                                                   int32_t* __restrict__ cnt) {
  const int lane = lane_id();
  const int64_t l0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kBoxLeaves;
  const int64_t l = l0 + lane;
  bool meet = false, inside = false;
  int32_t c = 0;
  if (lane < kBoxLeaves && l < n_leaves) {
    const NodeBox b = leaf_box[l];
    meet = inside = true;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      meet = meet && (double)b.lo[k] <= bb.hi[k] && (double)b.hi[k] >= bb.lo[k];
      inside = inside && (double)b.lo[k] >= bb.lo[k] && (double)b.hi[k] <= bb.hi[k];
    }
    if (meet && inside) c = b.count;
  }
  uint64_t cut = ballot(meet && !inside);
  while (cut) {
    int id[4];
    float4 p[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {  // past the last one: the same leaf again
      id[q] = cut ? __ffsll((unsigned long long)cut) - 1 : id[0];
      cut &= cut ? cut - 1 : 0;
      p[q] = pts[(l0 + id[q]) * SFK_LEAF + lane];
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const int in = popc64(ballot(bb.holds(p[q])));
      if (lane == id[q]) c = in;
    }
  }
  if (lane < kBoxLeaves && l < n_leaves) cnt[l] = c;
}

// pos: the counts' exclusive scan. Writes the in-box particles, their
// indices, their coordinates by axis (out_axes != nullptr) and the sentinels
// up to the sub-cloud's last slot.
__global__ __launch_bounds__(256) void k_box_write(
    const float4* __restrict__ pts, const int32_t* __restrict__ perm,
    const int32_t* __restrict__ cnt, const int64_t* __restrict__ pos, int32_t n_leaves, BoxB bb,
    int64_t n_b, int64_t n_slots_out, float4* __restrict__ out_pts,
    int32_t* __restrict__ out_perm, float* __restrict__ out_axes) {
  const int lane = lane_id();
  const int64_t l0 = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * kBoxLeaves;
  if (blockIdx.x == 0 && n_b + threadIdx.x < n_slots_out)
    // (w is a per-point inverse bandwidth: with 0 a slot would reach every node)
    out_pts[n_b + threadIdx.x] = make_float4(SFK_SENTINEL, SFK_SENTINEL, SFK_SENTINEL, 1.0f);
  int64_t at = 0;
  bool any = false;
  if (lane < kBoxLeaves && l0 + lane < n_leaves) {
    any = cnt[l0 + lane] > 0;
    if (any) at = pos[l0 + lane];
  }
  uint64_t m = ballot(any);
  while (m) {
    int id[4];
    float4 p[4];
    int32_t e[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      id[q] = m ? __ffsll((unsigned long long)m) - 1 : -1;
      m &= m ? m - 1 : 0;
      const int64_t src = (l0 + max(id[q], 0)) * SFK_LEAF + lane;
      if (id[q] >= 0) {
        p[q] = pts[src];
        const bool in = bb.holds(p[q]);
        e[q] = in ? perm[src] : 0;
      }
    }
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      if (id[q] < 0) break;
      const bool in = bb.holds(p[q]);
      const uint64_t im = ballot(in);
      const int64_t j = __shfl(at, id[q], 64) + popc64(im & lanemask_lt());
      if (in) {
        out_pts[j] = p[q];
        out_perm[j] = e[q];
        if (out_axes) {
          out_axes[j] = p[q].x;
          out_axes[n_b + j] = p[q].y;
          out_axes[2 * n_b + j] = p[q].z;
        }
      }
    }
  }
}

static BoxB make_box(const double* lo, const double* hi) {
  BoxB b;
  for (int k = 0; k < 3; ++k) {
    b.lo[k] = lo[k];
    b.hi[k] = hi[k];
  }
  return b;
}

hipError_t launch_box_count(const NodeBox* leaf_box, const float4* pts, int32_t n_leaves,
                            const double* lo, const double* hi, int32_t* cnt,
                            hipStream_t s) {
  if (n_leaves <= 0) return hipSuccess;
  const unsigned nb = (unsigned)((n_leaves + 4 * kBoxLeaves - 1) / (4 * kBoxLeaves));
  hipLaunchKernelGGL(k_box_count, dim3(nb), dim3(256), 0, s, leaf_box, pts, n_leaves,
                     make_box(lo, hi), cnt);
  return hipGetLastError();
}

hipError_t launch_box_write(const float4* pts, const int32_t* perm, const int32_t* cnt,
                            const int64_t* pos, int32_t n_leaves, const double* lo,
                            const double* hi, int64_t n_b, int64_t n_slots_out, float4* out_pts,
                            int32_t* out_perm, float* out_axes, hipStream_t s) {
  if (n_leaves <= 0) return hipSuccess;
  const unsigned nb = (unsigned)((n_leaves + 4 * kBoxLeaves - 1) / (4 * kBoxLeaves));
  hipLaunchKernelGGL(k_box_write, dim3(nb), dim3(256), 0, s, pts, perm, cnt, pos, n_leaves,
                     make_box(lo, hi), n_b, n_slots_out, out_pts, out_perm, out_axes);
  return hipGetLastError();
}

// float -> unsigned key with the same order (negative values flipped)
__host__ __device__ __forceinline__ uint32_t ord_of_bits(uint32_t b) {
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ uint32_t f2ord(float f) { return ord_of_bits(__float_as_uint(f)); }
__device__ __forceinline__ float ord2f(uint32_t u) {
  const uint32_t b = (u & 0x80000000u) ? (u & 0x7fffffffu) : ~u;
  return __uint_as_float(b);
}

// ---- Eq. 1's order statistics: radix selection ----
//
// A type-7 percentile needs the values of two neighbouring ranks, so Eq. 1
// reads four ranks per axis and no order of the rest. Each pass counts one
// digit of the keys that still share a wanted rank's leading digits; the next
// pass finds the digit that holds each rank and goes one digit down. Keys are
// the order-preserving bits of the coordinate minus those of the box's low
// corner: every particle lies in the closed box, so the highest set bit of
// the key range is known, the first digit spreads over the box (the raw
// leading bits, sign and exponent, would meet in a few counters) and a box
// that spans at most two octaves takes two passes of 12 bits, any box three.
//
// Bound by the counters' traffic and the launches: 2.1M particles are 25 MB a
// pass, 5 us, and a pass takes 21. The two passes and k_mbe_ell take 50 us
// where a radix sort of the three axes (5 passes over 12-byte pairs, with its
// scans) took 1.1 ms; with the in-box set taken leaf by leaf, 3.06 -> 2.54 ms
// for the whole estimate (100M clustered points, box of side 0.05, 128^3),
// 980 -> 740 us for 0.1M of 442k points at 64^3.
static constexpr int kSelBits = 12, kSelBins = 1 << kSelBits, kSelRanks = 4, kSelPasses = 3;
static constexpr int kSelNT = 1024;

struct SelState {  // after a pass, per axis and wanted rank
  uint32_t prefix[kSelRanks];  // the digits found, as a number
  uint32_t rank[kSelRanks];    // rank among the keys with that prefix
};

// Bits [shift, shift + width) of an axis's keys that pass `pass` counts; an
// axis whose bits are used up counts nothing (width 0).
struct SelAxes {
  uint32_t base[3];
  int32_t bits[3];
  __host__ __device__ int shift(int axis, int pass) const {
    const int r = bits[axis] - kSelBits * (pass + 1);
    return r > 0 ? r : 0;
  }
  __host__ __device__ int width(int axis, int pass) const {
    const int r = bits[axis] - kSelBits * pass;
    return r < 0 ? 0 : (r < kSelBits ? r : kSelBits);
  }
};

// Ranks i and i + 1 (at most n - 1) of the type-7 percentiles 0.2 and 0.8.
__device__ __forceinline__ int64_t type7_pos(int64_t n, double q, double* frac) {
  const double pos = (double)(n - 1) * q;
  const int64_t i = (int64_t)floor(pos);
  *frac = pos - (double)i;
  return i;
}
__device__ __forceinline__ uint32_t wanted_rank(int64_t n, int r) {
  double f;
  const int64_t i = type7_pos(n, r < 2 ? 0.20 : 0.80, &f) + (r & 1);
  return (uint32_t)(i < n ? i : n - 1);
}

// The wanted ranks' keys with equal prefixes share the first one's counters.
__device__ __forceinline__ int sel_slot(const SelState& st, int r) {
  int q = 0;
  while (st.prefix[q] != st.prefix[r]) ++q;
  return q;
}

// One wavefront: the digit that holds wanted rank r after pass `pass` counted
// (before: the state before that pass, hist: the axis's counters).
__device__ __forceinline__ void sel_descend(const SelState& before, int r,
                                            const uint32_t* __restrict__ hist, int width,
                                            uint32_t* prefix, uint32_t* rank) {
  *prefix = before.prefix[r];
  *rank = before.rank[r];
  if (width == 0) return;  // every digit was counted before
  const uint32_t* h = hist + (size_t)sel_slot(before, r) * kSelBins;
  constexpr int kPer = kSelBins / 64;
  uint32_t v[kPer], sum = 0;
#pragma unroll
  for (int i = 0; i < kPer; i += 4) {
    const uint4 q = *(const uint4*)(h + lane_id() * kPer + i);
    v[i] = q.x;
    v[i + 1] = q.y;
    v[i + 2] = q.z;
    v[i + 3] = q.w;
    sum += q.x + q.y + q.z + q.w;
  }
  const uint32_t inc = wave_incl_scan(sum);
  uint32_t left = *rank - (inc - sum), digit = 0;  // meant for the owner alone
  const uint64_t own = ballot(*rank >= inc - sum && *rank < inc);
  bool found = false;
#pragma unroll
  for (int i = 0; i < kPer; ++i) {
    if (!found && left < v[i]) {
      digit = (uint32_t)(lane_id() * kPer + i);
      found = true;
    }
    if (!found) left -= v[i];
  }
  const int src = own ? __ffsll((unsigned long long)own) - 1 : 63;
  *prefix = (*prefix << width) | (uint32_t)__shfl((int)digit, src, 64);
  *rank = (uint32_t)__shfl((int)left, src, 64);
}

// Pass `pass` over one axis (blockIdx.y): counters of this pass's digit for
// the keys that share a wanted prefix, in LDS, then added to the axis's.
__global__ __launch_bounds__(kSelNT) void k_axis_count(const float* __restrict__ axes, int64_t n_b,
                                                       SelAxes sa, int pass,
                                                       uint32_t* __restrict__ hist,
                                                       SelState* __restrict__ states) {
  __shared__ uint32_t cnt[kSelRanks * kSelBins];
  __shared__ SelState st;
  const int axis = blockIdx.y, w = threadIdx.x >> 6;
  const size_t pass_words = (size_t)3 * kSelRanks * kSelBins;
  if (pass == 0) {
    if (threadIdx.x < kSelRanks) {
      st.prefix[threadIdx.x] = 0;
      st.rank[threadIdx.x] = wanted_rank(n_b, (int)threadIdx.x);
    }
  } else if (w < kSelRanks) {
    uint32_t p, r;
    sel_descend(states[(pass - 1) * 3 + axis], w,
                hist + (pass - 1) * pass_words + (size_t)axis * kSelRanks * kSelBins,
                sa.width(axis, pass - 1), &p, &r);
    if (lane_id() == 0) {
      st.prefix[w] = p;
      st.rank[w] = r;
    }
  }
  const int width = sa.width(axis, pass), shift = sa.shift(axis, pass);
  const int words = pass == 0 ? kSelBins : kSelRanks * kSelBins;
  for (int i = threadIdx.x; i < words; i += kSelNT) cnt[i] = 0;
  __syncthreads();
  if (blockIdx.x == 0 && threadIdx.x < kSelRanks) {
    states[pass * 3 + axis].prefix[threadIdx.x] = st.prefix[threadIdx.x];
    states[pass * 3 + axis].rank[threadIdx.x] = st.rank[threadIdx.x];
  }
  if (width == 0) return;
  const float* x = axes + (size_t)axis * n_b;
  const uint32_t base = sa.base[axis], mask = (1u << width) - 1u;
  const int64_t stride = (int64_t)gridDim.x * kSelNT;
  const int64_t first = (int64_t)blockIdx.x * kSelNT + threadIdx.x;
  if (pass == 0) {
#pragma unroll 4
    for (int64_t i = first; i < n_b; i += stride)
      atomicAdd(&cnt[((f2ord(x[i]) - base) >> shift) & mask], 1u);
  } else {
    const int up = shift + width;  // < 32: a digit lies above it
    uint32_t pre[kSelRanks];
    int slot[kSelRanks];
#pragma unroll
    for (int r = 0; r < kSelRanks; ++r) {
      pre[r] = st.prefix[r];
      slot[r] = sel_slot(st, r) * kSelBins;
    }
#pragma unroll 4
    for (int64_t i = first; i < n_b; i += stride) {
      const uint32_t key = f2ord(x[i]) - base, top = key >> up;
      int at = -1;
#pragma unroll
      for (int r = 0; r < kSelRanks; ++r)
        if (top == pre[r]) at = slot[r];
      if (at >= 0) atomicAdd(&cnt[at + (int)((key >> shift) & mask)], 1u);
    }
  }
  __syncthreads();
  uint32_t* g = hist + pass * pass_words + (size_t)axis * kSelRanks * kSelBins;
  for (int i = threadIdx.x; i < words; i += kSelNT)
    if (cnt[i]) atomicAdd(&g[i], cnt[i]);
}

// Eq. 1: l_k = 2 (P80 - P20) / ln(N_B); a non-positive or non-finite
// result (N_B < 2, or P80 == P20) takes the cap 5 s_k of Eq. 6. One
// wavefront per axis and wanted rank takes the last digit down.
__global__ __launch_bounds__(64 * 3 * kSelRanks) void k_mbe_ell(
    const uint32_t* __restrict__ hist, const SelState* __restrict__ states, SelAxes sa,
    int passes, int64_t n_b, double lx, double ly, double lz, double hx, double hy, double hz,
    int rx, int ry, int rz, float* __restrict__ ell_out) {
  __shared__ double val[3 * kSelRanks];
  const int w = threadIdx.x >> 6, axis = w / kSelRanks, r = w % kSelRanks, last = passes - 1;
  uint32_t p, left;
  sel_descend(states[last * 3 + axis], r,
              hist + (size_t)(last * 3 + axis) * kSelRanks * kSelBins, sa.width(axis, last), &p,
              &left);
  if (lane_id() == 0) val[w] = (double)ord2f(p + sa.base[axis]);
  __syncthreads();
  if (threadIdx.x >= 3) return;
  const int k = threadIdx.x;
  const double lo = k == 0 ? lx : (k == 1 ? ly : lz);
  const double hi = k == 0 ? hx : (k == 1 ? hy : hz);
  const int res = k == 0 ? rx : (k == 1 ? ry : rz);
  const double cap = 5.0 * ((hi - lo) / (double)(res - 1));
  double l = __builtin_nan("");
  if (n_b >= 2) {
    const double* v = val + k * kSelRanks;
    double f20, f80;
    (void)type7_pos(n_b, 0.20, &f20);
    (void)type7_pos(n_b, 0.80, &f80);
    const double p20 = v[0] + f20 * (v[1] - v[0]);
    const double p80 = v[2] + f80 * (v[3] - v[2]);
    l = 2.0 * (p80 - p20) / log((double)n_b);
  }
  if (!(l > 0.0) || !isfinite(l)) l = cap;
  ell_out[k] = (float)l;
}

size_t axis_select_tmp_bytes() {
  return sizeof(uint32_t) * kSelPasses * 3 * kSelRanks * kSelBins +
         sizeof(SelState) * kSelPasses * 3;
}

// Eq. 1's lengths from the particles' coordinates (three arrays of n_b, all
// within the closed box [lo, hi]).
hipError_t launch_axis_select(const float* axes, int64_t n_b, const double* lo, const double* hi,
                              const int32_t* res, void* tmp, float* ell_out, hipStream_t s) {
  if (n_b <= 0) return hipSuccess;
  SelAxes sa;
  int passes = 1;
  for (int k = 0; k < 3; ++k) {
    // the floats at or outside the corners (a corner 0 admits both zeros)
    const float inf = std::numeric_limits<float>::infinity();
    float a = (float)lo[k], b = (float)hi[k];
    if ((double)a > lo[k]) a = std::nextafter(a, -inf);
    if ((double)b < hi[k]) b = std::nextafter(b, inf);
    if (a == 0.0f) a = -0.0f;
    if (b == 0.0f) b = 0.0f;
    uint32_t ab, bb;
    std::memcpy(&ab, &a, sizeof ab);
    std::memcpy(&bb, &b, sizeof bb);
    sa.base[k] = ord_of_bits(ab);
    const uint32_t range = ord_of_bits(bb) - sa.base[k];
    sa.bits[k] = 0;
    while (sa.bits[k] < 32 && (range >> sa.bits[k])) ++sa.bits[k];
    passes = std::max(passes, (sa.bits[k] + kSelBits - 1) / kSelBits);
  }
  uint32_t* hist = (uint32_t*)tmp;
  const size_t words = (size_t)passes * 3 * kSelRanks * kSelBins;
  SelState* states = (SelState*)(hist + (size_t)kSelPasses * 3 * kSelRanks * kSelBins);
  hipError_t e = launch_fill_f32((float*)hist, (int64_t)words, 0.0f, s);
  if (e != hipSuccess) return e;
  // 8 loads in flight a thread; 128 blocks an axis keep the adds into the
  // shared counters to a few thousand a block
  const int64_t nb = std::min<int64_t>((n_b + kSelNT * 8 - 1) / (kSelNT * 8), 128);
  for (int p = 0; p < passes; ++p)
    hipLaunchKernelGGL(k_axis_count, dim3((unsigned)nb, 3), dim3(kSelNT), 0, s, axes, n_b, sa, p,
                       hist, states);
  hipLaunchKernelGGL(k_mbe_ell, dim3(1), dim3(64 * 3 * kSelRanks), 0, s, hist, states, sa, passes,
                     n_b, lo[0], lo[1], lo[2], hi[0], hi[1], hi[2], res[0], res[1], res[2],
                     ell_out);
  return hipGetLastError();
}

// Trilinear interpolation of the pilot grid at each particle of B
// (f = (p - lo)(res - 1)/(hi - lo), cell clamped to [0, res - 2], t clamped
// to [0, 1]), in double; per-block sums for the mean (fixed order).
struct GridGeo {
  double lo[3], hi[3];
  int res[3];
};

__global__ __launch_bounds__(256) void k_trilinear(const float4* __restrict__ pts, int64_t n_b,
                                                   const float* __restrict__ grid, GridGeo gg,
                                                   double* __restrict__ pden,
                                                   double* __restrict__ block_sums) {
  __shared__ double lds[4];
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  double val = 0.0;
  if (j < n_b) {
    const float4 p = pts[j];
    const float pc[3] = {p.x, p.y, p.z};
    int ci[3];
    double tt[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double f = ((double)pc[k] - gg.lo[k]) * (double)(gg.res[k] - 1) / (gg.hi[k] - gg.lo[k]);
      int c = (int)floor(f);
      if (c < 0) c = 0;
      if (c > gg.res[k] - 2) c = gg.res[k] - 2;
      double t = f - (double)c;
      if (t < 0.0) t = 0.0;
      if (t > 1.0) t = 1.0;
      ci[k] = c;
      tt[k] = t;
    }
    double a = 0.0;
    for (int dz = 0; dz < 2; ++dz)
      for (int dy = 0; dy < 2; ++dy)
        for (int dx = 0; dx < 2; ++dx) {
          const double wgt = (dx ? tt[0] : 1.0 - tt[0]) * (dy ? tt[1] : 1.0 - tt[1]) *
                             (dz ? tt[2] : 1.0 - tt[2]);
          const int64_t idx = (int64_t)(ci[0] + dx) +
                              (int64_t)gg.res[0] * ((int64_t)(ci[1] + dy) +
                                                    (int64_t)gg.res[1] * (ci[2] + dz));
          a += wgt * (double)grid[idx];
        }
    pden[j] = a;
    val = a;
  }
  val = wave_sum(val);
  if (lane_id() == 0) lds[threadIdx.x >> 6] = val;
  __syncthreads();
  if (threadIdx.x == 0) block_sums[blockIdx.x] = ((lds[0] + lds[1]) + lds[2]) + lds[3];
}

// aveDen = (sum of block sums) / N_B, one block, fixed order.
__global__ __launch_bounds__(256) void k_mean(const double* __restrict__ block_sums, int nblk,
                                              int64_t n_b, double* __restrict__ ave) {
  __shared__ double lds[4];
  double s = 0.0;
  for (int i = threadIdx.x; i < nblk; i += 256) s += block_sums[i];
  s = wave_sum(s);
  if (lane_id() == 0) lds[threadIdx.x >> 6] = s;
  __syncthreads();
  if (threadIdx.x == 0) *ave = n_b > 0 ? (((lds[0] + lds[1]) + lds[2]) + lds[3]) / (double)n_b : 0.0;
}

// Eq. 6 per particle; pden <= 0 takes the cap. The last leaf's padding slots
// get finite parameters too (a zero would reach every node).
__global__ __launch_bounds__(256) void k_asl(const double* __restrict__ pden, int64_t n_b,
                                             const double* __restrict__ ave_p, float e0, float e1,
                                             float e2, GridGeo gg, float4* __restrict__ pparam,
                                             float* __restrict__ ell_out) {
  const double ave = *ave_p;
  const float e[3] = {e0, e1, e2};
  if (blockIdx.x == 0 && threadIdx.x < ((-n_b) & (SFK_LEAF - 1)))
    pparam[n_b + threadIdx.x] = make_float4(1.0f, 1.0f, 1.0f, 0.0f);
  for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n_b;
       j += (int64_t)gridDim.x * blockDim.x) {
    const double pd = pden[j];
    float l[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
      const double cap = 5.0 * ((gg.hi[k] - gg.lo[k]) / (double)(gg.res[k] - 1));
      double v;
      if (pd > 0.0) {
        v = (double)e[k] * cbrt(ave / pd);
        if (v > cap) v = cap;
      } else {
        v = cap;
      }
      l[k] = (float)v;
    }
    const double lx = l[0], ly = l[1], lz = l[2];
    pparam[j] = make_float4((float)(1.0 / lx), (float)(1.0 / ly), (float)(1.0 / lz),
                            (float)(1.0 / (lx * ly * lz)));
    if (ell_out) {
      ell_out[3 * j] = l[0];
      ell_out[3 * j + 1] = l[1];
      ell_out[3 * j + 2] = l[2];
    }
  }
}

hipError_t launch_trilinear_mean(const float4* pts, int64_t n_b, const float* grid,
                                 const double* lo, const double* hi, const int32_t* res,
                                 double* pden, double* block_sums, double* ave, hipStream_t s) {
  if (n_b <= 0) return hipSuccess;
  GridGeo gg;
  for (int k = 0; k < 3; ++k) {
    gg.lo[k] = lo[k];
    gg.hi[k] = hi[k];
    gg.res[k] = res[k];
  }
  const int nblk = (int)((n_b + 255) / 256);
  hipLaunchKernelGGL(k_trilinear, dim3(nblk), dim3(256), 0, s, pts, n_b, grid, gg, pden,
                     block_sums);
  hipLaunchKernelGGL(k_mean, dim3(1), dim3(256), 0, s, block_sums, nblk, n_b, ave);
  return hipGetLastError();
}

hipError_t launch_asl2(const double* pden, int64_t n_b, const double* ave, const float* ell0,
                       const double* lo, const double* hi, const int32_t* res, float4* pparam,
                       float* ell_out, hipStream_t s) {
  if (n_b <= 0) return hipSuccess;
  GridGeo gg;
  for (int k = 0; k < 3; ++k) {
    gg.lo[k] = lo[k];
    gg.hi[k] = hi[k];
    gg.res[k] = res[k];
  }
  const int64_t nb = std::min<int64_t>((n_b + 255) / 256, 65536);
  hipLaunchKernelGGL(k_asl, dim3((unsigned)nb), dim3(256), 0, s, pden, n_b, ave, ell0[0], ell0[1],
                     ell0[2], gg, pparam, ell_out);
  return hipGetLastError();
}

}  // namespace sfk
