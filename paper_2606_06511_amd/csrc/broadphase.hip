// Broad phase: candidate triangle pairs for the per-pair energy (Sec. 1.2 removes redundant
// pair tests with a spatial structure; this is a linear BVH over Morton-sorted triangles).
//
//   k_bp_init      reset the pair counter
//   k_tri_boxes    exact FP64 bounding box per triangle (optionally swept to a second position);
//                  per-block bounds of the box centres
//                  (order-preserving integer keys)
//   k_morton       reduce those bounds, then a 30-bit Morton code per box centre; counts of
//                  the top bits (about two triangles per bucket), each triangle taking its
//                  rank inside its bucket from the counting atomic
//   scan, scatter  counting sort of the triangles by bucket (order inside a bucket arbitrary)
//   k_levels       an implicit complete 4-ary tree over the sorted leaves: node (l, k) covers
//                  leaves [k 4^l, (k+1) 4^l); FP32 boxes (rounded outwards) are reduced by waves
//                  in registers, four levels per launch from the leaves, five per launch above,
//                  so building needs no atomics and no fences.  The first launch also writes the
//                  sorted leaves' vertex ids.  Each inner node also records a vertex all its
//                  triangles hold, if there is one.
//   k_traverse     a wave per group of 64 consecutive leaves searches the tree once for all of
//                  them and tests the leaves it meets against the 64 queries; a pair is confirmed
//                  by the exact closed FP64 box test and the shared-vertex test
//   k_traverse_heavy  the candidate batches and nodes that waves over their budget handed over
//   k_brute        all i < j without a shared vertex (no box test)

#include "internal.h"

namespace ttie {

constexpr int kBpBlock = 256;
constexpr int kBoundsBlocks = 512;  // partial-bounds slots in the workspace

__device__ __forceinline__ uint32_t f2key(float f) {
  const uint32_t b = __float_as_uint(f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}
__device__ __forceinline__ float key2f(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// zeroes the caller's pair count and the broad phase's counters (the LBVH and the hash do it in
// k_tri_boxes instead, saving a launch)
__global__ void k_bp_init(Counters* c, unsigned long long* npairs) {
  if (threadIdx.x == 0) {
    *npairs = 0;
    c->n_entries = 0;
    c->n_heavy = 0;
    c->n_batches = 0;
  }
}

// minimum and maximum over the wave's lanes, in lane 63 (the identity comes in where a pattern
// names no lane)
template <int kCtrl, int kRows>
__device__ __forceinline__ uint32_t dpp_or(uint32_t v, uint32_t id) {
  return (uint32_t)__builtin_amdgcn_update_dpp((int)id, (int)v, kCtrl, kRows, 0xf, false);
}
__device__ __forceinline__ uint32_t wave_min(uint32_t v) {
  v = min(v, dpp_or<0x111, 0xf>(v, ~0u));
  v = min(v, dpp_or<0x112, 0xf>(v, ~0u));
  v = min(v, dpp_or<0x114, 0xf>(v, ~0u));
  v = min(v, dpp_or<0x118, 0xf>(v, ~0u));
  v = min(v, dpp_or<0x142, 0xa>(v, ~0u));
  return min(v, dpp_or<0x143, 0xc>(v, ~0u));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) { return ~wave_min(~v); }

// A pass over bytes (a triangle's 12 read and its corners' 72, mostly cached; 60 written): 151 us
// for 4,194,304 triangles, however many threads a block has.  On small meshes its latency counts:
// with sums through registers instead of shared memory 3.2 us instead of 3.9 on 640 triangles (and
// k_morton 7.2 instead of 8.0).
__global__ void __launch_bounds__(kBpBlock) k_tri_boxes(const double* __restrict__ x, const double* __restrict__ x_end,
                                                        int64_t nv, const int32_t* __restrict__ tris, int64_t nt,
                                                        double* __restrict__ tbox, float* __restrict__ centre,
                                                        uint32_t* __restrict__ part, double* __restrict__ ext_part,
                                                        unsigned long long* npairs, Counters* ctr) {
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    *npairs = 0;
    ctr->n_entries = 0;
    ctr->n_heavy = 0;
    ctr->n_batches = 0;
  }
  constexpr int kW = kBpBlock / 64;
  __shared__ uint32_t sb[6][kW];
  __shared__ double sext[kW];
  uint32_t lmin[3] = {0xffffffffu, 0xffffffffu, 0xffffffffu}, lmax[3] = {0u, 0u, 0u};
  double ext = 0.0;  // sum of the boxes' largest extents (the hash grid's cell size)
  bool bad = false;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < nt; t += (int64_t)gridDim.x * blockDim.x) {
    double lo[3] = {0, 0, 0}, hi[3] = {0, 0, 0};
    // the row, then all nine coordinates at once (a triangle with an index out of range is
    // reported and gets the empty box at the origin)
    const int32_t vr[3] = {tris[3 * t], tris[3 * t + 1], tris[3 * t + 2]};
    const bool ok = vr[0] >= 0 && vr[0] < nv && vr[1] >= 0 && vr[1] < nv && vr[2] >= 0 && vr[2] < nv;
    if (ok) {
      double q[3][3];
#pragma unroll
      for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int c = 0; c < 3; ++c) q[k][c] = x[3 * (int64_t)vr[k] + c];
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        lo[c] = fmin(q[0][c], fmin(q[1][c], q[2][c]));
        hi[c] = fmax(q[0][c], fmax(q[1][c], q[2][c]));
      }
      if (x_end) {  // swept box: the triangle at both ends of the straight path
#pragma unroll
        for (int k = 0; k < 3; ++k)
#pragma unroll
          for (int c = 0; c < 3; ++c) q[k][c] = x_end[3 * (int64_t)vr[k] + c];
#pragma unroll
        for (int c = 0; c < 3; ++c) {
          lo[c] = fmin(lo[c], fmin(q[0][c], fmin(q[1][c], q[2][c])));
          hi[c] = fmax(hi[c], fmax(q[0][c], fmax(q[1][c], q[2][c])));
        }
      }
    } else {
      bad = true;
    }
    ext += fmax(hi[0] - lo[0], fmax(hi[1] - lo[1], hi[2] - lo[2]));
    double2* const row = reinterpret_cast<double2*>(tbox + 6 * t);
    row[0] = make_double2(lo[0], lo[1]);
    row[1] = make_double2(lo[2], hi[0]);
    row[2] = make_double2(hi[1], hi[2]);
    for (int c = 0; c < 3; ++c) {
      const uint32_t kc = f2key((float)(0.5 * (lo[c] + hi[c])));
      centre[3 * t + c] = (float)(0.5 * (lo[c] + hi[c]));
      lmin[c] = min(lmin[c], kc);
      lmax[c] = max(lmax[c], kc);
    }
  }
  if (bad) atomicCAS(&ctr->status, 0, STATUS_INDEX);
  // per-block partial bounds and extent sums; the next kernel reduces them (the kernel
  // boundary orders the two)
  const int wave = threadIdx.x / 64;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    const uint32_t a = wave_min(lmin[c]), b = wave_max(lmax[c]);
    if (__lane_id() == 63) {
      sb[c][wave] = a;
      sb[3 + c][wave] = b;
    }
  }
#pragma unroll
  for (int d = 32; d > 0; d >>= 1) ext += __shfl_xor(ext, d);
  if (__lane_id() == 0) sext[wave] = ext;
  __syncthreads();
  if (threadIdx.x < 6) {
    uint32_t v = sb[threadIdx.x][0];
    for (int w = 1; w < kW; ++w) v = threadIdx.x < 3 ? min(v, sb[threadIdx.x][w]) : max(v, sb[threadIdx.x][w]);
    part[6 * blockIdx.x + threadIdx.x] = v;
  }
  if (threadIdx.x == 0) {
    double e = 0.0;
    for (int w = 0; w < kW; ++w) e += sext[w];
    ext_part[blockIdx.x] = e;
  }
}

// spread the low 10 bits of v to every third bit
__device__ __forceinline__ uint32_t spread3(uint32_t v) {
  v &= 0x3ffu;
  v = (v | (v << 16)) & 0x030000ffu;
  v = (v | (v << 8)) & 0x0300f00fu;
  v = (v | (v << 4)) & 0x030c30c3u;
  v = (v | (v << 2)) & 0x09249249u;
  return v;
}

// the problem owning item t: the last p with off[p] <= t, clamped to [0, n_prob)
__device__ __forceinline__ int problem_of(const int64_t* __restrict__ off, int n_prob, int64_t t) {
  int lo = 0, hi = n_prob - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (off[mid] <= t) lo = mid;
    else hi = mid - 1;
  }
  return lo;
}

// Bucket of a triangle: its problem in the top bits, then the top mbits of its Morton code, so
// every problem's triangles form one contiguous range of the sorted order.
__global__ void __launch_bounds__(kBpBlock) k_morton(const float* __restrict__ centre, int64_t nt,
                                                     const uint32_t* __restrict__ part, int nparts,
                                                     const int64_t* __restrict__ tri_off, int n_prob, int mbits,
                                                     int32_t* __restrict__ hist, uint32_t* __restrict__ bucket,
                                                     int32_t* __restrict__ rank, Counters* ctr) {
  if (tri_off && blockIdx.x == 0) {
    // the problem ranges must tile [0, nt)
    bool bad = threadIdx.x == 0 && (tri_off[0] != 0 || tri_off[n_prob] != nt);
    for (int p = threadIdx.x; p < n_prob; p += kBpBlock) bad |= tri_off[p] > tri_off[p + 1];
    if (bad) atomicCAS(&ctr->status, 0, STATUS_INVALID);
  }
  // every block reduces the per-block bounds of k_tri_boxes (a few KB, cached)
  __shared__ uint32_t wb[6][kBpBlock / 64];
  uint32_t sb[6] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0u, 0u, 0u};
  for (int b = threadIdx.x; b < nparts; b += kBpBlock)
    for (int c = 0; c < 6; ++c) sb[c] = c < 3 ? min(sb[c], part[6 * b + c]) : max(sb[c], part[6 * b + c]);
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    const uint32_t v = c < 3 ? wave_min(sb[c]) : wave_max(sb[c]);
    if (__lane_id() == 63) wb[c][threadIdx.x / 64] = v;
  }
  __syncthreads();
#pragma unroll
  for (int c = 0; c < 6; ++c) {
    sb[c] = wb[c][0];
#pragma unroll
    for (int w = 1; w < kBpBlock / 64; ++w) sb[c] = c < 3 ? min(sb[c], wb[c][w]) : max(sb[c], wb[c][w]);
  }
  float lo[3], inv[3];
  for (int c = 0; c < 3; ++c) {
    lo[c] = key2f(sb[c]);
    const float ext = key2f(sb[3 + c]) - lo[c];
    inv[c] = ext > 0.f ? 1023.f / ext : 0.f;
  }
  const int lane = __lane_id();
  for (int64_t base = (int64_t)blockIdx.x * blockDim.x; base < nt; base += (int64_t)gridDim.x * blockDim.x) {
    const int64_t t = base + threadIdx.x;
    const bool active = t < nt;
    uint32_t bk = 0;
    if (active) {
      uint32_t q[3];
      for (int c = 0; c < 3; ++c) {
        const float f = (centre[3 * t + c] - lo[c]) * inv[c];
        q[c] = (uint32_t)fminf(fmaxf(f, 0.f), 1023.f);
      }
      const uint32_t code = (spread3(q[0]) << 2) | (spread3(q[1]) << 1) | spread3(q[2]);
      const uint32_t p = tri_off ? (uint32_t)problem_of(tri_off, n_prob, t) : 0u;
      bk = (p << mbits) | (code >> (30 - mbits));
      bucket[t] = bk;
    }
    // Neighbouring triangles share buckets: group the wave's lanes by bucket (ballots and scalar
    // reads only: with a lane exchange in the loop 7.1 us on 640 triangles, now 5.6),
    // then one lane per group reserves the group's ranks with a single atomic, all groups at
    // once.  The order inside a bucket is arbitrary.
    uint64_t todo = __ballot(active);
    uint64_t group = 0;
    while (todo) {
      const int leader = __ffsll((unsigned long long)todo) - 1;
      const uint32_t b = (uint32_t)__builtin_amdgcn_readlane((int)bk, leader);
      const uint64_t m = __ballot(active && bk == b) & todo;
      if ((m >> lane) & 1ull) group = m;
      todo &= ~m;
    }
    const int my_leader = active ? __ffsll((unsigned long long)group) - 1 : lane;
    int32_t gbase = 0;
    if (active && my_leader == lane) gbase = atomicAdd(&hist[bk], (int32_t)__popcll(group));
    gbase = __shfl(gbase, my_leader);
    if (active) rank[t] = gbase + (int32_t)__popcll(group & ((1ull << lane) - 1ull));
  }
}

// counting-sort scatter: triangle t goes to offset[bucket] + rank; then every bucket count is
// cleared for the next call
__global__ void __launch_bounds__(kBpBlock) k_scatter(int64_t nt, int64_t nbuckets, const uint32_t* __restrict__ bucket,
                                                      const int32_t* __restrict__ rank,
                                                      const int32_t* __restrict__ offset, int32_t* __restrict__ ids,
                                                      int32_t* __restrict__ hist) {
  const int64_t n = nt > nbuckets ? nt : nbuckets;
  for (int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; t < n; t += (int64_t)gridDim.x * blockDim.x) {
    if (t < nt) ids[offset[bucket[t]] + rank[t]] = (int32_t)t;
    if (t < nbuckets) hist[t] = 0;
  }
}

// Level geometry of the implicit 4-ary tree: m[l] = ceil(n / 4^l) nodes at level l, stored
// from off[l]; node (l, k) covers leaves [k 4^l, (k+1) 4^l) and its children are
// (l-1, 4k .. 4k+3), contiguous in memory; level L (m[L] = 1) is the root.
struct Levels {
  int L;
  int64_t m[24];
  int64_t off[24];
};

// FP32 node box, padded to two 16-byte halves.  The padding of lo holds, for an inner node, the
// bits of an int32: a vertex id that every triangle of the node's subtree holds, or kNoCommon
// (kEmpty for a node with no leaves, the identity of the merge).  A query that holds that
// vertex shares it with every leaf below, so none of them can be its candidate (Sec. 1: pairs
// with a shared vertex are adjacent), and a group of queries that all hold it skips the subtree:
// the boxes of a fan of thin triangles around one vertex all overlap.
struct Box32 {
  float lo[4];
  float hi[4];
};
constexpr int32_t kNoCommon = -1;
constexpr int32_t kEmpty = -2;

__device__ __forceinline__ int32_t box_common(const Box32& b) { return __float_as_int(b.lo[3]); }
__device__ __forceinline__ void set_common(Box32& b, int32_t v) { b.lo[3] = __int_as_float(v); }
__device__ __forceinline__ int32_t merge_common(int32_t a, int32_t b) {
  return a == kEmpty ? b : (b == kEmpty ? a : (a == b ? a : kNoCommon));
}
// what a sorted leaf holds besides its FP32 box: the triangle's vertex ids and its index
struct __align__(16) LeafIds {
  int32_t v[3];
  int32_t tri;
};
static_assert(sizeof(LeafIds) == kLeafBytes, "as the workspace is laid out");

__device__ __forceinline__ Box32 box_union(const Box32& a, const Box32& b) {
  Box32 r;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    r.lo[c] = fminf(a.lo[c], b.lo[c]);
    r.hi[c] = fmaxf(a.hi[c], b.hi[c]);
  }
  set_common(r, merge_common(box_common(a), box_common(b)));
  r.hi[3] = 0.0f;
  return r;
}

// The box of the lanes that the pattern pairs, united (every lane of the wave must call)
template <int kCtrl>
__device__ __forceinline__ Box32 box_union_dpp(const Box32& a) {
  Box32 b;
#pragma unroll
  for (int c = 0; c < 3; ++c) {
    b.lo[c] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a.lo[c]), kCtrl, 0xf, 0xf, true));
    b.hi[c] = __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(a.hi[c]), kCtrl, 0xf, 0xf, true));
  }
  set_common(b, __builtin_amdgcn_mov_dpp(box_common(a), kCtrl, 0xf, 0xf, true));
  return box_union(a, b);
}
// of a quad of lanes, a row of 16 from its quads', the wave from its rows', in every lane
__device__ __forceinline__ Box32 quad_union(const Box32& a) { return box_union_dpp<0x4e>(box_union_dpp<0xb1>(a)); }
__device__ __forceinline__ Box32 row_union(const Box32& a) { return box_union_dpp<0x128>(box_union_dpp<0x124>(a)); }
__device__ __forceinline__ Box32 wave_union(Box32 a) {
#pragma unroll
  for (int d = 16; d < 64; d <<= 1) {
    Box32 b;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      b.lo[c] = __shfl_xor(a.lo[c], d);
      b.hi[c] = __shfl_xor(a.hi[c], d);
    }
    set_common(b, __shfl_xor(box_common(a), d));
    a = box_union(a, b);
  }
  return a;
}

// The shared vertex of the up to four triangles of a quad of lanes (x = kEmpty: no triangle, in
// the last lanes): the first vertex of the first that every present one holds.
__device__ __forceinline__ int32_t common_of_quad(const int3& t) {
  const int32_t f[3] = {__builtin_amdgcn_mov_dpp(t.x, 0, 0xf, 0xf, true), __builtin_amdgcn_mov_dpp(t.y, 0, 0xf, 0xf, true),
                        __builtin_amdgcn_mov_dpp(t.z, 0, 0xf, 0xf, true)};
  int held = 0;
#pragma unroll
  for (int u = 0; u < 3; ++u) held |= (int)(t.x == kEmpty || t.x == f[u] || t.y == f[u] || t.z == f[u]) << u;
  held &= __builtin_amdgcn_mov_dpp(held, 0xb1, 0xf, 0xf, true);
  held &= __builtin_amdgcn_mov_dpp(held, 0x4e, 0xf, 0xf, true);
  if (f[0] == kEmpty) return kEmpty;
  return held & 1 ? f[0] : held & 2 ? f[1] : held & 4 ? f[2] : kNoCommon;
}

// Reduces levels l0+1 .. l0+4 (256 threads) or l0+1 .. l0+5 (1024 threads) from the boxes of
// level l0 (l0 = 0: made from the sorted leaves, which are written too).  Block b owns level-l0
// nodes [kThreads b, kThreads (b + 1)).  A wave makes three levels in registers, the block's first
// wave the last one or two from the waves' boxes.  Bound by the gathers of the leaf pass: 177 us
// for 4,194,304 leaves (186 with every level through LDS and two barriers); 7.6 us for 130,050.
// For a batch (tri_off != NULL) the leaf pass also writes qend[k]: the end of the sorted range of
// the problem owning leaf k (problem p + 1 starts at the offset of its first bucket).
template <int kThreads>
__global__ void __launch_bounds__(kThreads) k_levels(int l0, Levels lv, const double* __restrict__ tbox,
                                                     const int32_t* __restrict__ ids,
                                                     const int32_t* __restrict__ tris, Box32* __restrict__ boxes,
                                                     LeafIds* __restrict__ leaves, const int64_t* __restrict__ tri_off,
                                                     int n_prob, int mbits, const int32_t* __restrict__ offset,
                                                     int32_t* __restrict__ qend) {
  __shared__ Box32 sh[kThreads / 64];
  const int64_t k = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  Box32 bx;
  for (int c = 0; c < 3; ++c) {
    bx.lo[c] = 3.0e38f;
    bx.hi[c] = -3.0e38f;
  }
  set_common(bx, kEmpty);
  bx.hi[3] = 0.0f;
  int3 tv = make_int3(kEmpty, kEmpty, kEmpty);
  if (k < lv.m[l0]) {
    if (l0 == 0) {
      const int32_t t = ids[k];
      LeafIds r;
      for (int c = 0; c < 3; ++c) {
        bx.lo[c] = __double2float_rd(tbox[6 * (int64_t)t + c]);
        bx.hi[c] = __double2float_ru(tbox[6 * (int64_t)t + 3 + c]);
        r.v[c] = tris[3 * (int64_t)t + c];
      }
      r.tri = t;
      // a leaf with a negative id (reported as an index error) shares nothing
      tv = (r.v[0] < 0 || r.v[1] < 0 || r.v[2] < 0) ? make_int3(kNoCommon, kNoCommon, kNoCommon)
                                                   : make_int3(r.v[0], r.v[1], r.v[2]);
      set_common(bx, kNoCommon);  // a leaf box's padding is not read
      leaves[k] = r;
      if (tri_off) {
        const int p = problem_of(tri_off, n_prob, t);
        qend[k] = p + 1 < n_prob ? offset[(int64_t)(p + 1) << mbits] : (int32_t)lv.m[0];
      }
      boxes[lv.off[0] + k] = bx;
    } else {
      bx = boxes[lv.off[l0] + k];
    }
  }
  constexpr int kLevels = kThreads == 256 ? 4 : 5;
  static_assert(kThreads == 1 << (2 * kLevels), "a block reduces kThreads nodes to one");
  const int lane = __lane_id();
  // level l0 + j, of which this lane's node is the k >> 2j-th, one lane of each node writing
  const auto put = [&](int j, const Box32& r, int64_t node, bool writes) {
    if (writes && l0 + j <= lv.L && node < lv.m[l0 + j]) boxes[lv.off[l0 + j] + node] = r;
  };
  Box32 r = quad_union(bx);
  if (l0 == 0) set_common(r, common_of_quad(tv));  // level 1: the vertex its triangles share
  put(1, r, k >> 2, (lane & 3) == 0);
  if (l0 + 2 > lv.L) return;  // (the whole grid)
  r = row_union(r);
  put(2, r, k >> 4, (lane & 15) == 0);
  if (l0 + 3 > lv.L) return;
  r = wave_union(r);
  put(3, r, k >> 6, lane == 0);
  if (l0 + 4 > lv.L) return;
  if (lane == 0) sh[threadIdx.x / 64] = r;
  __syncthreads();
  if (threadIdx.x >= 64) return;
  constexpr int kN = kThreads / 64;  // 4 or 16 boxes left
  r = quad_union(sh[lane < kN ? lane : kN - 1]);
  put(4, r, (int64_t)blockIdx.x * (kN / 4) + lane / 4, lane < kN && (lane & 3) == 0);
  if constexpr (kLevels == 5) {
    r = row_union(r);
    put(5, r, blockIdx.x, lane == 0);
  }
}

__device__ __forceinline__ void wave_lds_sync() {
  __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// number of set bits of m below this lane
__device__ __forceinline__ int rank_below(uint64_t m) {
  return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// inclusive prefix sum over the wave's lanes (row shifts, then the rows' last lanes broadcast)
__device__ __forceinline__ int wave_incl_sum(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
  return v;
}

// Per-wave LDS staging of emitted pairs.  Each step every lane of the wave offers at most one
// pair; positions come from a ballot and the lanes below (mbcnt), so the staging needs no
// atomics.  Only a flush -- when the wave's buffer is nearly full, and once at the end --
// reserves global space, with one atomic for the whole buffer.
constexpr int kEmitCap = 128;  // of the hash kernels' waves

// Where emitted pairs go: the pair array, its capacity, the caller's pair count (the
// reservation counter itself, zeroed at the start of the broad phase) and the status word.
struct PairSink {
  int32_t* pairs;
  int64_t cap;
  unsigned long long* count;
  int32_t* status;
};

// reserves n slots; past the capacity the count still grows and TTIE_ERR_CAPACITY is latched
__device__ __forceinline__ int64_t sink_reserve(const PairSink& o, uint32_t n) {
  const int64_t base = (int64_t)atomicAdd(o.count, (unsigned long long)n);
  if (base + n > o.cap) atomicCAS(o.status, 0, STATUS_CAPACITY);
  return base;
}

template <int kCap>
struct WaveEmitter {
  int2* buf;       // this wave's kCap slots in LDS
  int count;       // wave-uniform fill level

  __device__ __forceinline__ void flush(const PairSink& o) {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    const int lane = __lane_id();
    int64_t base = 0;
    if (lane == 0) base = sink_reserve(o, (uint32_t)count);
    base = __shfl(base, 0);
    for (int i = lane; i < count; i += 64) {
      const int64_t slot = base + i;
      if (slot < o.cap) reinterpret_cast<int2*>(o.pairs)[slot] = buf[i];
    }
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
    count = 0;
  }

  __device__ __forceinline__ void push(bool want, int32_t a, int32_t b, const PairSink& o) {
    const uint64_t mask = __ballot(want);
    if (!mask) return;
    if (want) {
      const int lane = __lane_id();
      buf[count + __popcll(mask & ((1ull << lane) - 1ull))] = make_int2(min(a, b), max(a, b));
    }
    count += __popcll(mask);
    if (count > kCap - 64) flush(o);
  }
};

// End of an emitting kernel: one atomic reserves the space of all the block's waves (every
// thread of the block must arrive here).
template <int kWaves, int kCap>
__device__ __forceinline__ void block_flush(WaveEmitter<kCap>& em, int* wcount, int64_t* bbase, const PairSink& o) {
  const int wave = threadIdx.x / 64;
  if (__lane_id() == 0) wcount[wave] = em.count;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int w = 0; w < kWaves; ++w) tot += wcount[w];
    *bbase = tot ? sink_reserve(o, tot) : 0;
  }
  __syncthreads();
  int64_t base = *bbase;
  for (int w = 0; w < wave; ++w) base += wcount[w];
  for (int i = __lane_id(); i < em.count; i += 64) {
    const int64_t slot = base + i;
    if (slot < o.cap) reinterpret_cast<int2*>(o.pairs)[slot] = em.buf[i];
  }
}

// ---- the traversal: one wave per group of 64 consecutive leaves ---------------------------
// Group g holds the leaves [64 g, 64 g + 64) (a level-3 node), which lie close together in
// Morton order, so one search of the tree serves all of them: the wave pops up to 16 nodes from
// a stack in LDS, four lanes each load one child's box and test it against the group's box,
// overlapping inner children go back on the stack, overlapping leaves to a candidate list.
// Every 64 candidates are then tested against the 64 queries, a candidate per lane, the queries
// broadcast one after the other; the pairs whose boxes overlap are listed candidate by
// candidate, and 64 of these at a time take the exact closed box test and the shared-vertex
// test and are emitted.  On the noisy spheres a group visits about 100 nodes, meets about 120
// candidates besides its own leaves and keeps about 750 of their 11,000 combinations.
//
// Bound by instruction issue (on a 4,194,304-triangle sphere of 16.3 M candidates 3,860 VALU
// instructions a group, 60% of the issue peak) and the latency of the node loads.  With a depth-first search per leaf, whose waves lasted
// as long as their slowest lane's chain of dependent visits, the two kernels took 4.05 ms on a
// 4,194,304-triangle sphere of 20.8 M candidates, now 0.97 ms; 0.98 and 0.28 ms on a
// 1,048,576-triangle sphere of 4.6 M, 97 and 56 us on a 130,050-triangle cloth.  (Persistent waves,
// two tree levels a step and 32 nodes a step measured no faster, in more registers.)
//
// The candidate test runs on 10, 10 and 9 bit integers: a monotone map of the coordinates on
// the group's box, the same for queries and candidates, so boxes that overlap keep overlapping.
// The three high ends are packed in one word, with an empty guard bit above each field, and the
// three low ends in another, each as the guard's value less the end: the sum of the two has a
// guard bit set iff that high end is not below that low end, so two additions and one and
// decide the six comparisons of a pair.
//
// A pair is reported from the group of its first leaf: candidates are leaves after the group,
// and within the group those after the query.  A node whose triangles all hold the vertex that
// all the group's triangles hold is skipped (every pair of the two is adjacent): a fan of thin
// triangles around a pole would otherwise be tested all against all.
constexpr int kGroup = 64;
constexpr int kGroupLevel = 3;       // 4^3 = 64 leaves
constexpr int kTravWaves = 4;
constexpr int kTravThreads = 64 * kTravWaves;
constexpr int kTravMinWaves = 5;     // waves per SIMD that its registers are held to (4: 9% slower, 6: as fast)
constexpr int kEmitTrav = 512;       // a wave's pair buffer
constexpr int kSurv = 512;           // a wave's list of overlapping pairs
constexpr int kStack = 256;
// 16 nodes are popped while the stack holds at most kStackWide entries, one above that: a
// 16-node step leaves at most kStackWide + 48, and depth-first steps of one node add at most 3
// per level to it, 48 in all.
constexpr int kStackWide = kStack - 48 - 48;
constexpr uint32_t kGuard = (1u << 10) | (1u << 21) | (1u << 31);
// The budget (a launch parameter, 128 by default) counts three units for a step of 16 nodes and
// for 64 pairs tested, about 40 steps in all, where a usual group takes 20: candidates are
// handed over from there on, 64 in a batch.  Nodes are handed over after 3/8 of the budget in
// steps, which few groups reach, since a part that starts from one node repeats the group's
// setup for few candidates.
// Measured, broad phase of the 4,194,304-triangle sphere at 64, 96, 128, 192: 1.38, 1.25, 1.23,
// 1.22 ms; of the 1,048,576-triangle one: 0.40, 0.39, 0.41, 0.43 ms.
// With few groups -- all resident at once, or nearly: 5,120 waves are -- the kernel lasts as long as its
// slowest wave while most of the chip is idle, so there the default is half (a caller's budget is
// taken as it is): 1.14 to 1.9 times shorter broad phases, with the parts below, on batches of 36,000
// and 126,000 triangles and spheres of 63,000 and 370,000; on cloths of 130,000 and 149,000, whose
// groups are alike, 93 us instead of 96 and 93 instead of 90; on one of 1,207,458 292 instead of 278.
constexpr int64_t kTravFew = 1 << 19;  // triangles up to which the default budget is half
// The second kernel takes each batch in four parts while what was handed over does not fill its
// grid's waves: at most half as many nodes as waves (a node is a search of its own, which the parts
// before it would delay) and twice as many batches.  Broad phase with whole batches and with four
// parts, us (nodes, batches): spheres of 65,536 to 2,096,704 triangles 136 and 125 (16, 293), 199
// and 179 (470, 1595), 397 and 374 (350, 1850), 515 and 494 (339, 2942), 706 and 693 (1204, 5727);
// of 4,194,304 1164 and 1168 (3022, 10,088); heaps and mixed sizes 220 and 244 (2242, 678), 172 and
// 181 (3753, 1842), 163 and 170 (4643, 1769); batches of 6, 20 and 64 problems 122 and 112 (1144,
// 582), 194 and 201 (3381, 2503), 1195 and 1204 (7230, 3470).
__device__ __forceinline__ int trav_parts(int64_t nodes, int64_t batches, int64_t waves) {
  return 2 * nodes <= waves && batches <= 2 * waves ? 4 : 1;
}
// Queries overlapping one candidate from which adjacency is tested before the pairs are listed:
// 64 more comparisons a batch, which pay where nearly the whole group shares a vertex with it.
constexpr int kDense = 48;

// What a wave over its budget hands to k_traverse_heavy: the nodes still to be searched (as 1
// followed by two bits per level for the path from the root), and batches of 64 candidates
// still to be tested.  A few groups of a mesh have hundreds of times the usual work -- those
// of a dense fold or a fan, and those at a jump of the Morton curve -- and would each hold a
// wave long after the others are done.
struct TravNode {
  int32_t group;
  uint32_t node;
};
struct __align__(16) TravBatch {
  int32_t group, count, pad[2];
  int32_t leaf[64];
};
static_assert(sizeof(TravNode) == kTravNodeBytes && sizeof(TravBatch) == kTravBatchBytes, "as the workspace is laid out");
struct TravHeavy {
  TravNode* nodes;
  TravBatch* batches;
  uint32_t node_cap, batch_cap;
};
struct TravWave {
  uint32_t stack[kStack];
  int32_t cleaf[128];    // candidate leaves
  uint16_t surv[kSurv];  // overlapping pairs: candidate << 6 | query
};

// The wave's staged pairs.  All pairs of a wave of k_traverse hold one of its 64 queries, so a
// pair is staged as the query's lane and the other triangle, 5 bytes; a wave of k_traverse_heavy
// goes from group to group and stages both triangles.
struct GroupEmitter {
  struct Buffer {
    int32_t tri[kEmitTrav];
    uint8_t query[kEmitTrav];
  };
  Buffer* buf;
  int32_t qtri;  // the lane's query triangle
  int count;
  __device__ __forceinline__ void put(int at, int j, int32_t ta, int32_t tb) {
    buf->tri[at] = tb;
    buf->query[at] = (uint8_t)j;
  }
  // the pairs to pairs[base ...) (every lane calls)
  __device__ __forceinline__ void store(int64_t base, const PairSink& o) {
    for (int i0 = 0; i0 < count; i0 += 64) {
      const int i = min(i0 + __lane_id(), count - 1);
      const int32_t b = buf->tri[i], a = __shfl(qtri, buf->query[i]);
      const int64_t slot = base + i;
      if (i0 + __lane_id() < count && slot < o.cap) reinterpret_cast<int2*>(o.pairs)[slot] = make_int2(min(a, b), max(a, b));
    }
  }
};
struct PairEmitter {
  struct Buffer {
    int2 pair[kEmitTrav];
  };
  Buffer* buf;
  int32_t qtri;
  int count;
  __device__ __forceinline__ void put(int at, int, int32_t ta, int32_t tb) { buf->pair[at] = make_int2(min(ta, tb), max(ta, tb)); }
  __device__ __forceinline__ void store(int64_t base, const PairSink& o) {
    for (int i = __lane_id(); i < count; i += 64)
      if (base + i < o.cap) reinterpret_cast<int2*>(o.pairs)[base + i] = buf->pair[i];
  }
};

template <class Emitter>
__device__ __forceinline__ void emit(Emitter& em, bool want, int j, int32_t ta, int32_t tb, const PairSink& o) {
  const uint64_t m = __ballot(want);
  if (!m) return;
  if (want) em.put(em.count + rank_below(m), j, ta, tb);
  em.count += __popcll(m);
  if (em.count > kEmitTrav - 64) {
    wave_lds_sync();
    int64_t base = 0;
    if (__lane_id() == 0) base = sink_reserve(o, (uint32_t)em.count);
    em.store(__shfl(base, 0), o);
    wave_lds_sync();
    em.count = 0;
  }
}

template <class Emitter>
struct TravShared {
  TravWave w[kTravWaves];
  typename Emitter::Buffer stage[kTravWaves];
  int32_t lm[24];
  uint32_t loff[24];  // the level table
  int wcount[kTravWaves];
  int64_t bbase;
};

// The monotone map of one group's coordinates to small integers.  An axis on which the group
// has no extent to speak of, or an unbounded one, maps to 0 throughout, so nothing is rejected
// on it.
struct TravMap {
  float lo[3], scale[3];
  __device__ __forceinline__ void set(const Box32& b) {
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const float e = b.hi[c] - b.lo[c];
      const bool ok = e >= 1.0e-30f && e <= 3.0e38f;
      lo[c] = ok ? b.lo[c] : 0.0f;
      scale[c] = ok ? (c < 2 ? 1023.0f : 511.0f) / e : 0.0f;
    }
  }
  __device__ __forceinline__ uint32_t one(float v, int c) const {
    const float top = c < 2 ? 1023.0f : 511.0f;
    const float q = scale[c] > 0.0f ? (v - lo[c]) * scale[c] : 0.0f;
    return (uint32_t)fminf(fmaxf(q, 0.0f), top);
  }
  __device__ __forceinline__ uint32_t hi_word(const Box32& b) const {
    return one(b.hi[0], 0) | one(b.hi[1], 1) << 11 | one(b.hi[2], 2) << 22;
  }
  __device__ __forceinline__ uint32_t lo_word(const Box32& b) const {
    return kGuard - (one(b.lo[0], 0) | one(b.lo[1], 1) << 11 | one(b.lo[2], 2) << 22);
  }
};

__device__ __forceinline__ float size2(const Box32& b) {
  const float e = (b.hi[0] - b.lo[0]) + (b.hi[1] - b.lo[1]) + (b.hi[2] - b.lo[2]);
  return e * e;
}

// Half the margin by which two FP32 boxes must overlap for the FP64 boxes to overlap for
// certain: each end was rounded outwards by less than 2^-23 of itself (or 2^-149).  NaN, so
// that nothing is certain, for a box with an end that is huge or not finite.
__device__ __forceinline__ float box_margin(const Box32& b) {
  const float m = fabsf(b.lo[0]) + fabsf(b.hi[0]) + fabsf(b.lo[1]) + fabsf(b.hi[1]) + fabsf(b.lo[2]) + fabsf(b.hi[2]);
  return m < 1.0e30f ? 2.5e-7f * m + 1.0e-37f : __builtin_nanf("");
}

// The query word of lane (i - r) & 15 of the row, as the operand of an addition.
template <int r>
__device__ __forceinline__ uint32_t add_rotated(uint32_t q, uint32_t c) {
  return (uint32_t)__builtin_amdgcn_mov_dpp(q, r ? 0x120 + r : 0xe4, 0xf, 0xf, true) + c;
}
template <int r>
__device__ __forceinline__ uint32_t one_test(uint32_t qlo, uint32_t qhi, uint32_t clo, uint32_t chi) {
  return add_rotated<r>(qlo, chi) & add_rotated<r>(qhi, clo) & kGuard;
}
// The tests of a lane's candidate against the 16 queries of a row, their verdicts shifted into
// bits.  Four at a time: the comparisons' results are the carries of four additions, each read
// at least two instructions after it is written.
template <int r = 0>
__device__ __forceinline__ void row_tests(uint32_t& bits, uint32_t qlo, uint32_t qhi, uint32_t clo, uint32_t chi) {
  const uint32_t t0 = one_test<r>(qlo, qhi, clo, chi), t1 = one_test<r + 1>(qlo, qhi, clo, chi),
                 t2 = one_test<r + 2>(qlo, qhi, clo, chi), t3 = one_test<r + 3>(qlo, qhi, clo, chi);
  uint64_t c0, c1, c2, c3;
  asm("v_cmp_eq_u32 %1, %5, %6\n\t"
      "v_cmp_eq_u32 %2, %5, %7\n\t"
      "v_cmp_eq_u32 %3, %5, %8\n\t"
      "v_cmp_eq_u32 %4, %5, %9\n\t"
      "v_addc_co_u32 %0, %1, %0, %0, %1\n\t"
      "v_addc_co_u32 %0, %2, %0, %0, %2\n\t"
      "v_addc_co_u32 %0, %3, %0, %0, %3\n\t"
      "v_addc_co_u32 %0, %4, %0, %0, %4"
      : "+&v"(bits), "=&s"(c0), "=&s"(c1), "=&s"(c2), "=&s"(c3)
      : "s"(kGuard), "v"(t0), "v"(t1), "v"(t2), "v"(t3));
  if constexpr (r < 12) row_tests<r + 4>(bits, qlo, qhi, clo, chi);
}

// kVA: pairs sharing exactly one vertex are candidates; kBatch: the leaves are of several
// problems, whose ends qend holds (template arguments, so the default keeps the plain tests and its
// registers).  kHeavy: the rest of a search handed over by another wave: from the node `start`, or
// the tests of `most` candidates of `batch` from `first` on.
template <bool kVA, bool kBatch, bool kHeavy, class Emitter>
__device__ __forceinline__ void search_group(TravWave& sh, const int32_t* lm, const uint32_t* loff, int32_t n, int L,
                                             int32_t g, uint32_t start, const TravBatch* batch, int first, int most,
                                             const Box32* __restrict__ boxes,
                                             const LeafIds* __restrict__ leaves, const double* __restrict__ tbox,
                                             const int32_t* __restrict__ qend, const TravHeavy& heavy, int budget,
                                             Emitter& em, const PairSink& sink,
                                             Counters* ctr) {
  const int lane = __lane_id();
  const int32_t s0 = g * kGroup;
  const int nq = min(kGroup, n - s0);
  // the group's box and the queries' (lanes past the last leaf repeat it, and are masked out)
  const Box32 gb = L >= kGroupLevel ? boxes[loff[kGroupLevel] + (uint32_t)g] : boxes[loff[L]];
  const int32_t gcom = kVA ? kNoCommon : box_common(gb);
  const Box32 qb = boxes[(uint32_t)s0 + min(lane, nq - 1)];
  const LeafIds ql = leaves[s0 + min(lane, nq - 1)];
  TravMap map;
  map.set(gb);
  // (a lane past the last leaf gets a low word that sets no guard)
  const uint32_t qlo = lane < nq ? map.lo_word(qb) : 0u, qhi = map.hi_word(qb);
  em.qtri = ql.tri;
  const float qeps = box_margin(qb);
  // leaves up to the end of the problem of the group's last leaf
  const int32_t last = kBatch ? qend[s0 + nq - 1] : n;
  int nc = 0;          // candidates (uniform)
  int work = 0, steps = 0;  // steps of 16 nodes and of 64 pairs, three units each; steps of 16 nodes

  // The queries that a lane's box (clo, chi) overlaps, as bits.  The queries of row R (16 lanes)
  // come to the lanes of row R ^ v by one exchange, and to every lane of the row by 16 rotations,
  // which the additions take as their operand's lane pattern: at (v, r), bit
  // 31 - (16 (v & 1) + r) of word v >> 1, lane 16 R + i meets query 16 (R ^ v) + ((i - r) & 15).
  const int row = lane >> 4, li = lane & 15;
  const auto overlaps = [&](uint32_t clo, uint32_t chi, uint32_t (&m)[2]) {
    m[0] = m[1] = 0u;
#pragma unroll
    for (int v = 0; v < 4; ++v) {
      const uint32_t vlo = v ? __shfl_xor(qlo, 16 * v) : qlo, vhi = v ? __shfl_xor(qhi, 16 * v) : qhi;
      row_tests(m[v >> 1], vlo, vhi, clo, chi);
    }
  };
  // tests cnt <= 64 candidates, a lane each (box cb, ids cl, packed box clo, chi), against the
  // queries; own: the candidates are the queries, each paired with those before it
  const auto settle = [&](int cnt, bool own, int32_t leaf, const Box32& cb, const LeafIds& cl, uint32_t clo,
                          uint32_t chi) {
    // in a group over the end of a problem a candidate's queries are those from the first one, f, of
    // its own problem on (a batch of 1000 problems of 8 triangles in one place: 44 us, and 82 where
    // all the group's overlaps were listed and tested one by one)
    int f = 0;
    if (kBatch && qend[s0] != last) {
      const int32_t qe = qend[s0 + min(lane, nq - 1)];
#pragma unroll
      for (int b = 32; b > 0; b >>= 1) f += __shfl(qe, f + b - 1) <= leaf ? b : 0;
    }
    uint32_t m[2];
    overlaps(clo, chi, m);
    // lanes past the last candidate, and a query's own leaf and those before it, do not count
    if (lane >= cnt) m[0] = m[1] = 0u;
    if (own) {
      const auto before = [&](int v) { return (row ^ v) < row ? 0xffffu : 0u; };
      // in the own row, ((i - r) & 15) < i iff 1 <= r <= i
      m[0] &= (0x7fffu & ~(0x7fffu >> li)) << 16 | before(1);
      m[1] &= before(2) << 16 | before(3);
    }
    if (kBatch && f > 0) {
      // (the row's queries q from f on, as bit (15 - li + q) & 15: turned right by 1 + li)
      const auto from = [&](int v) {
        const uint32_t tail = (0xffffu << min(max(f - 16 * (row ^ v), 0), 16)) & 0xffffu;
        return (tail * 0x10001u >> (1 + li)) & 0xffffu;
      };
      m[0] &= from(0) << 16 | from(1);
      m[1] &= from(2) << 16 | from(3);
    }
    int p = __popc(m[0]) + __popc(m[1]);
    if (!kVA && __ballot(p >= kDense)) {
      // many queries at once (a fan, a fold): most of them share a vertex with the candidate
#pragma unroll 4
      for (int j = 0; j < 64; ++j) {
        const int32_t v[3] = {__builtin_amdgcn_readlane(ql.v[0], j), __builtin_amdgcn_readlane(ql.v[1], j),
                              __builtin_amdgcn_readlane(ql.v[2], j)};
        const int jv = (j >> 4) ^ row;
        const uint32_t clear = is_adjacent(v, cl.v, false) ? 0x80000000u >> (16 * (jv & 1) + ((li - j) & 15)) : 0u;
        if (jv < 2) m[0] &= ~clear;
        else m[1] &= ~clear;
      }
      p = __popc(m[0]) + __popc(m[1]);
    }
    const float ceps = box_margin(cb);
    // the pairs go through the list kSurv at a time, candidate by candidate
    const int incl = wave_incl_sum(p);
    const int total = __builtin_amdgcn_readlane(incl, 63);
    int at = incl - p;
    for (int w0 = 0; w0 < total; w0 += kSurv) {
      const int stop = min(incl, w0 + kSurv), ns = min(total - w0, kSurv);
      while (at < stop) {
        const int w = m[0] ? 0 : 1;
        const int b = __builtin_clz(w ? m[1] : m[0]);
        const uint32_t bit = 0x80000000u >> b;
        if (w) m[1] ^= bit;
        else m[0] ^= bit;
        const int j = ((row ^ (2 * w + (b >> 4))) << 4) | ((li - b) & 15);
        sh.surv[at - w0] = (uint16_t)(lane << 6 | j);
        ++at;
      }
      wave_lds_sync();
      work += 3 * ((ns + 63) >> 6);
      for (int b0 = 0; b0 < ns; b0 += 64) {
        bool want = b0 + lane < ns;
        const int it = want ? sh.surv[b0 + lane] : 0;
        const int k = it >> 6, j = it & 63;
        float d = __shfl(cb.hi[0], k) - __shfl(qb.lo[0], j);
        d = fminf(d, __shfl(qb.hi[0], j) - __shfl(cb.lo[0], k));
        d = fminf(d, __shfl(cb.hi[1], k) - __shfl(qb.lo[1], j));
        d = fminf(d, __shfl(qb.hi[1], j) - __shfl(cb.lo[1], k));
        d = fminf(d, __shfl(cb.hi[2], k) - __shfl(qb.lo[2], j));
        d = fminf(d, __shfl(qb.hi[2], j) - __shfl(cb.lo[2], k));
        const float eps = __shfl(ceps, k) + __shfl(qeps, j);
        const int32_t av[3] = {__shfl(ql.v[0], j), __shfl(ql.v[1], j), __shfl(ql.v[2], j)};
        const int32_t bv[3] = {__shfl(cl.v[0], k), __shfl(cl.v[1], k), __shfl(cl.v[2], k)};
        const int32_t ta = __shfl(ql.tri, j), tb = __shfl(cl.tri, k);
        want = want && !(d < 0.0f) && !is_adjacent(av, bv, kVA);
        if (want && !(d >= eps)) {
          // within the rounding of the FP32 boxes: the FP64 ones decide
          const double* A = tbox + 6 * (int64_t)ta;
          const double* B = tbox + 6 * (int64_t)tb;
#pragma unroll
          for (int c = 0; c < 3; ++c) want = want & (A[c] <= B[3 + c]) & (B[c] <= A[3 + c]);
        }
        emit(em, want, j, ta, tb, sink);
      }
      wave_lds_sync();  // the list is written again
    }
  };
  // A group is loosely packed when its box is much larger than what its quads of leaves (or,
  // of a quad that is itself loose, its leaves) cover: at a jump of the Morton curve, or around
  // one large triangle.  Its search then tests the queries' boxes too, so that it does not meet
  // everything between them.
  bool loose = false;
  if (!kHeavy || !batch) {
    const float s1 = lane < nq ? size2(qb) : 0.0f;
    Box32 quad = qb;
    float s4 = s1;
#pragma unroll
    for (int d = 1; d < 4; d <<= 1) {
#pragma unroll
      for (int c = 0; c < 3; ++c) {
        quad.lo[c] = fminf(quad.lo[c], __shfl_xor(quad.lo[c], d));
        quad.hi[c] = fmaxf(quad.hi[c], __shfl_xor(quad.hi[c], d));
      }
      s4 += __shfl_xor(s4, d);
    }
    const float sq = size2(quad);
    float tot = sq > 4.0f * s4 ? s1 : ((lane & 3) == 0 && lane < nq ? sq : 0.0f);
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) tot += __shfl_xor(tot, d);
    loose = size2(gb) > 4.0f * tot;
  }
  const auto meets = [](const Box32& a, const Box32& b) {
    return (a.lo[0] <= b.hi[0]) & (b.lo[0] <= a.hi[0]) & (a.lo[1] <= b.hi[1]) & (b.lo[1] <= a.hi[1]) &
           (a.lo[2] <= b.hi[2]) & (b.lo[2] <= a.hi[2]);
  };
  // whether node (l, c) can hold a candidate
  Box32 b{};
  const auto meets_group = [&](int l, int32_t c) {
    b = boxes[loff[l] + (uint32_t)c];
    bool ov = meets(gb, b) && !(gcom >= 0 && l > 0 && box_common(b) == gcom);
    return ov;
  };
  // the first node of level l that may hold leaves after the group
  const auto first_node = [&](int l) {
    return l > kGroupLevel ? g >> (2 * (l - kGroupLevel)) : (g + 1) << (2 * (kGroupLevel - l));
  };

  int sp = 0;
  if (kHeavy) {
    if (batch) {
      nc = max(0, min(batch->count - first, most));  // (none in a part past the last one)
      if (lane < nc) sh.cleaf[lane] = batch->leaf[first + lane];
    } else {
      if (lane == 0) sh.stack[0] = start;
      sp = 1;
    }
  } else {
    // start at the lowest level of at most 64 nodes, a lane each
    int ls = L;
    while (ls > 0 && lm[ls - 1] <= 64) --ls;
    if (ls > 0) {
      const bool ov = lane < lm[ls] && lane >= first_node(ls) && lane <= (last - 1) >> (2 * ls) && meets_group(ls, lane);
      const uint64_t m = __ballot(ov);
      if (ov) sh.stack[rank_below(m)] = (1u << (2 * (L - ls))) + (uint32_t)lane;
      sp = __popcll(m);
    }
  }
  wave_lds_sync();
  bool may_defer = !kHeavy;
  // the group's own leaves are the first candidates, then those the search finds, 64 at a time
  for (bool own = !kHeavy;; own = false) {
    while (!own && nc < 64 && sp > 0) {
      if (may_defer && steps > 3 * budget / 8) {
        // the nodes still to be searched, as far as the list has room
        uint32_t base = 0;
        if (lane == 0) base = atomicAdd(&ctr->n_heavy, (uint32_t)sp);
        base = __shfl(base, 0);
        const int fit = base < heavy.node_cap ? (int)min((uint32_t)sp, heavy.node_cap - base) : 0;
        for (int i = lane; i < fit; i += 64) heavy.nodes[base + i] = TravNode{g, sh.stack[sp - 1 - i]};
        sp -= fit;
        may_defer = false;
        if (sp == 0) break;
      }
      work += 3;
      ++steps;
      const int take = sp <= kStackWide ? min(sp, 16) : 1;
      const int t = lane >> 2;
      const bool act = t < take;
      const uint32_t code = act ? sh.stack[sp - 1 - t] : 1u;
      sp -= take;
      wave_lds_sync();
      const int depth = (31 - __builtin_clz(code)) >> 1;
      const int lc = max(L - depth - 1, 0);
      const int32_t c = (int32_t)(4u * (code - (1u << (2 * depth))) + (uint32_t)(lane & 3));
      bool ov = act && c >= first_node(lc) && c <= (last - 1) >> (2 * lc) && c < lm[lc] && meets_group(lc, c);
      if (loose && __ballot(ov)) {
        uint32_t m[2];
        overlaps(map.lo_word(b), map.hi_word(b), m);
        ov = ov && (m[0] | m[1]);
      }
      const uint64_t inner = __ballot(ov && lc > 0), leaf = __ballot(ov && lc == 0);
      if (ov && lc > 0) sh.stack[sp + rank_below(inner)] = 4u * code + (uint32_t)(lane & 3);
      sp += __popcll(inner);
      if (ov && lc == 0) sh.cleaf[nc + rank_below(leaf)] = c;
      nc += __popcll(leaf);
      wave_lds_sync();
    }
    const int cnt = own ? nq : min(nc, 64);
    if (cnt == 0) break;
    bool handed = false;
    if (!kHeavy && !own && work > budget) {  // over the budget: left to another wave, if the list has room
      uint32_t at = 0;
      if (lane == 0) at = atomicAdd(&ctr->n_batches, 1u);
      at = __shfl(at, 0);
      if (at < heavy.batch_cap) {
        if (lane == 0) {
          heavy.batches[at].group = g;
          heavy.batches[at].count = cnt;
        }
        if (lane < cnt) heavy.batches[at].leaf[lane] = sh.cleaf[lane];
        handed = true;
      }
    }
    if (!handed) {
      const int32_t leaf = own ? s0 + min(lane, nq - 1) : sh.cleaf[lane < cnt ? lane : 0];
      const Box32 cb = boxes[(uint32_t)leaf];
      const LeafIds cl = leaves[leaf];
      settle(cnt, own, leaf, cb, cl, map.lo_word(cb), map.hi_word(cb));
    }
    if (!own) {  // the rest of the list moves to its start
      nc -= cnt;
      const int32_t rest = sh.cleaf[64 + lane];
      wave_lds_sync();
      if (lane < nc) sh.cleaf[lane] = rest;
      wave_lds_sync();
    }
  }
}

template <class Shared>
__device__ __forceinline__ void level_table(Shared& sh, const Levels& lv) {
  if (threadIdx.x < 24) {
    sh.lm[threadIdx.x] = (int32_t)lv.m[threadIdx.x];
    sh.loff[threadIdx.x] = (uint32_t)lv.off[threadIdx.x];
  }
  __syncthreads();
}

// End of a block: one atomic reserves the space of all its waves.
template <class Emitter, class Shared>
__device__ __forceinline__ void end_emit(Emitter& em, Shared& sh, const PairSink& o) {
  const int wave = threadIdx.x / 64;
  if (__lane_id() == 0) sh.wcount[wave] = em.count;
  __syncthreads();
  if (threadIdx.x == 0) {
    uint32_t tot = 0;
    for (int w = 0; w < kTravWaves; ++w) tot += sh.wcount[w];
    sh.bbase = tot ? sink_reserve(o, tot) : 0;
  }
  __syncthreads();
  int64_t base = sh.bbase;
  for (int w = 0; w < wave; ++w) base += sh.wcount[w];
  em.store(base, o);
}

template <bool kVA, bool kBatch>
__global__ void __launch_bounds__(kTravThreads, kTravMinWaves) k_traverse(int64_t n64, Levels lv, const Box32* __restrict__ boxes,
                                                           const LeafIds* __restrict__ leaves,
                                                           const double* __restrict__ tbox,
                                                           const int32_t* __restrict__ qend, TravHeavy heavy, int budget,
                                                           int32_t* pairs, int64_t cap, unsigned long long* npairs,
                                                           Counters* ctr) {
  __shared__ TravShared<GroupEmitter> sh;
  const PairSink sink{pairs, cap, npairs, &ctr->status};
  level_table(sh, lv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  const int64_t g = xcd_block(blockIdx.x, gridDim.x) * kTravWaves + wave;
  GroupEmitter em{&sh.stage[wave], 0, 0};
  if (g * kGroup < n64)
    search_group<kVA, kBatch, false>(sh.w[wave], sh.lm, sh.loff, (int32_t)n64, lv.L, (int32_t)g, 0u, nullptr, 0, 0, boxes,
                             leaves, tbox, qend, heavy, budget, em, sink, ctr);
  end_emit(em, sh, sink);
}

// What the waves over their budget handed over, a wave per batch, part of a batch or node.
template <bool kVA, bool kBatch>
__global__ void __launch_bounds__(kTravThreads, kTravMinWaves) k_traverse_heavy(int64_t n64, Levels lv, const Box32* __restrict__ boxes,
                                                                 const LeafIds* __restrict__ leaves,
                                                                 const double* __restrict__ tbox,
                                                                 const int32_t* __restrict__ qend, TravHeavy heavy,
                                                                 int32_t* pairs, int64_t cap,
                                                                 unsigned long long* npairs, Counters* ctr) {
  __shared__ TravShared<PairEmitter> sh;
  const PairSink sink{pairs, cap, npairs, &ctr->status};
  const int64_t batches = min(ctr->n_batches, heavy.batch_cap), nn = min(ctr->n_heavy, heavy.node_cap);
  const int parts = trav_parts(nn, batches, (int64_t)gridDim.x * kTravWaves);
  const int most = 64 / parts;  // candidates of a batch that a wave takes
  const int64_t nb = parts * batches;
  if ((int64_t)blockIdx.x * kTravWaves >= nb + nn) return;  // (the whole block)
  level_table(sh, lv);
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x / 64);
  PairEmitter em{&sh.stage[wave], 0, 0};
  for (int64_t i = (int64_t)blockIdx.x * kTravWaves + wave; i < nb + nn; i += (int64_t)gridDim.x * kTravWaves) {
    const TravBatch* batch = i < nb ? heavy.batches + i / parts : nullptr;
    const TravNode node = i < nb ? TravNode{batch->group, 0u} : heavy.nodes[i - nb];
    search_group<kVA, kBatch, true>(sh.w[wave], sh.lm, sh.loff, (int32_t)n64, lv.L, node.group, node.node, batch,
                            (int)(i % parts) * most, most, boxes, leaves, tbox, qend, heavy, 0, em, sink, ctr);
  }
  end_emit(em, sh, sink);
}

// All i < j without a shared vertex.  A block takes kBruteRows rows i and kBpBlock columns j,
// keeps each thread's (column's) verdicts as bits, and reserves the space of all of them with
// one atomic.  The pairs come by the million; with a reservation for every 128 of them the
// atomics on the one counter, about 20 ns each, were the whole cost (3,260,220 pairs: 632 us, now
// 27 us, of which the 26 MB of stores are 5).
constexpr int kBruteRows = 16;

__global__ void __launch_bounds__(kBpBlock) k_brute(const int32_t* __restrict__ tris, int64_t nt, int32_t* pairs,
                                                    int64_t cap, unsigned long long* npairs, int va, Counters* ctr) {
  const PairSink sink{pairs, cap, npairs, &ctr->status};
  __shared__ int wtot[kBpBlock / 64];
  __shared__ int64_t sbase;
  const int lane = __lane_id(), wave = threadIdx.x / 64;
  const int64_t jtiles = (nt + kBpBlock - 1) / kBpBlock, itiles = (nt + kBruteRows - 1) / kBruteRows;
  for (int64_t tile = blockIdx.x; tile < itiles * jtiles; tile += gridDim.x) {
    const int64_t i0 = tile / jtiles * kBruteRows, jb = tile % jtiles * kBpBlock;
    if (jb + kBpBlock <= i0 + 1) continue;  // no j > i here
    const int64_t j = jb + threadIdx.x;
    uint32_t bits = 0;
    if (j < nt) {
      const int32_t vj[3] = {tris[3 * j], tris[3 * j + 1], tris[3 * j + 2]};
      const int rows = (int)min((int64_t)kBruteRows, min(nt - i0, j - i0));
      for (int r = 0; r < rows; ++r) {
        const int32_t* ti = tris + 3 * (i0 + r);
        const int32_t vi[3] = {ti[0], ti[1], ti[2]};
        bits |= (uint32_t)!is_adjacent(vi, vj, va) << r;
      }
    }
    int tot = 0;
#pragma unroll
    for (int r = 0; r < kBruteRows; ++r) tot += __popcll(__ballot((bits >> r) & 1u));
    if (lane == 0) wtot[wave] = tot;
    __syncthreads();
    if (threadIdx.x == 0) {
      int all = 0;
      for (int w = 0; w < kBpBlock / 64; ++w) all += wtot[w];
      sbase = all ? sink_reserve(sink, (uint32_t)all) : 0;
    }
    __syncthreads();
    int64_t at = sbase;
    for (int w = 0; w < wave; ++w) at += wtot[w];
#pragma unroll
    for (int r = 0; r < kBruteRows; ++r) {
      const bool want = (bits >> r) & 1u;
      const uint64_t m = __ballot(want);
      const int64_t slot = at + rank_below(m);
      if (want && slot < cap) reinterpret_cast<int2*>(pairs)[slot] = make_int2((int32_t)(i0 + r), (int32_t)j);
      at += __popcll(m);
    }
    __syncthreads();  // wtot and sbase are used again
  }
}

// ---- spatial hashing (the broad phase of Sec. 1.2) -----------------------------------------
// A uniform grid of cell size h (twice the mean largest box extent) anchored at the lowest box
// centre.  Every triangle is entered in each cell its FP64 box covers; entries are counting-
// sorted by a hash of the cell (MurmurHash3's 64-bit finalizer), and a thread per entry tests
// the later entries of its bucket that name the same cell.  A pair is reported only from its
// reference cell -- the componentwise maximum of the two boxes' lowest cells, which both boxes
// cover exactly when they overlap -- so each overlapping pair is found once, and the result is
// the same canonical set as the LBVH's.
//
//   k_hash_cells    grid parameters (every block reduces the box partials the same way), cell
//                   ranges, entries reserved per wave with one atomic, bucket ranks
//   scan            bucket offsets
//   k_hash_scatter  entries to their sorted places; bucket counts cleared for the next call
//   k_hash_pairs    same-cell tests within buckets, exact box and shared-vertex tests, emission
constexpr int kCellBits = 21;             // signed cell coordinates packed into 63 bits
constexpr int64_t kCellLimit = 1 << 20;   // |cell index| bound

struct HashGrid {
  double org[3];
  double h;
};

__device__ __forceinline__ int64_t cell_of(double v, double org, double h) { return (int64_t)floor((v - org) / h); }

__device__ __forceinline__ uint64_t cell_key(int64_t cx, int64_t cy, int64_t cz) {
  const uint64_t m = (1ull << kCellBits) - 1;
  return (((uint64_t)cx & m) << (2 * kCellBits)) | (((uint64_t)cy & m) << kCellBits) | ((uint64_t)cz & m);
}

__device__ __forceinline__ uint32_t hash_bucket(uint64_t k, int bits) {
  k ^= k >> 33;
  k *= 0xff51afd7ed558ccdull;
  k ^= k >> 33;
  k *= 0xc4ceb9fe1a85ec53ull;
  k ^= k >> 33;
  return (uint32_t)(k >> (64 - bits));
}

__global__ void __launch_bounds__(kBpBlock) k_hash_cells(const double* __restrict__ tbox, int64_t nt,
                                                         const uint32_t* __restrict__ part,
                                                         const double* __restrict__ ext_part, int nparts, int hbits,
                                                         int32_t* __restrict__ hist, uint64_t* __restrict__ key,
                                                         int32_t* __restrict__ tri, int32_t* __restrict__ rank,
                                                         int64_t ecap, HashGrid* grid, Counters* ctr) {
  __shared__ uint32_t red[6][kBpBlock];
  __shared__ double rext[kBpBlock];
  __shared__ HashGrid sg;
  uint32_t v[6] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0u, 0u, 0u};
  double e = 0.0;
  for (int b = threadIdx.x; b < nparts; b += kBpBlock) {
    for (int c = 0; c < 6; ++c) v[c] = c < 3 ? min(v[c], part[6 * b + c]) : max(v[c], part[6 * b + c]);
    e += ext_part[b];
  }
  for (int c = 0; c < 6; ++c) red[c][threadIdx.x] = v[c];
  rext[threadIdx.x] = e;
  __syncthreads();
  for (int w = kBpBlock / 2; w > 0; w >>= 1) {
    if (threadIdx.x < w) {
      for (int c = 0; c < 6; ++c)
        red[c][threadIdx.x] = c < 3 ? min(red[c][threadIdx.x], red[c][threadIdx.x + w])
                                    : max(red[c][threadIdx.x], red[c][threadIdx.x + w]);
      rext[threadIdx.x] += rext[threadIdx.x + w];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    double span = 0.0;
    for (int c = 0; c < 3; ++c) {
      sg.org[c] = (double)key2f(red[c][0]);
      span = fmax(span, (double)key2f(red[3 + c][0]) - sg.org[c]);
    }
    double h = 2.0 * rext[0] / (double)nt;
    // keep the cell indices of the scene far inside the packed range
    const double hmin = span / (double)(kCellLimit / 4);
    if (!(h > hmin)) h = hmin;
    if (!(h > 0.0) || !(h < 1.0e300)) h = 1.0;
    sg.h = h;
    if (blockIdx.x == 0) *grid = sg;
  }
  __syncthreads();
  const HashGrid g = sg;
  int status = 0;
  const int lane = __lane_id();
  for (int64_t base = (int64_t)blockIdx.x * kBpBlock; base < nt; base += (int64_t)gridDim.x * kBpBlock) {
    const int64_t t = base + threadIdx.x;
    int64_t lo[3] = {0, 0, 0}, hi[3] = {-1, -1, -1};
    uint32_t n = 0;
    if (t < nt) {
      bool ok = true;
      for (int c = 0; c < 3; ++c) {
        lo[c] = cell_of(tbox[6 * t + c], g.org[c], g.h);
        hi[c] = cell_of(tbox[6 * t + 3 + c], g.org[c], g.h);
        ok = ok && lo[c] > -kCellLimit && hi[c] < kCellLimit && hi[c] >= lo[c] && hi[c] - lo[c] < 1024;
      }
      if (ok) {
        const int64_t cnt = (hi[0] - lo[0] + 1) * (hi[1] - lo[1] + 1) * (hi[2] - lo[2] + 1);
        if (cnt <= (1 << 20)) n = (uint32_t)cnt;
        else ok = false;
      }
      if (!ok) status = STATUS_UNSUPPORTED;  // a box far outside the grid or over a million cells
    }
    // wave prefix sum of the entry counts, one atomic per wave
    uint32_t incl = n;
    for (int d = 1; d < 64; d <<= 1) {
      const uint32_t y = __shfl_up(incl, d);
      if (lane >= d) incl += y;
    }
    const uint32_t total = __shfl(incl, 63);
    uint64_t wbase = 0;
    if (lane == 63 && total) wbase = atomicAdd(reinterpret_cast<unsigned long long*>(&ctr->n_entries), (unsigned long long)total);
    wbase = __shfl(wbase, 63);
    int64_t slot = (int64_t)wbase + incl - n;
    for (int64_t cx = lo[0]; cx <= hi[0] && n; ++cx)
      for (int64_t cy = lo[1]; cy <= hi[1]; ++cy)
        for (int64_t cz = lo[2]; cz <= hi[2]; ++cz, ++slot) {
          if (slot >= ecap) {
            status = STATUS_CAPACITY;
            continue;
          }
          const uint64_t k = cell_key(cx, cy, cz);
          key[slot] = k;
          tri[slot] = (int32_t)t;
          rank[slot] = atomicAdd(&hist[hash_bucket(k, hbits)], 1);
        }
  }
  if (status) atomicCAS(&ctr->status, 0, status);
}

__global__ void __launch_bounds__(kBpBlock) k_hash_scatter(const Counters* ctr, int64_t ecap, int64_t nbuckets, int hbits,
                                                           const uint64_t* __restrict__ key,
                                                           const int32_t* __restrict__ tri,
                                                           const int32_t* __restrict__ rank,
                                                           const int32_t* __restrict__ offset,
                                                           uint64_t* __restrict__ skey, int32_t* __restrict__ stri,
                                                           int32_t* __restrict__ hist) {
  const int64_t ne = min((int64_t)ctr->n_entries, ecap);
  const int64_t n = ne > nbuckets ? ne : nbuckets;
  for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n; e += (int64_t)gridDim.x * blockDim.x) {
    if (e < ne) {
      const uint64_t k = key[e];
      const int64_t pos = (int64_t)offset[hash_bucket(k, hbits)] + rank[e];
      skey[pos] = k;
      stri[pos] = tri[e];
    }
    if (e < nbuckets) hist[e] = 0;
  }
}

// one entry's view of its bucket: its triangle's FP64 box, lowest cell and vertices
struct HashQuery {
  uint64_t key;
  int32_t tri;
  int64_t end;  // end of the bucket in sorted order
  double lo[3], hi[3];
  int64_t cell[3];
  int32_t v[3];
};

__device__ __forceinline__ HashQuery hash_query(int64_t e, int64_t ne, int64_t nbuckets, int hbits,
                                                const int32_t* __restrict__ offset, const uint64_t* __restrict__ skey,
                                                const int32_t* __restrict__ stri, const double* __restrict__ tbox,
                                                const int32_t* __restrict__ tris, const HashGrid& g) {
  HashQuery h;
  h.key = skey[e];
  h.tri = stri[e];
  const uint32_t b = hash_bucket(h.key, hbits);
  h.end = (int64_t)b + 1 < nbuckets ? offset[b + 1] : ne;
  for (int c = 0; c < 3; ++c) {
    h.lo[c] = tbox[6 * (int64_t)h.tri + c];
    h.hi[c] = tbox[6 * (int64_t)h.tri + 3 + c];
    h.cell[c] = cell_of(h.lo[c], g.org[c], g.h);
    h.v[c] = tris[3 * (int64_t)h.tri + c];
  }
  return h;
}

// entry j of the same bucket: a candidate iff it names the same cell, the closed FP64 boxes
// overlap, this cell is the pair's reference cell, and no vertex is shared
__device__ __forceinline__ bool hash_test(const HashQuery& h, int64_t j, const uint64_t* __restrict__ skey,
                                          const int32_t* __restrict__ stri, const double* __restrict__ tbox,
                                          const int32_t* __restrict__ tris, const HashGrid& g, bool va,
                                          int32_t& other) {
  if (skey[j] != h.key) return false;
  other = stri[j];
  bool hit = true;
  int64_t ref[3];
  for (int c = 0; c < 3; ++c) {
    const double blo = tbox[6 * (int64_t)other + c], bhi = tbox[6 * (int64_t)other + 3 + c];
    hit = hit && h.lo[c] <= bhi && blo <= h.hi[c];
    const int64_t bc = cell_of(blo, g.org[c], g.h);
    ref[c] = h.cell[c] > bc ? h.cell[c] : bc;
  }
  if (!hit || cell_key(ref[0], ref[1], ref[2]) != h.key) return false;
  const int32_t vo[3] = {tris[3 * (int64_t)other], tris[3 * (int64_t)other + 1], tris[3 * (int64_t)other + 2]};
  return !is_adjacent(h.v, vo, va);
}

// A thread tests at most `hbudget` (a launch parameter, 64 by default) later entries of its
// bucket; the rest of a longer bucket
// (the cells where many triangles meet, e.g. the fan around a pole) goes to k_hash_heavy, where
// a whole wave shares it.

__global__ void __launch_bounds__(kBpBlock) k_hash_pairs(const Counters* ctr, int64_t ecap, int64_t nbuckets, int hbits,
                                                         const int32_t* __restrict__ offset,
                                                         const uint64_t* __restrict__ skey,
                                                         const int32_t* __restrict__ stri,
                                                         const double* __restrict__ tbox,
                                                         const int32_t* __restrict__ tris, const HashGrid* grid,
                                                         int hbudget, int va, int32_t* __restrict__ heavy,
                                                         int32_t* pairs,
                                                         int64_t cap,
                                                         unsigned long long* npairs, Counters* out_ctr) {
  const PairSink sink{pairs, cap, npairs, &out_ctr->status};
  __shared__ int2 stage[kBpBlock / 64][kEmitCap];
  __shared__ int wcount[kBpBlock / 64];
  __shared__ int64_t bbase;
  WaveEmitter<kEmitCap> em{stage[threadIdx.x / 64], 0};
  const int64_t ne = min((int64_t)ctr->n_entries, ecap);
  const HashGrid g = *grid;
  for (int64_t base = (int64_t)blockIdx.x * kBpBlock; base < ne; base += (int64_t)gridDim.x * kBpBlock) {
    const int64_t e = base + threadIdx.x;
    const bool active = e < ne;
    HashQuery h;
    int64_t stop = 0;
    if (active) {
      h = hash_query(e, ne, nbuckets, hbits, offset, skey, stri, tbox, tris, g);
      stop = min(h.end, e + 1 + hbudget);
    }
    const bool defer = active && h.end > stop;
    const uint32_t slot = wave_slot(defer, &out_ctr->n_heavy);
    if (defer) heavy[slot] = (int32_t)e;  // slot < ne <= ecap
    // the loop runs while any lane has work, so the emitter always sees the whole wave
    for (int64_t j = e + 1; __ballot(active && j < stop); ++j) {
      int32_t other = 0;
      const bool want = active && j < stop && hash_test(h, j, skey, stri, tbox, tris, g, va, other);
      em.push(want, h.tri, other, sink);
    }
  }
  block_flush<kBpBlock / 64>(em, wcount, &bbase, sink);
}

// one wave per deferred entry: its lanes stride over the rest of the bucket
__global__ void __launch_bounds__(kBpBlock) k_hash_heavy(const Counters* ctr, int64_t ecap, int64_t nbuckets, int hbits,
                                                         const int32_t* __restrict__ offset,
                                                         const uint64_t* __restrict__ skey,
                                                         const int32_t* __restrict__ stri,
                                                         const double* __restrict__ tbox,
                                                         const int32_t* __restrict__ tris, const HashGrid* grid,
                                                         int hbudget, int va, const int32_t* __restrict__ heavy,
                                                         int32_t* pairs,
                                                         int64_t cap, unsigned long long* npairs, Counters* out_ctr) {
  const PairSink sink{pairs, cap, npairs, &out_ctr->status};
  __shared__ int2 stage[kBpBlock / 64][kEmitCap];
  __shared__ int wcount[kBpBlock / 64];
  __shared__ int64_t bbase;
  WaveEmitter<kEmitCap> em{stage[threadIdx.x / 64], 0};
  const int64_t ne = min((int64_t)ctr->n_entries, ecap);
  const int64_t nh = min((int64_t)ctr->n_heavy, ne);
  const HashGrid g = *grid;
  const int waves = gridDim.x * (kBpBlock / 64);
  for (int64_t it = (int64_t)blockIdx.x * (kBpBlock / 64) + threadIdx.x / 64; it < nh; it += waves) {
    const int64_t e = heavy[it];
    const HashQuery h = hash_query(e, ne, nbuckets, hbits, offset, skey, stri, tbox, tris, g);
    for (int64_t jb = e + 1 + hbudget; jb < h.end; jb += 64) {
      const int64_t j = jb + __lane_id();
      int32_t other = 0;
      const bool want = j < h.end && hash_test(h, j, skey, stri, tbox, tris, g, va, other);
      em.push(want, h.tri, other, sink);
    }
  }
  block_flush<kBpBlock / 64>(em, wcount, &bbase, sink);
}



static unsigned bp_grid(int64_t n, unsigned cap = 4096) {
  int64_t g = (n + kBpBlock - 1) / kBpBlock;
  if (g < 1) g = 1;
  if (g > cap) g = cap;
  return (unsigned)g;
}

// Every level is stored padded to a multiple of 4 nodes, so a node's four children are one aligned
// 128-byte line (the padding is neither written nor read: the search tests c < m[l] first).
static int64_t pad4(int64_t m) { return (m + 3) & ~(int64_t)3; }

Levels make_levels(int64_t n) {
  Levels lv{};
  int64_t off = 0, m = n;
  int l = 0;
  for (;; ++l) {
    lv.m[l] = m;
    lv.off[l] = off;
    off += pad4(m);
    if (m <= 1) break;
    m = (m + 3) / 4;
  }
  lv.L = l;
  return lv;
}

hipError_t launch_broadphase(Ctx* c, const ttie_mesh* m, int method, const double* x_end, int n_prob,
                             const int64_t* tri_off, int32_t* pairs, int64_t capacity, int64_t* n_pairs, hipStream_t s) {
  const Layout& L = c->L;
  Counters* ctr = wsp<Counters>(c, L.counters);
  const int64_t nt = m->n_tris;
  unsigned long long* npairs = reinterpret_cast<unsigned long long*>(n_pairs);
  const int va = (method & TTIE_BROAD_VERTEX_ADJACENT) ? 1 : 0;
  method &= 0xff;
  if (method == TTIE_BROAD_BRUTE || nt < 2) k_bp_init<<<1, 64, 0, s>>>(ctr, npairs);
  if (method == TTIE_BROAD_BRUTE) {
    const int64_t tiles = ((nt + kBpBlock - 1) / kBpBlock) * ((nt + kBruteRows - 1) / kBruteRows);
    stage_begin(c, TTIE_STAGE_BP_TRAVERSE, s);
    k_brute<<<(unsigned)std::max<int64_t>(1, std::min<int64_t>(tiles, 1 << 16)), kBpBlock, 0, s>>>(m->tris, nt, pairs,
                                                                                                   capacity, npairs, va,
                                                                                                   ctr);
    stage_end(c, TTIE_STAGE_BP_TRAVERSE, s);
  } else if (method == TTIE_BROAD_HASH && nt >= 2) {
    double* tbox = wsp<double>(c, L.bvh_tbox);
    const unsigned gb = bp_grid(nt, kBoundsBlocks);
    int hbits = 8;
    while (hbits < kMortonBucketBits && ((int64_t)1 << hbits) < 2 * nt) ++hbits;
    const int64_t nbuckets = (int64_t)1 << hbits;
    const int64_t ecap = (int64_t)kHashEntriesPerTri * c->lim.max_tris;
    int32_t* hist = wsp<int32_t>(c, L.bvh_hist);
    int32_t* offset = wsp<int32_t>(c, L.bvh_offset);
    uint64_t* key = wsp<uint64_t>(c, L.hash_key);
    int32_t* tri = wsp<int32_t>(c, L.hash_tri);
    uint64_t* skey = wsp<uint64_t>(c, L.hash_skey);
    int32_t* stri = wsp<int32_t>(c, L.hash_stri);
    HashGrid* grid = wsp<HashGrid>(c, L.hash_grid);
    stage_begin(c, TTIE_STAGE_BP_BOXES, s);
    k_tri_boxes<<<gb, kBpBlock, 0, s>>>(m->x, x_end, m->n_verts, m->tris, nt, tbox, wsp<float>(c, L.bvh_centroid),
                                        wsp<uint32_t>(c, L.bvh_part), wsp<double>(c, L.bvh_ext), npairs, ctr);
    k_hash_cells<<<bp_grid(nt), kBpBlock, 0, s>>>(tbox, nt, wsp<uint32_t>(c, L.bvh_part), wsp<double>(c, L.bvh_ext),
                                                  (int)gb, hbits, hist, key, tri, wsp<int32_t>(c, L.hash_rank), ecap,
                                                  grid, ctr);
    stage_end(c, TTIE_STAGE_BP_BOXES, s);
    stage_begin(c, TTIE_STAGE_BP_SORT, s);
    hipError_t e = launch_scan_i32(c, hist, offset, nbuckets, s);
    if (e != hipSuccess) return e;
    k_hash_scatter<<<bp_grid(std::max<int64_t>(4 * nt, nbuckets)), kBpBlock, 0, s>>>(
        ctr, ecap, nbuckets, hbits, key, tri, wsp<int32_t>(c, L.hash_rank), offset, skey, stri, hist);
    stage_end(c, TTIE_STAGE_BP_SORT, s);
    stage_begin(c, TTIE_STAGE_BP_TRAVERSE, s);
    int32_t* heavy = wsp<int32_t>(c, L.hash_rank);  // the ranks are consumed by the scatter
    const int hb = (int)ctx_param(c, TTIE_PARAM_HASH_BUDGET);
    k_hash_pairs<<<bp_grid(4 * nt, 8192), kBpBlock, 0, s>>>(ctr, ecap, nbuckets, hbits, offset, skey, stri, tbox,
                                                           m->tris, grid, hb, va, heavy, pairs, capacity, npairs, ctr);
    stage_end(c, TTIE_STAGE_BP_TRAVERSE, s);
    stage_begin(c, TTIE_STAGE_BP_HEAVY, s);
    k_hash_heavy<<<512, kBpBlock, 0, s>>>(ctr, ecap, nbuckets, hbits, offset, skey, stri, tbox, m->tris, grid, hb, va,
                                          heavy, pairs, capacity, npairs, ctr);
    stage_end(c, TTIE_STAGE_BP_HEAVY, s);
  } else if (method == TTIE_BROAD_LBVH && nt >= 2) {
    double* tbox = wsp<double>(c, L.bvh_tbox);
    float* centre = wsp<float>(c, L.bvh_centroid);
    uint32_t* k1 = wsp<uint32_t>(c, L.bvh_keys);
    int32_t* v1 = wsp<int32_t>(c, L.bvh_vals);
    int32_t* v2 = wsp<int32_t>(c, L.bvh_vals2);
    Box32* boxes = wsp<Box32>(c, L.bvh_boxes);
    LeafIds* leaves = wsp<LeafIds>(c, L.bvh_leaves);
    int32_t* qend = wsp<int32_t>(c, L.bvh_qend);
    const Levels lv = make_levels(nt);
    stage_begin(c, TTIE_STAGE_BP_BOXES, s);
    const unsigned gb = bp_grid(nt, kBoundsBlocks);
    // buckets: about two triangles per bucket; a batch spends the top bits on the problem
    int bits = 8;
    while (bits < kMortonBucketBits && ((int64_t)1 << (bits + 1)) <= nt) ++bits;
    int pbits = 0;
    if (!tri_off) n_prob = 1;
    while ((1 << pbits) < n_prob) ++pbits;
    const int mbits = std::min(std::max(bits - pbits, 3), kMortonBucketBits - pbits);
    const int64_t nbuckets = (int64_t)1 << (pbits + mbits);
    int32_t* hist = wsp<int32_t>(c, L.bvh_hist);
    int32_t* offset = wsp<int32_t>(c, L.bvh_offset);
    k_tri_boxes<<<gb, kBpBlock, 0, s>>>(m->x, x_end, m->n_verts, m->tris, nt, tbox, wsp<float>(c, L.bvh_centroid),
                                        wsp<uint32_t>(c, L.bvh_part), wsp<double>(c, L.bvh_ext), npairs, ctr);
    k_morton<<<bp_grid(nt), kBpBlock, 0, s>>>(centre, nt, wsp<uint32_t>(c, L.bvh_part), (int)gb, tri_off, n_prob,
                                              mbits, hist, k1, v1, ctr);
    stage_end(c, TTIE_STAGE_BP_BOXES, s);
    stage_begin(c, TTIE_STAGE_BP_SORT, s);
    hipError_t e = launch_scan_i32(c, hist, offset, nbuckets, s);
    if (e != hipSuccess) return e;
    k_scatter<<<bp_grid(std::max<int64_t>(nt, nbuckets)), kBpBlock, 0, s>>>(nt, nbuckets, k1, v1, offset, v2, hist);
    stage_end(c, TTIE_STAGE_BP_SORT, s);
    stage_begin(c, TTIE_STAGE_BP_BUILD, s);
    // leaves to level 4 in blocks of 256, then five levels per launch in blocks of 1024 (a
    // tree of up to 4^9 leaves takes two launches)
    for (int l0 = 0; l0 < lv.L; l0 += l0 == 0 ? 4 : 5) {
      if (l0 == 0)
        k_levels<256><<<(unsigned)((lv.m[0] + 255) / 256), 256, 0, s>>>(0, lv, tbox, v2, m->tris, boxes, leaves,
                                                                         tri_off, n_prob, mbits, offset, qend);
      else
        k_levels<1024><<<(unsigned)((lv.m[l0] + 1023) / 1024), 1024, 0, s>>>(l0, lv, tbox, v2, m->tris, boxes, leaves,
                                                                             tri_off, n_prob, mbits, offset, qend);
    }
    stage_end(c, TTIE_STAGE_BP_BUILD, s);
    stage_begin(c, TTIE_STAGE_BP_TRAVERSE, s);
    // a wave per 64 leaves, block count rounded up to a multiple of the 8 XCDs
    const int64_t per = kGroup * kTravWaves;
    const int64_t nb = ((nt + per - 1) / per + 7) / 8 * 8;
    const TravHeavy heavy{wsp<TravNode>(c, L.trav_nodes), wsp<TravBatch>(c, L.trav_batches), L.trav_node_cap,
                          L.trav_batch_cap};
    const bool own = c->param[TTIE_PARAM_TRAV_BUDGET] != 0;  // set by the caller
    const int budget = (int)ctx_param(c, TTIE_PARAM_TRAV_BUDGET) / (nt <= kTravFew && !own ? 2 : 1);
    // (the batch's broad phase has no vertex-adjacent option)
    const auto traverse = tri_off ? k_traverse<false, true> : va ? k_traverse<true, false> : k_traverse<false, false>;
    const auto traverse_heavy =
        tri_off ? k_traverse_heavy<false, true> : va ? k_traverse_heavy<true, false> : k_traverse_heavy<false, false>;
    traverse<<<(unsigned)nb, kTravThreads, 0, s>>>(nt, lv, boxes, leaves, tbox, qend, heavy,
                                                   budget, pairs, capacity, npairs, ctr);
    stage_end(c, TTIE_STAGE_BP_TRAVERSE, s);
    stage_begin(c, TTIE_STAGE_BP_HEAVY, s);
    traverse_heavy<<<1024, kTravThreads, 0, s>>>(nt, lv, boxes, leaves, tbox, qend, heavy, pairs, capacity, npairs, ctr);
    stage_end(c, TTIE_STAGE_BP_HEAVY, s);
  }
  return hipGetLastError();
}

}  // namespace ttie
