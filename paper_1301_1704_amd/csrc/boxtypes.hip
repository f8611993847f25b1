// Simulated partition and source box types (Section 3).
//
// Partition (Section 3.2): the boxes of the partition level l_par go to the
// ranks in consecutive Morton ranges balanced by receiver points. The
// nonempty receiver box whose first point is the p-th of M (in Morton order;
// p is its bookmark) goes to rank min(R - 1, floor(R p / M)); every other
// Morton index of l_par takes the rank of the nearest nonempty receiver box
// before it (rank 0 if none), so each rank holds one consecutive range.
//
// Box types (Section 3.1, Algorithm 6) for rank J, with l_crit = l_par - 1:
// below l_crit every source box is DOMESTIC. At l_crit a box whose nonempty
// source children (at l_par) are all elsewhere is IMPORT, one with children
// on J and elsewhere is ROOT, and one with all children on J is EXPORT when
// a receiver box with a nonempty receiver child elsewhere has it in its M2L
// list E4, else DOMESTIC. From l_par down a box belongs to the owner of its
// l_par ancestor (its Morton index shifted right, Section 3.2): on J it is
// EXPORT when a receiver box of another rank has it in E4, else DOMESTIC;
// elsewhere it is IMPORT when a receiver box of J has it in E4, else OTHER.
//
// The E4 lists of the build give "r has k in E4(r)" directly, so the marks
// are made by the receivers: a receiver reads its list and marks the source
// boxes it names. A receiver whose whole M2L region lies in l_par boxes of
// its own rank cannot mark anything, nor can a receiver of another rank whose
// region has no box of this rank; only the others are listed and read.
#include "../../include/fmmds.h"
#include "device.h"
#include "internal.h"

namespace fmmds {

constexpr uint32_t kMarkBlocks = 2048;  // per level, 8192 waves walk its work list

// Coordinate of a Morton index on one axis (bits 3b + axis).
__device__ __forceinline__ uint32_t axis_coord(uint64_t key, int axis) {
  return (uint32_t)compact3(key >> axis);
}

template <typename KeyT>
__global__ __launch_bounds__(256) void k_partition(const KeyT* __restrict__ rkey,
                                                   const uint32_t* __restrict__ rbegin,
                                                   uint32_t n_boxes, uint32_t n_points,
                                                   uint32_t n_ranks, uint64_t n_idx,
                                                   uint32_t* __restrict__ owner) {
  for (uint64_t m = blockIdx.x * 256ull + threadIdx.x; m < n_idx; m += gridDim.x * 256ull) {
    uint32_t lo = 0, hi = n_boxes;  // first box with key > m
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if ((uint64_t)rkey[mid] <= m) lo = mid + 1;
      else hi = mid;
    }
    uint32_t o = 0;
    if (lo > 0) {
      const uint64_t p = rbegin[lo - 1];
      o = (uint32_t)min<uint64_t>(n_ranks - 1, (uint64_t)n_ranks * p / n_points);
    }
    owner[m] = o;
  }
}

// Box types, every level in two launches (grid y: the levels from a first one on).
//
// k_types_init: per source box, the type it has if no list names it (DOMESTIC or
// OTHER; at the critical level IMPORT, ROOT or DOMESTIC), and per receiver,
// whether its E4 list has to be read; those receivers go to the level's work
// list, one atomic per block.
// k_types_mark: one wave per listed receiver at a time; the source boxes its list
// names become EXPORT or IMPORT. Every writer of a box stores the same value, so
// plain byte stores do.
//
// Critical level: receivers with a nonempty receiver child on another rank.
// Levels l >= l_par: the M2L region of r is, per axis, the level-l coordinates
// 2(p - 1) .. 2(p + 1) + 1 around its parent coordinate p; their l_par ancestors
// are that range shifted right by l - l_par. Marks need a region with another
// rank than r's, and a receiver of another rank marks only boxes of `rank`, so
// its region must also touch `rank`. The region is the parent's, and below l_par
// so is r's owner: there one thread decides for all children of a parent.
//
// What bounds it: one read of every box's key and the lists near rank borders.
// On the 2 x 2^24 uniform build (13M boxes a side, 64 ranks, l_par = 4), four
// launches per level (marks cleared, receivers picked one by one, marked, types
// written) took 340 us with the partition; these two take 140 us (105 us of kernels).
template <typename KeyT>
__device__ __forceinline__ bool region_picked(const BoxTypes& a, uint64_t kp, uint32_t sh,
                                              uint32_t o_r) {
  const int32_t top = (1 << a.l_par) - 1;
  int32_t lo[3], hi[3];
  for (int d = 0; d < 3; ++d) {
    const int32_t p = (int32_t)axis_coord(kp, d);
    lo[d] = max(0, (2 * (p - 1)) >> sh);
    hi[d] = min(top, (2 * (p + 1) + 1) >> sh);
  }
  bool mixed = false, touches = o_r == a.rank;
  for (int32_t z = lo[2]; z <= hi[2]; ++z)
    for (int32_t y = lo[1]; y <= hi[1]; ++y)
      for (int32_t x = lo[0]; x <= hi[0]; ++x) {
        const uint32_t o = a.owner[spread3((uint32_t)x) | (spread3((uint32_t)y) << 1) |
                                   (spread3((uint32_t)z) << 2)];
        mixed |= o != o_r;
        touches |= o == a.rank;
      }
  return mixed && touches;
}

// The block's picks [first, first + n) of each thread to the level's work list.
__device__ __forceinline__ void append_work(const BoxTypesLevel& v, uint32_t first, uint32_t n) {
  __shared__ uint32_t s_w[5];
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  const uint32_t incl = wave_incl_scan(n);
  __syncthreads();  // (s_w of the round before)
  if (lane == 63) s_w[w] = incl;
  __syncthreads();
  const uint32_t total = s_w[0] + s_w[1] + s_w[2] + s_w[3];
  if (total == 0) return;  // the whole block
  if (threadIdx.x == 0) s_w[4] = atomicAdd(v.n_work, total);
  __syncthreads();
  uint32_t at = s_w[4] + incl - n;
  for (uint32_t i = 0; i < w; ++i) at += s_w[i];
  for (uint32_t i = 0; i < n; ++i) v.work[at + i] = first + i;
}

template <typename KeyT>
__global__ __launch_bounds__(256) void k_types_init(BoxTypes a, uint32_t first) {
  const uint32_t l = first + blockIdx.y;
  const BoxTypesLevel& v = a.lv[l];
  const uint32_t l_crit = a.l_par - 1;
  const uint64_t t0 = blockIdx.x * 256ull + threadIdx.x, step = gridDim.x * 256ull;
  if (l < l_crit) {
    for (uint64_t k = t0; k < v.n_src; k += step) v.types[k] = FMMDS_BOX_DOMESTIC;
    return;
  }
  if (l == l_crit) {
    const KeyT* __restrict__ sk = (const KeyT*)a.lv[a.l_par].skey;
    for (uint64_t k = t0; k < v.n_src; k += step) {
      bool on = false, off = false;
      for (uint32_t c = v.schild[k]; c < v.schild[k + 1]; ++c) {
        const bool here = a.owner[(uint64_t)sk[c]] == a.rank;
        on |= here;
        off |= !here;
      }
      v.types[k] = !on ? FMMDS_BOX_IMPORT : off ? FMMDS_BOX_ROOT : FMMDS_BOX_DOMESTIC;
    }
    const KeyT* __restrict__ rk = (const KeyT*)a.lv[a.l_par].rkey;
    for (uint64_t r0 = blockIdx.x * 256ull; r0 < v.n_recv; r0 += step) {
      const uint64_t r = r0 + threadIdx.x;
      bool pick = false;
      if (r < v.n_recv)
        for (uint32_t c = v.rchild[r]; c < v.rchild[r + 1]; ++c)
          pick |= a.owner[(uint64_t)rk[c]] != a.rank;
      append_work(v, (uint32_t)r, pick ? 1u : 0u);
    }
    return;
  }
  const uint32_t sh = l - a.l_par;
  const KeyT* __restrict__ sk = (const KeyT*)v.skey;
  for (uint64_t k = t0; k < v.n_src; k += step)
    v.types[k] = a.owner[(uint64_t)sk[k] >> (3 * sh)] == a.rank ? FMMDS_BOX_DOMESTIC
                                                                 : FMMDS_BOX_OTHER;
  if (sh == 0) {  // each receiver has its own owner
    const KeyT* __restrict__ rk = (const KeyT*)v.rkey;
    for (uint64_t r0 = blockIdx.x * 256ull; r0 < v.n_recv; r0 += step) {
      const uint64_t r = r0 + threadIdx.x;
      bool pick = false;
      if (r < v.n_recv) {
        const uint64_t kr = (uint64_t)rk[r];
        pick = region_picked<KeyT>(a, kr >> 3, 0, a.owner[kr]);
      }
      append_work(v, (uint32_t)r, pick ? 1u : 0u);
    }
    return;
  }
  const BoxTypesLevel& u = a.lv[l - 1];
  const KeyT* __restrict__ pk = (const KeyT*)u.rkey;
  for (uint64_t p0 = blockIdx.x * 256ull; p0 < u.n_recv; p0 += step) {
    const uint64_t p = p0 + threadIdx.x;
    uint32_t first = 0, n = 0;
    if (p < u.n_recv) {
      const uint64_t kp = (uint64_t)pk[p];
      if (region_picked<KeyT>(a, kp, sh, a.owner[kp >> (3 * (sh - 1))])) {
        first = u.rchild[p];
        n = u.rchild[p + 1] - first;
      }
    }
    append_work(v, first, n);
  }
}

// A listed receiver's E4 entries (at most 189) are read three 64-entry chunks at
// once, every load before any store (on this GPU a wait for a load also waits
// for earlier stores).
template <typename KeyT>
__global__ __launch_bounds__(256) void k_types_mark(BoxTypes a, uint32_t first) {
  const uint32_t l = first + blockIdx.y;
  const BoxTypesLevel& v = a.lv[l];
  const bool deep = l >= a.l_par;
  const uint32_t sh = deep ? l - a.l_par : 0;
  const KeyT* __restrict__ rk = (const KeyT*)v.rkey;
  const KeyT* __restrict__ sk = (const KeyT*)v.skey;
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t n = *v.n_work;
  const uint32_t n_waves = gridDim.x * 4;
  for (uint32_t w = blockIdx.x * 4 + (threadIdx.x >> 6); w < n; w += n_waves) {
    const uint32_t r = v.work[w];
    const uint32_t lo = v.e4_off[r], hi = v.e4_off[r + 1];
    const bool r_here = deep && a.owner[(uint64_t)rk[r] >> (3 * sh)] == a.rank;
    uint32_t k[3];
    bool set[3];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      const uint32_t i = lo + 64u * c + lane;
      k[c] = i < hi ? v.e4_ent[i] : 0xFFFFFFFFu;
    }
#pragma unroll
    for (int c = 0; c < 3; ++c) {
      set[c] = false;
      if (k[c] == 0xFFFFFFFFu) continue;
      if (deep) set[c] = (a.owner[(uint64_t)sk[k[c]] >> (3 * sh)] == a.rank) != r_here;
      else set[c] = v.types[k[c]] == FMMDS_BOX_DOMESTIC;
    }
    // (a deep box on this rank named by a receiver elsewhere: EXPORT; one
    // elsewhere named by a receiver here: IMPORT)
#pragma unroll
    for (int c = 0; c < 3; ++c)
      if (set[c]) v.types[k[c]] = r_here ? FMMDS_BOX_IMPORT : FMMDS_BOX_EXPORT;
  }
}

void launch_partition(bool key64, const void* rkey, const uint32_t* rbegin, uint32_t n_boxes,
                      uint32_t n_points, uint32_t n_ranks, uint32_t l_par, uint32_t* owner,
                      hipStream_t s) {
  const uint64_t n_idx = 1ull << (3 * l_par);
  const uint32_t g = (uint32_t)std::min<uint64_t>((n_idx + 255) / 256, 65536);
  if (key64)
    hipLaunchKernelGGL(k_partition<uint64_t>, dim3(g), dim3(256), 0, s, (const uint64_t*)rkey,
                       rbegin, n_boxes, n_points, n_ranks, n_idx, owner);
  else
    hipLaunchKernelGGL(k_partition<uint32_t>, dim3(g), dim3(256), 0, s, (const uint32_t*)rkey,
                       rbegin, n_boxes, n_points, n_ranks, n_idx, owner);
}

void launch_box_types(bool key64, const BoxTypes& a, uint32_t first, uint32_t last,
                      hipStream_t s) {
  uint64_t most = 1;
  for (uint32_t l = first; l <= last; ++l)
    most = std::max<uint64_t>(most, std::max(a.lv[l].n_src, a.lv[l].n_recv));
  const uint32_t listed = std::max(first, a.l_par - 1);  // no lists are read above
  const dim3 init((uint32_t)std::min<uint64_t>((most + 255) / 256, 8192), last - first + 1);
  const dim3 mark((uint32_t)std::min<uint64_t>((most + 3) / 4, kMarkBlocks),
                  last >= listed ? last - listed + 1 : 0);
  if (key64) hipLaunchKernelGGL(k_types_init<uint64_t>, init, dim3(256), 0, s, a, first);
  else hipLaunchKernelGGL(k_types_init<uint32_t>, init, dim3(256), 0, s, a, first);
  if (mark.y == 0) return;
  if (key64) hipLaunchKernelGGL(k_types_mark<uint64_t>, mark, dim3(256), 0, s, a, listed);
  else hipLaunchKernelGGL(k_types_mark<uint32_t>, mark, dim3(256), 0, s, a, listed);
}

}  // namespace fmmds
