// E2 neighbor lists and E4 (M2L) interaction lists per level.
//
// Definitions (Section 1.4): for a receiver box r at level l, E2(r) holds the
// nonempty source boxes within one box of r in every coordinate (r included);
// E4(r) holds the nonempty source boxes that are children of boxes in
// E2(parent(r)) at level l - 1 but are not in E2(r). The paper enumerates the
// candidate boxes from de-interleaved coordinates (Section 2.3) and looks them
// up in a dense per-box rank array (Algorithm 4).
//
// Here the candidates come from the parent level's E2 list: the children of
// the nonempty source boxes s in E2(parent(r)) are exactly the nonempty
// source boxes of E2(r) and E4(r) together, they sit at consecutive ranks
// child[s] .. child[s] + popcount(mask[s]) - 1 in octant order, and walking
// E2(parent(r)) in ascending rank then the children in octant order yields
// ascending ranks. No search and no dense array are needed. Whether a child
// in octant o of a neighbor at offset (dx, dy, dz) from the parent is within
// one box of r (octant q) is decided per axis:
//   d = 0: always;  d = +1: child bit 0 and r bit 1;  d = -1: child bit 1 and
//   r bit 0;
// giving an 8-bit mask over the child octants.
#include <cstddef>

#include "device.h"
#include "internal.h"

namespace fmmds {

// A box's 16-byte node (device.h) holds what a neighbor needs of it: first
// child, child octant mask, and the two lowest octal digits of its key, which
// give the offset of two boxes at most one apart: per axis the two digits'
// bits, kept in place, subtract to 0, to the axis' lowest bit (+1) or to both
// of its bits (-1).
//
// Counting (level 2, and every level of a build in the least memory; else the
// fill of each level counts the next): one half-wave (32 lanes) per receiver box
// p of level l - 1; lane j takes the j-th entry s of E2(p) (at most 27) and
// counts, for each of the 8 receiver octants q, the children of s adjacent to a
// receiver child in octant q; two packed half-wave scans give the E2 count of
// every receiver child of p at once (E4 = all children minus E2).
//
// Filling: two receiver boxes p per wave, one per half-wave for the setup.
// The children of all s in E2(p), in ascending rank, form one union list U
// (at most 216 boxes), the same for every receiver child of p; the half-wave
// writes U once to LDS together with, per entry, the 8-bit mask of receiver
// octants it is adjacent to. Then the whole wave takes each p in turn: each
// lane keeps its share of U in registers, and for each receiver child the
// wave splits U into the child's E2 and E4 lists with one ballot per 64
// entries: order is kept, so both come out ascending.
// The lists of p's children are consecutive in memory, so the split goes to
// LDS and leaves in 16-byte stores. Measured on the 2 x 2^24-point uniform
// build, finest level (7.7 GB of entries): splitting straight to memory with
// 4-byte stores, with a neighbor's key, mask and first child in three arrays,
// took 2041 us, half of a wave's time in its loads; one node per neighbor and
// staged lists take 1640 us (4.7 TB/s; as many bytes stored the same way from
// registers, by a kernel that does nothing else, 1280 us).
// What bounds it now: the stores share the path to memory with the neighbor
// loads (the loads and the split without the stores take 880 us). Neither
// persistent waves that load ahead (2170 us) nor larger staging buffers and so
// fewer waves (all levels together: 2.19 ms with 8 waves per SIMD, 2.22 with 7,
// 2.46 with 5) overlap them better.
constexpr int kUnion = 220;      // >= 27 * 8 children of E2(p), and a slot for absent octants
constexpr uint32_t kFillE2 = 436;  // LDS words for E2 entries of two parents (<= 2 * 216 + 3)
constexpr uint32_t kFillE4 = 844;  // LDS words for staged E4 entries
constexpr uint32_t kFillWords = kFillE2 + kFillE4;
static_assert(2 * 2 * kUnion + 128 <= kFillWords, "U and the count slots share the staging space");

// Offset of a neighbor from p: low digits of both keys -> per axis 0, 1 or
// (-1) both bits of the axis.
struct Offset {
  uint32_t x, y, z;  // 0, +1: 1 / 2 / 4, -1: 9 / 18 / 36
};
__device__ __forceinline__ Offset node_offset(uint32_t sk, uint32_t pk) {
  return {((sk & 0x09u) - (pk & 0x09u)) & 0x09u, ((sk & 0x12u) - (pk & 0x12u)) & 0x12u,
          ((sk & 0x24u) - (pk & 0x24u)) & 0x24u};
}
// v0, v+ or v- by an axis offset d of node_offset with lowest bit `low`.
__device__ __forceinline__ uint32_t by_offset(uint32_t d, uint32_t low, uint32_t v0, uint32_t vp,
                                              uint32_t vm) {
  const uint32_t v = d == low ? vp : vm;
  return d == 0 ? v0 : v;
}

// E2 count of octant q from the packed words: octants 0..3 sit in bits
// 8 + 6q of word a (bits 0..7 hold the count of all children), 4..7 in bits
// 6(q - 4) of word b.
__device__ __forceinline__ uint32_t octant_field(uint32_t a, uint32_t b, uint32_t q) {
  return q < 4 ? (a >> (8 + 6 * q)) & 63u : (b >> (6 * (q - 4))) & 63u;
}

__device__ __forceinline__ void count_children(const ListLevelArgs& a, uint64_t p, uint32_t j,
                                               uint32_t* __restrict__ cnt2,
                                               uint32_t* __restrict__ cnt4) {
  const uint32_t n_up = a.n_recv_up_dev ? *a.n_recv_up_dev : a.n_recv_up;
  if (p >= n_up) return;  // whole half-wave
  // upbase: batch rank of the set's first box at level - 1 (parent-level E2
  // entries are stored relative to it).
  uint32_t j0, cnt, upbase = 0;
  if (a.up_all) {
    j0 = 0;
    cnt = a.n_src_up_dev ? *a.n_src_up_dev : a.n_src_up;
  } else {
    j0 = a.e2_off_up[p];
    cnt = a.e2_off_up[p + 1] - j0;
  }
  if (a.first_up) {
    const uint32_t set = (uint32_t)(a.recv_key_up[p] >> (3 * (a.level - 1)));
    upbase = a.first_up[set];
    if (a.up_all) cnt = a.first_up[set + 1] - upbase;
    if (a.set_level[set] < a.level) cnt = 0;  // the set's lists stop above this level
  }
  const uint2 np = *(const uint2*)&a.recv_node_up[p];
  const uint32_t rmask = np.y & 0xFFu, rfirst = np.x;
  uint32_t wa = 0, wb = 0;
  if (j < cnt) {
    const uint32_t s = upbase + (a.up_all ? j : a.e2_ent_up[j0 + j]);
    const uint2 ns = *(const uint2*)&a.src_node_up[s];
    const Offset d = node_offset(ns.y >> 8, np.y >> 8);
    const uint32_t m = ns.y & 0xFFu;
    // Children of s adjacent to a receiver child whose axis bit is 0 / 1:
    // offset 0: all; +1: child bit 0 and receiver bit 1; -1: child bit 1 and
    // receiver bit 0. Octants with the x / y / z bit clear: 0x55 / 0x33 / 0x0F.
    const uint32_t ax0 = by_offset(d.x, 1, 0xFFu, 0u, 0xAAu);
    const uint32_t ax1 = by_offset(d.x, 1, 0xFFu, 0x55u, 0u);
    const uint32_t ay0 = by_offset(d.y, 2, 0xFFu, 0u, 0xCCu);
    const uint32_t ay1 = by_offset(d.y, 2, 0xFFu, 0x33u, 0u);
    const uint32_t az0 = by_offset(d.z, 4, 0xFFu, 0u, 0xF0u);
    const uint32_t az1 = by_offset(d.z, 4, 0xFFu, 0x0Fu, 0u);
    wa = (uint32_t)__popc(m);
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) {
      const uint32_t adj = ((q & 1u) ? ax1 : ax0) & ((q & 2u) ? ay1 : ay0) & ((q & 4u) ? az1 : az0);
      const uint32_t c2 = __popc(m & adj);
      if (q < 4) wa |= c2 << (8 + 6 * q);
      else wb |= c2 << (6 * (q - 4));
    }
  }
  // Each field's sum over the half-wave stays in range: all children <= 216,
  // E2 of one octant <= 27.
  const uint32_t ta = __shfl(half_incl_scan(wa), 31, 32);
  const uint32_t tb = __shfl(half_incl_scan(wb), 31, 32);
  // Lane j writes the counts of receiver child j (octant: the j-th set bit
  // of the mask), so the children's counts leave in one store each.
  if (j < (uint32_t)__popc(rmask)) {
    uint32_t mm = rmask;
    for (uint32_t t = 0; t < j; ++t) mm &= mm - 1;
    const uint32_t n2 = octant_field(ta, tb, (uint32_t)__builtin_ctz(mm));
    cnt2[rfirst + j] = n2;
    cnt4[rfirst + j] = (ta & 0xFFu) - n2;
  }
}

__global__ __launch_bounds__(256) void k_list_count(ListLevelArgs a, uint32_t* __restrict__ cnt2,
                                                    uint32_t* __restrict__ cnt4) {
  count_children(a, (uint64_t)xcd_block(blockIdx.x, gridDim.x) * 8 + (threadIdx.x >> 5),
                 threadIdx.x & 31u, cnt2, cnt4);
}

// One wave copies the metadata block to the host's pinned memory and then sets
// `published`: the host, which polls it, reads the totals some 20 us earlier
// than after a copy command and a stream synchronization. It sizes arrays by
// them, so every lane's words are released to the system before the flag is
// stored, and each word is stored once: the totals of pub.level and the
// overflow flag, the scan's own, in place of the block's.
__device__ __forceinline__ void publish_meta(const Publish& pub, uint64_t total2, uint64_t total4,
                                             uint32_t lane) {
  const uint32_t* from = (const uint32_t*)pub.meta;
  uint32_t* to = (uint32_t*)pub.to;
  const uint32_t at2 = offsetof(DevMeta, list_total) / 4 + 2u * pub.level;
  const uint32_t at4 = at2 + 2u * (kMaxLevel + 1);
  const bool over = total2 > 0xFFFFFFFFull || total4 > 0xFFFFFFFFull;
  for (uint32_t i = lane; i < offsetof(DevMeta, published) / 4; i += 64) {
    uint32_t v = from[i];
    if (i - at2 < 2u) v = (uint32_t)(total2 >> (32u * (i - at2)));
    if (i - at4 < 2u) v = (uint32_t)(total4 >> (32u * (i - at4)));
    if (i == offsetof(DevMeta, overflow) / 4 && over) v = 1u;
    __hip_atomic_store(to + i, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "");
  __builtin_amdgcn_wave_barrier();
  if (lane == 0)
    __hip_atomic_store(&pub.to->published, pub.level, __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_SYSTEM);
}

// A plain build's level 2 (at most 8 parents, 64 boxes): the counts and their
// offsets in one block, one launch (5 us) less than with the general scan.
__global__ __launch_bounds__(256) void k_list_first(ListLevelArgs a, ScanArgs sc) {
  __shared__ uint32_t s_cnt[2][64], s_tot[2];
  const uint32_t n = sc.n_dev ? *sc.n_dev : sc.n, lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  count_children(a, threadIdx.x >> 5, threadIdx.x & 31u, s_cnt[0], s_cnt[1]);
  __syncthreads();
  if (w < 2) {
    const uint32_t v = lane < n ? s_cnt[w][lane] : 0u;
    const uint32_t inc = wave_incl_scan(v);
    uint32_t* off = w ? sc.off4 : sc.off2;
    if (lane < n) off[lane] = inc - v;
    if (lane == 63) {  // (64 boxes of at most 64 entries: no overflow)
      off[n] = inc;
      *(w ? sc.total4 : sc.total2) = inc;
      s_tot[w] = inc;
    }
  }
  __syncthreads();
  if (sc.pub.to && w == 0) publish_meta(sc.pub, s_tot[0], s_tot[1], lane);
}

// LDS written by other lanes of this wave is read after this point (and the
// other way round): the LDS serves one wave's accesses in order, so this only
// keeps the compiler from moving them.
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// Staged words [b, e) at `lds` (b = g % 4 on the first flush of a run, later
// 0) are entries [g, ...) of `ent`, which is 16-byte aligned: whole 16-byte
// groups are stored, and where the run starts or ends inside a group its ragged
// words in one 4-byte store (lanes 0..3 the head, 4..7 the tail). Unless the
// run ends here (last), the words past the last whole group move to the front.
// Leaves the new b, e and g.
__device__ __forceinline__ void flush_entries(uint32_t* lds, uint32_t& b, uint32_t& e, uint32_t& g,
                                              uint32_t* __restrict__ ent, bool last, uint32_t lane) {
  wave_sync();
  const uint32_t a4 = (b + 3u) & ~3u, e4 = max(e & ~3u, a4);
  uint32_t* out = ent + ((uint64_t)g - b);  // entry of LDS word 0
  for (uint32_t i = 4u * lane + a4; i < e4; i += 256u) *(uint4*)(out + i) = *(const uint4*)(lds + i);
  if (last || b != 0) {
    const uint32_t i = lane < 4 ? b + lane : e4 + lane - 4u;
    const uint32_t stop = lane < 4 ? min(a4, e) : e;
    if (lane < (last ? 8u : 4u) && i < stop) out[i] = lds[i];
  }
  if (!last) {  // (a4 <= e here: a flush that is not the last holds many words)
    const uint32_t v = lds[e4 + (lane & 3u)];
    wave_sync();
    if (lane < 4) lds[lane] = v;
    g += e4 - b;
    b = 0;
    e -= e4;
  }
  wave_sync();
}

// NEXT: also write the counts of level + 1 (see ListLevelArgs). Take a
// receiver child r of p (octant q). E2 of r's children lies in the 4 x 4 x 4
// boxes of level + 1 around r's 2 x 2 x 2 (cells -1..2 per axis), and the
// candidates (the children of E2(r)) in the 6 x 6 x 6 around it. Lane j holds
// the 4 x 4 x 4 grid of s_j's grandchildren (its node); with s_j at offset d
// from p, its cell Y sits at 4d + Y - 2q from r per axis, so the part inside
// r's 4 x 4 x 4 window is a mask of the grid (by d and q per axis) rotated by
// one amount. ORing it over the lanes gives the window's occupancy W; the E2
// count of r's child q' is the population of W under the 3 x 3 x 3 cells at
// q'. The candidates' number is the sum over the lanes of the grid's
// population under the child octants within E2(r).
//
// A wave takes PAIRS consecutive pairs of parents, all of whose loads (three
// dependent ones: p's node and list range, then the list entries, then the
// neighbors' nodes) are made before the first pair's stores, so that one wait
// serves them all: with two pairs the sparse levels of a 2M-point level-13
// build take 1.43 ms in all against 1.60 ms with one (uniform level 8: 1641 us
// either way; its full level 7, 448 against 423 us).
template <bool NEXT, bool BATCH, uint32_t PAIRS>
__device__ __forceinline__ void fill_wave(const ListLevelArgs& a,
                                          const uint32_t* __restrict__ off2,
                                          const uint32_t* __restrict__ off4,
                                          uint32_t* __restrict__ ent2,
                                          uint32_t* __restrict__ ent4,
                                          uint32_t (&s_all)[4][kFillWords]) {
  // per wave: first U of both parents (8 bytes an entry), with NEXT also
  // the windows of the receiver children; then the staged E2 and E4 entries
  const uint32_t lane = threadIdx.x & 63u, j = lane & 31u, hf = lane >> 5;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  uint32_t* lds = s_all[w];
  const uint32_t n_up = a.n_recv_up_dev ? *a.n_recv_up_dev : a.n_recv_up;
  const uint64_t p0 = ((uint64_t)xcd_block(blockIdx.x, gridDim.x) * 4 + w) * (2 * PAIRS);
  if (p0 >= n_up) return;  // whole wave: no parent
  // Per pair, one half-wave per parent p (lane j: the j-th entry s of E2(p)).
  // Every load is made, from a place that is there where its value is not
  // wanted (a branch around a load waits for it): absent parents repeat the
  // last one, lanes past the list its last entry.
  uint2 np_[PAIRS], nr_[PAIRS];    // p's node; NEXT: child j's first child and mask
  uint4 ns_[PAIRS];                // s's node
  uint32_t j0[PAIRS], cnt[PAIRS];  // E2(p)
  uint32_t o2_[PAIRS], o4_[PAIRS]; // where the lists of p's children start
  // batch: rank of the set's first box at level - 1 (entries of E2(p) are
  // relative to it) and at level, and the set's own level
  uint32_t upbase[PAIRS], base_[PAIRS], lev[PAIRS], ent[PAIRS];
  uint64_t key[PAIRS];
#pragma unroll
  for (uint32_t i = 0; i < PAIRS; ++i) {
    const uint32_t p = (uint32_t)min(p0 + 2 * i + hf, (uint64_t)n_up - 1);
    np_[i] = *(const uint2*)&a.recv_node_up[p];
    key[i] = BATCH ? a.recv_key_up[p] : 0;
    j0[i] = cnt[i] = 0;
    if (!a.up_all) {
      j0[i] = a.e2_off_up[p];
      cnt[i] = a.e2_off_up[p + 1];
    }
  }
  const uint32_t n_src_up = a.n_src_up_dev ? *a.n_src_up_dev : a.n_src_up;
#pragma unroll
  for (uint32_t i = 0; i < PAIRS; ++i) {
    const uint2 np = np_[i];
    o2_[i] = off2[np.x];
    o4_[i] = off4[np.x];
    upbase[i] = base_[i] = lev[i] = 0;
    if (BATCH) {
      const uint32_t set = (uint32_t)(key[i] >> (3 * (a.level - 1)));
      base_[i] = a.first_cur[set];
      upbase[i] = a.first_up[set];
      lev[i] = a.set_level[set];
      if (a.up_all) cnt[i] = a.first_up[set + 1];
    } else if (a.up_all) {
      cnt[i] = n_src_up;
    }
    if (!a.up_all) {
      cnt[i] -= j0[i];
      ent[i] = a.e2_ent_up[cnt[i] ? j0[i] + min(j, cnt[i] - 1u) : 0u];
    }
    nr_[i] = make_uint2(0, 0);
    if (NEXT)
      nr_[i] = *(const uint2*)&a.recv_node_cur[np.x + min(j, (uint32_t)__popc(np.y & 0xFFu) - 1u)];
  }
#pragma unroll
  for (uint32_t i = 0; i < PAIRS; ++i) {
    if (BATCH) {
      if (a.up_all) cnt[i] -= upbase[i];  // (it was the set's end)
      if (lev[i] < a.level) cnt[i] = 0;  // the set's lists stop above this level
    }
    if (a.up_all) ent[i] = cnt[i] ? min(j, cnt[i] - 1u) : 0u;
    const uint4* s = &a.src_node_up[cnt[i] ? upbase[i] + ent[i] : 0u];
    ns_[i] = make_uint4(0, 0, 0, 0);
    if (NEXT) {
      ns_[i] = *s;
    } else {
      const uint2 v = *(const uint2*)s;
      ns_[i].x = v.x, ns_[i].y = v.y;
    }
  }

#pragma unroll 1
  for (uint32_t i = 0; i < PAIRS; ++i) {
  if (PAIRS > 1 && p0 + 2 * i >= n_up) return;
  const bool live = p0 + 2 * i + hf < n_up;
  const uint2 np = make_uint2(np_[0].x, live ? np_[0].y : 0u), nr = nr_[0];
  uint4 ns = ns_[0];
  if (!live || j >= cnt[0]) ns.y = ns.z = ns.w = 0;  // lanes without an entry: no children
  const uint32_t my_o2 = o2_[0], my_o4 = o4_[0], base = base_[0];
  const bool next_zero = BATCH && lev[0] < a.level + 1;  // the set has no lists at level + 1
#pragma unroll
  for (uint32_t t = 0; t + 1 < PAIRS; ++t) {
    np_[t] = np_[t + 1], nr_[t] = nr_[t + 1], ns_[t] = ns_[t + 1], cnt[t] = cnt[t + 1];
    o2_[t] = o2_[t + 1], o4_[t] = o4_[t + 1], base_[t] = base_[t + 1], lev[t] = lev[t + 1];
  }
  const uint32_t rmask = np.y & 0xFFu;
  const Offset d = node_offset(ns.y >> 8, np.y >> 8);
  const uint32_t m = ns.y & 0xFFu;  // (no children on lanes without an entry)
  const uint32_t pm0 = (uint32_t)__builtin_amdgcn_readlane(rmask, 0),
                 pm1 = (uint32_t)__builtin_amdgcn_readlane(rmask, 32);

  if (NEXT) {
    // per axis and receiver octant bit: the grid cells inside the window (K)
    // and those of the child octants within E2 (C)
    const uint32_t kx[2] = {by_offset(d.x, 1, 0x77777777u, 0u, 0x88888888u),
                            by_offset(d.x, 1, 0xEEEEEEEEu, 0x11111111u, 0u)};
    const uint32_t ky[2] = {by_offset(d.y, 2, 0x0FFF0FFFu, 0u, 0xF000F000u),
                            by_offset(d.y, 2, 0xFFF0FFF0u, 0x000F000Fu, 0u)};
    const uint32_t kl[2] = {by_offset(d.z, 4, 0xFFFFFFFFu, 0u, 0u),
                            by_offset(d.z, 4, 0xFFFF0000u, 0x0000FFFFu, 0u)};
    const uint32_t kh[2] = {by_offset(d.z, 4, 0x0000FFFFu, 0u, 0xFFFF0000u),
                            by_offset(d.z, 4, 0xFFFFFFFFu, 0u, 0u)};
    const uint32_t cx[2] = {by_offset(d.x, 1, 0xFFFFFFFFu, 0u, 0xCCCCCCCCu),
                            by_offset(d.x, 1, 0xFFFFFFFFu, 0x33333333u, 0u)};
    const uint32_t cy[2] = {by_offset(d.y, 2, 0xFFFFFFFFu, 0u, 0xFF00FF00u),
                            by_offset(d.y, 2, 0xFFFFFFFFu, 0x00FF00FFu, 0u)};
    const uint32_t cl[2] = {by_offset(d.z, 4, 0xFFFFFFFFu, 0u, 0u),
                            by_offset(d.z, 4, 0xFFFFFFFFu, 0xFFFFFFFFu, 0u)};
    const uint32_t ch[2] = {by_offset(d.z, 4, 0xFFFFFFFFu, 0u, 0xFFFFFFFFu),
                            by_offset(d.z, 4, 0xFFFFFFFFu, 0u, 0u)};
    // rotation: per axis 4 d + 1 - 2 q cells of stride 1, 4, 16
    const uint32_t rot = 21u + by_offset(d.x, 1, 0u, 4u, 60u) + by_offset(d.y, 2, 0u, 16u, 48u);
    uint32_t* slot = lds + 4 * kUnion + 32 * hf;  // 4 words per octant
#pragma unroll
    for (uint32_t q = 0; q < 8; ++q) {
      if (!(((pm0 | pm1) >> q) & 1u)) continue;
      const uint32_t qx = q & 1u, qy = (q >> 1) & 1u, qz = q >> 2;
      const uint64_t in = (uint64_t)(ns.z & kx[qx] & ky[qy] & kl[qz]) |
                          (uint64_t)(ns.w & kx[qx] & ky[qy] & kh[qz]) << 32;
      const uint32_t sh = (rot - 2u * qx - 8u * qy - 32u * qz) & 63u;
      const uint64_t w = in << sh | in >> ((64u - sh) & 63u);
      const uint32_t all = (uint32_t)__popc(ns.z & cx[qx] & cy[qy] & cl[qz]) +
                           (uint32_t)__popc(ns.w & cx[qx] & cy[qy] & ch[qz]);
      const uint32_t wl = half_or_last((uint32_t)w), wh = half_or_last((uint32_t)(w >> 32));
      const uint32_t sum = half_incl_scan(all);
      if (j == 31u) *(uint4*)(slot + 4 * q) = make_uint4(wl, wh, sum, 0u);
    }
    wave_sync();
    // lane 8 q + q': child q' of p's child in octant q, each parent in turn
    const uint32_t q = lane >> 3, qq = lane & 7u;
    const uint32_t ex = (qq & 1u) ? 0xEEEEEEEEu : 0x77777777u,
                   ey = (qq & 2u) ? 0xFFF0FFF0u : 0x0FFF0FFFu,
                   el = (qq & 4u) ? 0xFFFF0000u : 0xFFFFFFFFu,
                   eh = (qq & 4u) ? 0xFFFFFFFFu : 0x0000FFFFu;
#pragma unroll
    for (uint32_t hh = 0; hh < 2; ++hh) {
      const uint32_t pm = hh ? pm1 : pm0;
      const bool nz = __builtin_amdgcn_readlane(next_zero ? 1 : 0, 32 * hh) != 0;
      const uint32_t i = (uint32_t)__popc(pm & ((1u << q) - 1u));
      const uint32_t rm = (uint32_t)__shfl((int)(nr.y & 0xFFu), (int)(32 * hh + i));
      const uint32_t rc = (uint32_t)__shfl((int)nr.x, (int)(32 * hh + i));
      if (((pm >> q) & 1u) && ((rm >> qq) & 1u)) {
        const uint4 v = *(const uint4*)(lds + 4 * kUnion + 32 * hh + 4 * q);
        const uint32_t c2 = (uint32_t)__popc(v.x & ex & ey & el) + (uint32_t)__popc(v.y & ex & ey & eh);
        const uint32_t at = rc + (uint32_t)__popc(rm & ((1u << qq) - 1u));
        a.cnt2_next[at] = nz ? 0u : c2;
        a.cnt4_next[at] = nz ? 0u : v.z - c2;
      }
    }
  }

  // U: per child of s_j its rank and the receiver octants it is adjacent to.
  // Per axis, receiver octants (bits: receivers with the x / y / z bit set
  // 0xAA / 0xCC / 0xF0) a child with axis bit 0 / 1 touches: offset 0: all;
  // +1 (s above p on the axis): a child with bit 0 touches the receivers with
  // bit 1; -1: a child with bit 1 touches the receivers with bit 0. Laid out
  // as one byte per child octant, octants 0..3 in lo, 4..7 in hi.
  const uint32_t c = (uint32_t)__popc(m);
  const uint32_t incl = half_incl_scan(c);
  {
    const uint32_t ax = by_offset(d.x, 1, 0xFFFFFFFFu, 0x00AA00AAu, 0x55005500u);
    const uint32_t ay = by_offset(d.y, 2, 0xFFFFFFFFu, 0x0000CCCCu, 0x33330000u);
    const uint32_t lo = ax & ay & by_offset(d.z, 4, 0xFFFFFFFFu, 0xF0F0F0F0u, 0u);
    const uint32_t hi = ax & ay & by_offset(d.z, 4, 0xFFFFFFFFu, 0u, 0x0F0F0F0Fu);
    uint2* U = (uint2*)lds + kUnion * hf;
    uint32_t at = incl - c, rank = ns.x - base;
#pragma unroll
    for (uint32_t o = 0; o < 8; ++o) {
      const uint32_t bit = (m >> o) & 1u;
      // absent octants write to a slot past U
      U[bit ? at : (uint32_t)kUnion - 1u] = make_uint2(rank, (o < 4 ? lo : hi) >> (8 * (o & 3u)));
      at += bit;
      rank += bit;
    }
  }
  wave_sync();
  // Both parents' U into registers (slots past its end: adjacent to none).
  uint32_t u[2][4], ad[2][4], T[2];
#pragma unroll
  for (uint32_t hh = 0; hh < 2; ++hh) {
    T[hh] = (uint32_t)__builtin_amdgcn_readlane(incl, 32 * hh + 31);
    const uint2* U = (const uint2*)lds + kUnion * hh;
#pragma unroll
    for (uint32_t k = 0; k < 4; ++k) {
      const uint32_t idx = 64u * k + lane;
      const uint2 v = U[min(idx, (uint32_t)kUnion - 1u)];
      u[hh][k] = v.x;
      ad[hh][k] = idx < T[hh] ? v.y : 0u;
    }
  }
  wave_sync();
  // Split, the whole wave on one parent at a time, into LDS. Lanes past U's
  // end write past the staged E4 entries, where the next chunk (or nothing)
  // writes again. Both parents' lists are one run (the second's children
  // follow the first's).
  uint32_t* st2 = lds;
  uint32_t* st4 = lds + kFillE2;
  uint32_t g2 = (uint32_t)__builtin_amdgcn_readlane((int)my_o2, 0),
           g4 = (uint32_t)__builtin_amdgcn_readlane((int)my_o4, 0);
  uint32_t b2 = g2 & 3u, b4 = g4 & 3u, e2 = b2, e4 = b4;  // staged: [b, e) of st2 / st4
#pragma unroll
  for (uint32_t hh = 0; hh < 2; ++hh) {
    uint32_t qm = hh ? pm1 : pm0;
#pragma unroll 1
    while (qm) {
      const uint32_t bit = (uint32_t)__builtin_amdgcn_readfirstlane((int)(qm & (0u - qm)));
      qm &= qm - 1;
      if (e4 + T[hh] + 64u > kFillE4)  // the child might not fit
        flush_entries(st4, b4, e4, g4, ent4, false, lane);
#pragma unroll
      for (uint32_t k = 0; k < 4; ++k) {
        if (64u * k < T[hh]) {
          const bool is2 = (ad[hh][k] & bit) != 0u;
          const uint64_t bal = __ballot(is2);
          const uint32_t i2 = __builtin_amdgcn_mbcnt_hi(
              (uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, e2));
          lds[is2 ? i2 : kFillE2 + e2 + e4 + lane - i2] = u[hh][k];
          const uint32_t n2 = (uint32_t)__popcll(bal);
          e2 += n2;
          e4 += min(T[hh] - 64u * k, 64u) - n2;
        }
      }
    }
  }
  flush_entries(st4, b4, e4, g4, ent4, true, lane);
  flush_entries(st2, b2, e2, g2, ent2, true, lane);
  }
}

// (As many waves per SIMD as the registers allow without scratch memory, which the
// runtime takes from the device when a kernel first runs on a queue: on a full
// device that ends the queue.)
template <bool NEXT, bool BATCH, uint32_t PAIRS>
__global__ __launch_bounds__(256, NEXT && PAIRS > 1 ? (BATCH ? 6 : 7) : 8) void k_list_fill(
    ListLevelArgs a, const uint32_t* __restrict__ off2, const uint32_t* __restrict__ off4,
    uint32_t* __restrict__ ent2, uint32_t* __restrict__ ent4) {
  __shared__ __align__(16) uint32_t s_all[4][kFillWords];
  fill_wave<NEXT, BATCH, PAIRS>(a, off2, off4, ent2, ent4, s_all);
}

// A coarse level of a plain build, whose next level has at most kScanSmall
// boxes: the block that finishes last (`done` counts them) also turns the next
// level's counts into offsets. Level 2 of a 4097-point build: fill, gap and scan
// took 5.7 + 3.8 + 4.6 us, this 8.2. Whole builds with it and without, us: 600
// points at level 5 88 / 93, 3000 90 / 94, 4096 at level 4 74.6 / 77.5, 65536 at
// level 5 112 / 114. kScanSmall is what one block's registers hold. The counter
// releases each block's counts and acquires the others' for the block that scans
// them, which a grid of many blocks pays for many times. Trees whose levels have as
// many boxes as points, scanned by the fills (without kScanParents) and apart: at
// level 10 513 points 176 / 180, 700 180 / 184, 800 182 / 184, 900 185.5 / 184.5, 1000
// 186.5 / 185; at level 8 3000 167 / 150, 4096 180 / 153.
constexpr uint32_t kScanSmallItems = kScanSmall / 256;
__global__ __launch_bounds__(256) void k_list_fill_scan(ListLevelArgs a,
                                                           const uint32_t* __restrict__ off2,
                                                           const uint32_t* __restrict__ off4,
                                                           uint32_t* __restrict__ ent2,
                                                           uint32_t* __restrict__ ent4,
                                                           ScanArgs sc,
                                                           uint32_t* __restrict__ done) {
  __shared__ __align__(16) uint32_t s_all[4][kFillWords];
  __shared__ uint32_t s_done, s_w[2][4], s_tot[2];
  fill_wave<true, false, 1>(a, off2, off4, ent2, ent4, s_all);
  __syncthreads();
  if (threadIdx.x == 0)
    s_done = __hip_atomic_fetch_add(done, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT);
  __syncthreads();
  if (s_done + 1 != gridDim.x) return;  // whole block
  const uint32_t n = sc.n_dev ? *sc.n_dev : sc.n;
  const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
  // The counts, read 256 consecutive ones at a time into LDS (E4 in the high
  // half; at most 216), from which each thread takes kScanSmallItems consecutive
  // ones (65536 points, level 3 to 4, fill and scan: 16.8 us with each thread
  // reading its own, now 14.0).
  static_assert(kScanSmall <= 4 * kFillWords, "the counts fit the staging space");
  uint32_t* st = &s_all[0][0];
  {
    uint32_t c2[kScanSmallItems], c4[kScanSmallItems];
#pragma unroll
    for (uint32_t i = 0; i < kScanSmallItems; ++i) {
      const uint32_t k = min(256u * i + threadIdx.x, max(n, 1u) - 1u);
      c2[i] = sc.cnt2[k];
      c4[i] = sc.cnt4[k];
    }
#pragma unroll
    for (uint32_t i = 0; i < kScanSmallItems; ++i) {
      const uint32_t k = 256u * i + threadIdx.x;
      st[k] = k < n ? c4[i] << 16 | c2[i] : 0u;
    }
  }
  __syncthreads();
  const uint32_t base = threadIdx.x * kScanSmallItems;
  uint32_t v[kScanSmallItems], sum2 = 0, sum4 = 0;
#pragma unroll
  for (uint32_t i = 0; i < kScanSmallItems; ++i) {
    v[i] = st[base + i];
    sum2 += v[i] & 0xFFFFu;
    sum4 += v[i] >> 16;
  }
  const uint32_t inc2 = wave_incl_scan(sum2), inc4 = wave_incl_scan(sum4);
  if (lane == 63) {
    s_w[0][w] = inc2;
    s_w[1][w] = inc4;
  }
  __syncthreads();
  uint32_t pre2 = inc2 - sum2, pre4 = inc4 - sum4;
  for (uint32_t i = 0; i < w; ++i) {
    pre2 += s_w[0][i];
    pre4 += s_w[1][i];
  }
  // (at most kScanSmall * 216 entries: no overflow)
  if (threadIdx.x == 255) {
    sc.off2[n] = s_tot[0] = pre2 + sum2;
    sc.off4[n] = s_tot[1] = pre4 + sum4;
    *sc.total2 = pre2 + sum2;
    *sc.total4 = pre4 + sum4;
  }
  // the offsets out through LDS the same way
  auto put = [&](uint32_t pre, uint32_t shift, uint32_t* off) {
    __syncthreads();
#pragma unroll
    for (uint32_t i = 0; i < kScanSmallItems; ++i) {
      st[base + i] = pre;
      pre += (v[i] >> shift) & 0xFFFFu;
    }
    __syncthreads();
    for (uint32_t k = threadIdx.x; k < n; k += 256) off[k] = st[k];
  };
  put(pre2, 0, sc.off2);
  put(pre4, 16, sc.off4);
  __syncthreads();
  if (sc.pub.to && w == 0) publish_meta(sc.pub, s_tot[0], s_tot[1], lane);
}

__global__ __launch_bounds__(64) void k_publish(Publish pub) {
  publish_meta(pub, 0, 0, threadIdx.x);
}

void launch_publish(const Publish& pub, hipStream_t s) {
  hipLaunchKernelGGL(k_publish, dim3(1), dim3(64), 0, s, pub);
}

void launch_list_first(const ListLevelArgs& a, const ScanArgs& sc, hipStream_t s) {
  hipLaunchKernelGGL(k_list_first, dim3(1), dim3(256), 0, s, a, sc);
}

void launch_list_count(const ListLevelArgs& a, uint32_t* cnt2, uint32_t* cnt4, hipStream_t s) {
  if (a.n_recv_up == 0) return;  // with n_recv_up_dev: the capacity
  hipLaunchKernelGGL(k_list_count, dim3(div_up(a.n_recv_up, 8)), dim3(256), 0, s, a, cnt2, cnt4);
}

constexpr uint32_t kFillTwoPairs = 1u << 16;

void launch_list_fill(const ListLevelArgs& a, const uint32_t* off2, const uint32_t* off4,
                      uint32_t* ent2, uint32_t* ent4, hipStream_t s, const ScanArgs& next,
                      uint32_t* done) {
  if (a.n_recv_up == 0) return;
  // Two pairs of parents per wave once that still fills the chip's 8192 wave
  // slots twice; below, the level is one round of waves and takes as long as
  // one of them does.
  const bool two = a.n_recv_up >= kFillTwoPairs;
  const dim3 grid(div_up(a.n_recv_up, two ? 16 : 8));
  if (done) {
    hipLaunchKernelGGL(k_list_fill_scan, grid, dim3(256), 0, s, a, off2, off4, ent2, ent4, next,
                       done);
    return;
  }
#define FMMDS_FILL(N, B, P)                                                                      \
  hipLaunchKernelGGL((k_list_fill<N, B, P>), grid, dim3(256), 0, s, a, off2, off4, ent2, ent4)
#define FMMDS_FILL_P(N, B)                                                                       \
  do {                                                                                           \
    if (two) FMMDS_FILL(N, B, 2);                                                                \
    else FMMDS_FILL(N, B, 1);                                                                    \
  } while (0)
  if (a.cnt2_next) {
    if (a.first_up) FMMDS_FILL_P(true, true);
    else FMMDS_FILL_P(true, false);
  } else {
    if (a.first_up) FMMDS_FILL_P(false, true);
    else FMMDS_FILL_P(false, false);
  }
#undef FMMDS_FILL_P
#undef FMMDS_FILL
}

// ---------------------------------------------------------------------------
// Exclusive scans of the per-box E2 and E4 list lengths into CSR offsets (the
// scan that turns NumRecvE2NeiNEBox into NeighborBookmark, Algorithm 4), both
// in one single pass. off[n] = total; the totals also go to total[0..1], and
// the overflow flag is set if a total does not fit 32-bit offsets. Wave 0
// chains the E2 sums across tiles, wave 1 the E4 sums, at the same time.
// Each thread owns 16 consecutive boxes, read and written with 16-byte
// accesses (both count arrays and both offset arrays start 16-byte aligned).
// ---------------------------------------------------------------------------
// 1024 threads x 16 counts per tile: a quarter of the tiles (and of the
// look-back chain) of 256-thread tiles; the largest scan (10.6M boxes) took
// 98 us with 4096-count tiles.
constexpr int kScanBlock = 1024;
constexpr int kScanItems = 16;
constexpr int kScanTile = kScanBlock * kScanItems;  // 16384 boxes

__global__ __launch_bounds__(kScanBlock) void k_scan_counts2(
    ScanArgs sc, uint64_t* __restrict__ status2, uint64_t* __restrict__ status4,
    uint32_t* __restrict__ tile_counter) {
  const uint32_t* __restrict__ cnt2 = sc.cnt2;
  const uint32_t* __restrict__ cnt4 = sc.cnt4;
  uint32_t* __restrict__ off2 = sc.off2;
  uint32_t* __restrict__ off4 = sc.off4;
  __shared__ uint32_t s_w[2][kScanBlock / 64];
  __shared__ uint64_t s_excl[2], s_tot[2];
  __shared__ uint32_t s_tile;
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t n = sc.n_dev ? *sc.n_dev : sc.n;
  if (tid == 0) s_tile = atomicAdd(tile_counter, 1u);
  __syncthreads();
  const uint32_t tile = s_tile;
  if ((uint64_t)tile * kScanTile >= n) return;  // whole block: surplus tile
  const uint64_t base = (uint64_t)tile * kScanTile + (uint64_t)tid * kScanItems;
  uint32_t v2[kScanItems], v4[kScanItems];
  const bool full = base + kScanItems <= n;  // 16-byte loads and stores
  if (full) {
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q) {
      const uint4 a2 = ((const uint4*)(cnt2 + base))[q];
      const uint4 a4 = ((const uint4*)(cnt4 + base))[q];
      v2[4 * q] = a2.x, v2[4 * q + 1] = a2.y, v2[4 * q + 2] = a2.z, v2[4 * q + 3] = a2.w;
      v4[4 * q] = a4.x, v4[4 * q + 1] = a4.y, v4[4 * q + 2] = a4.z, v4[4 * q + 3] = a4.w;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      const bool ok = base + i < n;
      v2[i] = ok ? cnt2[base + i] : 0;
      v4[i] = ok ? cnt4[base + i] : 0;
    }
  }
  uint32_t sum2 = 0, sum4 = 0;
#pragma unroll
  for (int i = 0; i < kScanItems; ++i) {
    sum2 += v2[i];
    sum4 += v4[i];
  }
  const uint32_t inc2 = wave_incl_scan(sum2), inc4 = wave_incl_scan(sum4);
  if (lane == 63) {
    s_w[0][w] = inc2;
    s_w[1][w] = inc4;
  }
  __syncthreads();
  uint32_t wpre2 = 0, wpre4 = 0, tot2 = 0, tot4 = 0;
  for (uint32_t i = 0; i < kScanBlock / 64; ++i) {
    if (i < w) {
      wpre2 += s_w[0][i];
      wpre4 += s_w[1][i];
    }
    tot2 += s_w[0][i];
    tot4 += s_w[1][i];
  }
  if (w == 0) {
    const uint64_t ex = lookback_wave(status2, tile, tot2);
    if (lane == 0) s_excl[0] = ex;
  } else if (w == 1) {
    const uint64_t ex = lookback_wave(status4, tile, tot4);
    if (lane == 0) s_excl[1] = ex;
  }
  __syncthreads();
  uint64_t pre2 = s_excl[0] + wpre2 + inc2 - sum2;
  uint64_t pre4 = s_excl[1] + wpre4 + inc4 - sum4;
  bool ovf = false;
  if (full) {
#pragma unroll
    for (int q = 0; q < kScanItems / 4; ++q) {
      uint4 o2, o4;
      o2.x = (uint32_t)pre2, pre2 += v2[4 * q], o4.x = (uint32_t)pre4, pre4 += v4[4 * q];
      o2.y = (uint32_t)pre2, pre2 += v2[4 * q + 1], o4.y = (uint32_t)pre4, pre4 += v4[4 * q + 1];
      o2.z = (uint32_t)pre2, pre2 += v2[4 * q + 2], o4.z = (uint32_t)pre4, pre4 += v4[4 * q + 2];
      o2.w = (uint32_t)pre2, pre2 += v2[4 * q + 3], o4.w = (uint32_t)pre4, pre4 += v4[4 * q + 3];
      ((uint4*)(off2 + base))[q] = o2;
      ((uint4*)(off4 + base))[q] = o4;
    }
    if (base + kScanItems == n) {
      off2[n] = (uint32_t)pre2;
      off4[n] = (uint32_t)pre4;
      *sc.total2 = s_tot[0] = pre2;
      *sc.total4 = s_tot[1] = pre4;
    }
  } else {
#pragma unroll
    for (int i = 0; i < kScanItems; ++i) {
      if (base + i < n) {
        off2[base + i] = (uint32_t)pre2;
        off4[base + i] = (uint32_t)pre4;
        pre2 += v2[i];
        pre4 += v4[i];
        if (base + i + 1 == n) {
          off2[n] = (uint32_t)pre2;
          off4[n] = (uint32_t)pre4;
          *sc.total2 = s_tot[0] = pre2;
          *sc.total4 = s_tot[1] = pre4;
        }
      }
    }
  }
  ovf = (pre2 > 0xFFFFFFFFull) || (pre4 > 0xFFFFFFFFull);
  if (ovf) atomicOr(sc.overflow, 1u);
  if (sc.pub.to && (uint64_t)(tile + 1) * kScanTile >= n) {  // the last tile
    __syncthreads();
    if (w == 0) publish_meta(sc.pub, s_tot[0], s_tot[1], lane);
  }
}

uint32_t scan_tiles(uint32_t n) { return div_up(n, kScanTile); }

void launch_scan_counts2(const ScanArgs& sc, uint64_t* status2, uint64_t* status4,
                         uint32_t* tile_counter, hipStream_t s) {
  if (sc.n == 0) return;
  hipLaunchKernelGGL(k_scan_counts2, dim3(scan_tiles(sc.n)), dim3(kScanBlock), 0, s, sc, status2,
                     status4, tile_counter);
}

}  // namespace fmmds
