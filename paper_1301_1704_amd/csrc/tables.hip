// Nonempty-box tables: box boundaries of every level, parents, children and
// the list kernels' records, from the sorted points.
//
// The paper scans a dense histogram of all 8^lmax boxes (Section 2.3,
// Algorithm 3), which costs memory and time in the number of boxes. Here the
// sorted keys already group the points by box, so a box starts wherever the
// key differs from the previous one (adjacent difference) and the starts are
// compacted by a scan: the cost follows the nonempty boxes only. A box's
// parent is its Morton index shifted by one level (Section 3.2), so the same
// comparison, on the keys shifted, finds the boxes of every coarser level.
#include "device.h"
#include "internal.h"

namespace fmmds {

constexpr int kCompWaves = kCompBlock / 64;

struct P3 {
  float x, y, z;
};

// ---------------------------------------------------------------------------
// The finest level alone, with a chained scan (the dense variant's ordering
// of very full boxes): from the sorted (key, index) pairs write the
// permutation and the reordered coordinates (Algorithm 5, steps 3 and 6:
// SortedSrc / SortedRecv and RecvPermutationIdx) and compact the finest
// level's nonempty boxes: their keys and bookmarks (Algorithm 3's NonEmptyIdx
// and Bookmark).
// ---------------------------------------------------------------------------
template <bool PACKED, typename KeyT>
__global__ __launch_bounds__(kCompBlock) void k_leaf(
    const uint64_t* __restrict__ sk, const uint32_t* __restrict__ sv, const P3* __restrict__ xyz,
    uint32_t n, uint32_t* __restrict__ perm, P3* __restrict__ sorted_xyz,
    KeyT* __restrict__ leaf_key, uint32_t* __restrict__ leaf_begin, uint64_t* __restrict__ status,
    uint32_t* __restrict__ tile_counter, uint32_t* __restrict__ n_out) {
  __shared__ uint32_t s_cnt[kCompItems * kCompWaves];
  __shared__ uint64_t s_excl;
  __shared__ uint32_t s_tile;
  const uint32_t tid = threadIdx.x, w = tid >> 6;
  if (tid == 0) s_tile = atomicAdd(tile_counter, 1u);
  __syncthreads();
  const uint32_t tile = s_tile;
  const uint64_t tbase = (uint64_t)tile * kCompTile;

  uint64_t key[kCompItems];
  uint32_t incl[kCompItems];
  uint32_t flags = 0;
#pragma unroll
  for (int i = 0; i < kCompItems; ++i) {
    const uint64_t e = tbase + (uint64_t)i * kCompBlock + tid;
    const bool valid = e < n;
    uint64_t kk = 0, kp = 0;
    uint32_t idx = 0;
    if (valid) {
      const uint64_t el = sk[e];
      kk = PACKED ? (el >> 32) : el;
      idx = PACKED ? (uint32_t)el : sv[e];
      if (e > 0) kp = PACKED ? (sk[e - 1] >> 32) : sk[e - 1];
      perm[e] = idx;
      if (xyz) sorted_xyz[e] = xyz[idx];  // null: the coordinates are already in place
    }
    const bool f = valid && (e == 0 || kk != kp);
    const uint64_t ball = __ballot(f);
    incl[i] = mbcnt(ball) + (f ? 1u : 0u);
    flags |= (f ? 1u : 0u) << i;
    key[i] = kk;
    if ((tid & 63) == 0) s_cnt[i * kCompWaves + w] = (uint32_t)__popcll(ball);
  }
  const uint64_t texcl = tile_flags_prefix<kCompItems * kCompWaves>(s_cnt, &s_excl, status, tile);
#pragma unroll
  for (int i = 0; i < kCompItems; ++i) {
    const uint64_t e = tbase + (uint64_t)i * kCompBlock + tid;
    const uint64_t rank_incl = texcl + s_cnt[i * kCompWaves + w] + incl[i];
    if ((flags >> i) & 1u) {
      leaf_key[rank_incl - 1] = (KeyT)key[i];
      leaf_begin[rank_incl - 1] = (uint32_t)e;
    }
    if (e + 1 == n) {
      leaf_begin[rank_incl] = n;
      *n_out = (uint32_t)rank_incl;
    }
  }
}

void launch_leaf(bool packed, bool key64, const uint64_t* sk, const uint32_t* sv,
                 const float* xyz, uint32_t n, uint32_t* perm, float* sorted_xyz, void* leaf_key,
                 uint32_t* leaf_begin, uint64_t* status, uint32_t* tile_counter, uint32_t* n_out,
                 hipStream_t s) {
  const uint32_t grid = div_up(n, kCompTile);
#define FMMDS_LEAF(P, K)                                                                         \
  hipLaunchKernelGGL((k_leaf<P, K>), dim3(grid), dim3(kCompBlock), 0, s, sk, sv, (const P3*)xyz, \
                     n, perm, (P3*)sorted_xyz, (K*)leaf_key, leaf_begin, status, tile_counter,    \
                     n_out)
  if (packed && key64) FMMDS_LEAF(true, uint64_t);
  else if (packed) FMMDS_LEAF(true, uint32_t);
  else if (key64) FMMDS_LEAF(false, uint64_t);
  else FMMDS_LEAF(false, uint32_t);
#undef FMMDS_LEAF
}

// ---------------------------------------------------------------------------
// Every level at once from the sorted points (the plain build and the
// rebuild): reduce, scan, write. A point e starts a new box at level l iff
// its key and the previous point's key differ above the lowest 3 (L - l)
// bits, i.e. iff l >= d(e), where d(e) = L - (highest differing bit) / 3 (0
// for the first point; L + 1, no new box, for equal keys). So one pass over
// the points has every level's box starts:
//   k_tab_count  per tile of 2048 points and per level, the number of box
//                starts (one ballot per level and item);
//   k_tab_scan   per level, the exclusive scan of those counts over the
//                tiles, and the level's box count;
//   k_tab_write  per point: the permutation, the coordinates, and for every
//                level l >= d(e) the box's key, bookmark (the point itself),
//                parent (the level l - 1 box holding the point) and first
//                child (the level l + 1 box starting at the point);
//   k_tab_nodes  per box of levels 1..L-1, the record the list kernels read
//                (first child, child octants, low key digits, grandchildren).
// The tile prefixes come from the scan, so no kernel waits on another tile.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t new_box_level(uint64_t k, uint64_t kp, uint32_t L) {
  const uint64_t x = k ^ kp;
  if (x == 0) return L + 1;
  const uint32_t m = (63u - (uint32_t)__clzll((long long)x)) / 3u;  // highest differing digit
  return m >= L ? 0u : L - m;
}

template <bool PACKED>
__device__ __forceinline__ uint64_t elem_key(uint64_t el) {
  return PACKED ? (el >> 32) : el;
}

// A thread's elements of a tile and the ones before them, all loaded at once:
// without a branch around any (points past the end repeat the last one), since
// a branch waits for its loads.
template <bool PACKED, int ITEMS>
__device__ __forceinline__ void load_keys(const uint64_t* __restrict__ sk, uint32_t n,
                                          uint64_t first, uint64_t (&el)[ITEMS],
                                          uint64_t (&prev)[ITEMS]) {
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint64_t e = min(first + (uint64_t)i * (kCompTile / ITEMS), (uint64_t)n - 1);
    el[i] = sk[e];
    prev[i] = sk[e - (e ? 1u : 0u)];
  }
}
// d(e), with no new box past the end.
__device__ __forceinline__ uint32_t first_level(uint64_t e, uint32_t n, uint64_t k, uint64_t kp,
                                                uint32_t L) {
  const uint32_t d = e == 0 ? 0u : new_box_level(k, kp, L);
  return e < n ? d : L + 1;
}

template <bool PACKED>
__global__ __launch_bounds__(kCompBlock) void k_tab_count(const uint64_t* __restrict__ sk,
                                                          uint32_t n, uint32_t L, uint32_t tiles,
                                                          uint32_t* __restrict__ cnt) {
  __shared__ uint32_t s_c[kMaxLevel + 1][kCompWaves];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const uint64_t tbase = (uint64_t)blockIdx.x * kCompTile;
  uint64_t key[kCompItems], kp[kCompItems];
  load_keys<PACKED, kCompItems>(sk, n, tbase + tid, key, kp);
  uint32_t d[kCompItems];
#pragma unroll
  for (int i = 0; i < kCompItems; ++i)
    d[i] = first_level(tbase + (uint64_t)i * kCompBlock + tid, n, elem_key<PACKED>(key[i]),
                       elem_key<PACKED>(kp[i]), L);
  for (uint32_t l = 0; l <= L; ++l) {
    uint32_t c = 0;
#pragma unroll
    for (int i = 0; i < kCompItems; ++i) c += (uint32_t)__popcll(__ballot(d[i] <= l));
    if (lane == 0) s_c[l][w] = c;
  }
  __syncthreads();
  if (tid <= L) {
    uint32_t c = 0;
#pragma unroll
    for (int ww = 0; ww < kCompWaves; ++ww) c += s_c[tid][ww];
    cnt[(uint64_t)tid * tiles + blockIdx.x] = c;
  }
}

// One block per level: exclusive scan of the level's tile counts, in chunks
// of 4096, and the level's box count.
constexpr int kTabScanBlock = 1024;
__global__ __launch_bounds__(kTabScanBlock) void k_tab_scan(const uint32_t* __restrict__ cnt,
                                                            uint32_t tiles,
                                                            uint32_t* __restrict__ pre,
                                                            uint32_t* __restrict__ n_boxes) {
  constexpr int W = kTabScanBlock / 64;
  __shared__ uint32_t s_w[W];
  const uint32_t l = blockIdx.x, tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  const uint32_t* c = cnt + (uint64_t)l * tiles;
  uint32_t* o = pre + (uint64_t)l * tiles;
  uint32_t carry = 0;
  for (uint64_t base = 0; base < tiles; base += 4u * kTabScanBlock) {
    uint32_t v[4], sum = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t j = base + 4u * tid + i;
      v[i] = j < tiles ? c[j] : 0u;
      sum += v[i];
    }
    const uint32_t inc = wave_incl_scan(sum);
    if (lane == 63) s_w[w] = inc;
    __syncthreads();
    uint32_t run = carry + inc - sum, total = 0;
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
      run += (uint32_t)ww < w ? s_w[ww] : 0u;
      total += s_w[ww];
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint64_t j = base + 4u * tid + i;
      if (j < tiles) o[j] = run;
      run += v[i];
    }
    carry += total;
    __syncthreads();
  }
  if (tid == 0) n_boxes[l] = carry;
}

// With a batch (set_off != nullptr) the key carries the set id from bit
// `set_shift` up and the permutation is written relative to the set's first
// point; a set boundary differs in those bits, so it starts a box at every
// level.
//
// GATHER: the coordinates follow (else they are already in place).
//
// A tile of 2048 points is 2 items a thread of 1024, or 4 of 512. Few tiles (one
// round of blocks on the chip's 256 CUs, two a CU): what bounds the kernel is
// one wave's serial chain over its items and levels, so the fewer items the
// better. 4097 points at level 3: 12.4 us with 8 items a thread, 9.2 with 4, 7.7
// with 2; 65536 at level 5: 16.3, 11.3, 9.3; two sets of 1M and 0.7M: 53, 48, 43
// together. Many tiles: the gather of the coordinates (12 random bytes a point,
// a whole line fetched each) bounds it, and blocks that start and end together
// hinder each other: a batch of 512 sets 1063 us with 8 items, 1021 with 4, 1057
// with 2; two sets of 2^24 914, 902, 896; where nothing is gathered 280, 276,
// 316.
constexpr uint32_t kTabWideTiles = 512;
template <bool PACKED, typename KeyT, bool GATHER, int BLOCK>
__global__ __launch_bounds__(BLOCK) void k_tab_write(
    const uint64_t* __restrict__ sk, const uint32_t* __restrict__ sv, const P3* __restrict__ xyz,
    uint32_t n, uint32_t L, uint32_t tiles, const uint32_t* __restrict__ cnt,
    const uint32_t* __restrict__ pre, uint32_t* __restrict__ n_boxes, TabLevels T,
    uint32_t* __restrict__ perm, P3* __restrict__ sorted_xyz,
    const uint64_t* __restrict__ set_off, uint32_t set_shift) {
  constexpr int ITEMS = kCompTile / BLOCK, WAVES = BLOCK / 64, NSLOT = ITEMS * WAVES;
  __shared__ uint32_t s_c[kMaxLevel + 1][NSLOT];
  const uint32_t tid = threadIdx.x, lane = tid & 63u, w = tid >> 6;
  // Consecutive tiles on one XCD: with a batch each set's coordinate gather
  // then stays within one XCD's L2 (the batched table pass 1550 -> 1094 us for
  // 512 sets); a single set's gather is random over all of it either way.
  const uint32_t tile = xcd_block(blockIdx.x, gridDim.x);
  const uint64_t tbase = (uint64_t)tile * kCompTile;
  uint64_t key[ITEMS], kp[ITEMS];
  uint32_t d[ITEMS], idx[ITEMS];
  float x[ITEMS], y[ITEMS], z[ITEMS];
  load_keys<PACKED, ITEMS>(sk, n, tbase + tid, key, kp);
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint64_t e = tbase + (uint64_t)i * BLOCK + tid;
    idx[i] = PACKED ? (uint32_t)key[i] : sv[min(e, (uint64_t)n - 1)];
    key[i] = elem_key<PACKED>(key[i]);
    d[i] = first_level(e, n, key[i], elem_key<PACKED>(kp[i]), L);
  }
  // (all in flight while the box starts are counted)
  if (GATHER) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const P3 p = xyz[idx[i]];
      x[i] = p.x, y[i] = p.y, z[i] = p.z;
    }
  }
  if (set_off) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) idx[i] -= (uint32_t)set_off[key[i] >> set_shift];
  }
  // per level and (item, wave) slot: the number of box starts
  for (uint32_t l = 0; l <= L; ++l) {
#pragma unroll
    for (int i = 0; i < ITEMS; ++i) {
      const uint64_t b = __ballot(d[i] <= l);
      if (lane == 0) s_c[l][i * WAVES + w] = (uint32_t)__popcll(b);
    }
  }
  __syncthreads();
  // slots in point order (item, then wave): exclusive prefixes plus the tile's
  // prefix from the scan, one level per wave at a time
  for (uint32_t l = w; l <= L; l += WAVES) {
    const uint32_t v = lane < NSLOT ? s_c[l][lane] : 0u;
    const uint32_t inc = wave_incl_scan(v);
    uint32_t before;
    if (pre) {
      before = pre[(uint64_t)l * tiles + tile];
    } else {  // at most 64 tiles: the scan of their counts is one load a lane
      const uint32_t c = lane < tile ? cnt[l * tiles + lane] : 0u;
      before = (uint32_t)__shfl((int)wave_incl_scan(c), 63, 64);
      if (tile + 1 == tiles && lane == 63) n_boxes[l] = before + inc;
    }
    if (lane < NSLOT) s_c[l][lane] = before + inc - v;
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint64_t e = tbase + (uint64_t)i * BLOCK + tid;
    if (e < n) {
      perm[e] = idx[i];
      if (GATHER) sorted_xyz[e] = P3{x[i], y[i], z[i]};
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint64_t e = tbase + (uint64_t)i * BLOCK + tid;
    const uint32_t slot = i * WAVES + w;
    // inclusive count of box starts up to this point: at level l - 1 (prev),
    // l (cur) and l + 1 (next)
    auto incl = [&](uint32_t l) {
      const bool f = d[i] <= l;
      return s_c[l][slot] + mbcnt(__ballot(f)) + (f ? 1u : 0u);
    };
    uint32_t prev = 0, cur = incl(0);
    for (uint32_t l = 0; l <= L; ++l) {
      const uint32_t next = l < L ? incl(l + 1) : 0u;
      if (e < n) {
        if (d[i] <= l) {
          const uint32_t r = cur - 1;
          ((KeyT*)T.key[l])[r] = (KeyT)(key[i] >> (3 * (L - l)));
          T.begin[l][r] = (uint32_t)e;
          if (l >= 1) T.parent[l][r] = prev - 1;
          if (l < L) T.child[l][r] = next - 1;
        }
        if (e + 1 == n) {  // sentinels: cur = boxes of level l, next = of level l + 1
          T.begin[l][cur] = n;
          if (l < L) T.child[l][cur] = next;
        }
      }
      prev = cur;
      cur = next;
    }
  }
}

// The list kernels' records of the boxes of levels 1..L-1 (device.h), from the
// boxes of level l = 0..L-2 (grid y = level): a box's i-th child's children
// give the child's octant mask and its first two words; the children's masks
// laid out as a grid are the box's own last two words. So every key is read
// once. G lanes share a box, each taking every G-th child: 8 where boxes have
// many children, 1 where most have one or two and eight lanes would idle.
template <typename KeyT, uint32_t G>
__device__ __forceinline__ void tab_nodes(const TabLevels& T, uint32_t l, uint32_t nl) {
  const uint32_t i = threadIdx.x & (G - 1u);
  const uint32_t* __restrict__ child = T.child[l];
  const uint32_t* __restrict__ child1 = T.child[l + 1];
  const KeyT* __restrict__ key1 = (const KeyT*)T.key[l + 1];
  const KeyT* __restrict__ key2 = (const KeyT*)T.key[l + 2];
  uint4* __restrict__ node = T.node[l];
  uint4* __restrict__ node1 = T.node[l + 1];
  constexpr uint32_t kBoxes = 256u / G;
  for (uint64_t j = (uint64_t)blockIdx.x * kBoxes + threadIdx.x / G; j < nl;
       j += (uint64_t)gridDim.x * kBoxes) {
    const uint32_t c0 = child[j], c1 = child[j + 1];
    uint64_t grid = 0;
    for (uint32_t c = c0 + i; c < c1; c += G) {
      const uint32_t k = (uint32_t)key1[c];
      const uint32_t g0 = child1[c], g1 = child1[c + 1];
      uint32_t m = 0;
      for (uint32_t g = g0; g < g1; ++g) m |= 1u << ((uint32_t)key2[g] & 7u);
      *(uint2*)&node1[c] = make_uint2(g0, m | (k & 63u) << 8);
      grid |= node_grid(k & 7u, m);
    }
    if (!node) continue;
    uint32_t lo = (uint32_t)grid, hi = (uint32_t)(grid >> 32);
#pragma unroll
    for (int o = 1; o < (int)G; o <<= 1) {
      lo |= (uint32_t)__shfl_xor((int)lo, o, (int)G);
      hi |= (uint32_t)__shfl_xor((int)hi, o, (int)G);
    }
    if (i == 0) ((uint2*)&node[j])[1] = make_uint2(lo, hi);
  }
}

template <typename KeyT>
__global__ __launch_bounds__(256) void k_tab_nodes(TabLevels T, uint32_t first,
                                                   const uint32_t* __restrict__ n_boxes) {
  const uint32_t l = first + blockIdx.y;
  const uint32_t nl = n_boxes[l];
  if (n_boxes[l + 1] < 3ull * nl) tab_nodes<KeyT, 1>(T, l, nl);
  else tab_nodes<KeyT, 8>(T, l, nl);
}

void launch_nodes(bool key64, const TabLevels& T, uint32_t first, uint32_t levels,
                  const uint32_t* n_boxes, uint32_t node_cap, hipStream_t s) {
  const dim3 grid(std::max<uint32_t>(1, std::min<uint32_t>(div_up(node_cap, 32), 2048)), levels);
  if (key64) hipLaunchKernelGGL(k_tab_nodes<uint64_t>, grid, dim3(256), 0, s, T, first, n_boxes);
  else hipLaunchKernelGGL(k_tab_nodes<uint32_t>, grid, dim3(256), 0, s, T, first, n_boxes);
}

uint32_t tab_tiles(uint32_t n) { return div_up(n, kCompTile); }

void launch_tables(bool packed, bool key64, const uint64_t* sk, const uint32_t* sv,
                   const float* xyz, uint32_t n, uint32_t L, uint32_t* cnt, uint32_t* pre,
                   const TabLevels& T, uint32_t* perm, float* sorted_xyz, uint32_t* n_boxes,
                   uint32_t node_cap, hipStream_t s, int phase, const uint64_t* set_off,
                   uint32_t set_shift) {
  const uint32_t tiles = tab_tiles(n);
  if (phase == 0) {
    if (packed)
      hipLaunchKernelGGL(k_tab_count<true>, dim3(tiles), dim3(kCompBlock), 0, s, sk, n, L, tiles, cnt);
    else
      hipLaunchKernelGGL(k_tab_count<false>, dim3(tiles), dim3(kCompBlock), 0, s, sk, n, L, tiles, cnt);
  } else if (phase == 1) {
    if (tiles > kTabSmallTiles)
      hipLaunchKernelGGL(k_tab_scan, dim3(L + 1), dim3(kTabScanBlock), 0, s, cnt, tiles, pre, n_boxes);
  } else if (phase == 2) {
#define FMMDS_TABWB(P, K, B)                                                                     \
  hipLaunchKernelGGL((xyz ? k_tab_write<P, K, true, B> : k_tab_write<P, K, false, B>),           \
                     dim3(tiles), dim3(B), 0, s, sk, sv, (const P3*)xyz, n, L, tiles, cnt,       \
                     tiles > kTabSmallTiles ? pre : nullptr, n_boxes, T, perm, (P3*)sorted_xyz,  \
                     set_off, set_shift)
#define FMMDS_TABW(P, K)                                                                         \
  do {                                                                                           \
    if (tiles <= kTabWideTiles) FMMDS_TABWB(P, K, 1024);                                         \
    else FMMDS_TABWB(P, K, 512);                                                                 \
  } while (0)
    if (packed && key64) FMMDS_TABW(true, uint64_t);
    else if (packed) FMMDS_TABW(true, uint32_t);
    else if (key64) FMMDS_TABW(false, uint64_t);
    else FMMDS_TABW(false, uint32_t);
#undef FMMDS_TABW
#undef FMMDS_TABWB
  } else if (L >= 2) {
    launch_nodes(key64, T, 0, L - 1, n_boxes, node_cap, s);
  }
}

// ---------------------------------------------------------------------------
// K8: largest box occupancy of every level 2..L (for the cluster-size depth
// rule, Section 2.1), all levels in one launch (grid y = level - 2).
// ---------------------------------------------------------------------------
// A block takes 4096 consecutive boxes, its loads all made at once (indices
// clamped to the sentinel, which give 0). What bounds it is the atomics on each
// level's one word, which are serialized: one per block, and only where the
// block's maximum is above the word as it stands (a stale word is a lower one,
// so none is missed). Two sets of 2^24 clustered points, levels 2..10: 18
// launches 166 us, two launches 97 us; one set of 2M points, levels 2..13: 100 us,
// now 46.
constexpr int kOccItems = 16;

__global__ __launch_bounds__(256) void k_max_occupancy(OccLevels lv,
                                                       const uint32_t* __restrict__ n_boxes,
                                                       uint32_t* max_occ) {
  const uint32_t l = blockIdx.y + 2, n = n_boxes[l];
  const uint32_t* __restrict__ begin = lv.begin[l];
  const uint64_t j0 = (uint64_t)blockIdx.x * (256u * kOccItems) + threadIdx.x;
  if ((uint64_t)blockIdx.x * (256u * kOccItems) >= n) return;  // whole block
  uint32_t b0[kOccItems], b1[kOccItems], m = 0;
#pragma unroll
  for (int i = 0; i < kOccItems; ++i) {
    const uint64_t j = j0 + 256u * (uint32_t)i;
    b0[i] = begin[min(j, (uint64_t)n)];
    b1[i] = begin[min(j + 1, (uint64_t)n)];
  }
#pragma unroll
  for (int i = 0; i < kOccItems; ++i) m = max(m, b1[i] - b0[i]);
  __shared__ uint32_t s_m[4];
  m = wave_max(m);
  if ((threadIdx.x & 63) == 0) s_m[threadIdx.x >> 6] = m;
  __syncthreads();
  if (threadIdx.x == 0) {
    m = max(max(s_m[0], s_m[1]), max(s_m[2], s_m[3]));
    if (m > __hip_atomic_load(&max_occ[l], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
      atomicMax(&max_occ[l], m);
  }
}

void launch_max_occupancy(const OccLevels& lv, uint32_t L, uint32_t cap, const uint32_t* n_boxes,
                          uint32_t* max_occ, hipStream_t s) {
  if (L < 2) return;
  const dim3 grid(std::max<uint32_t>(1, div_up(cap, 256u * kOccItems)), L - 1);
  hipLaunchKernelGGL(k_max_occupancy, grid, dim3(256), 0, s, lv, n_boxes, max_occ);
}

}  // namespace fmmds
