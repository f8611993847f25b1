// Key generation and LSD radix sort of (Morton key, point index) pairs.
//
// The paper reorders points by the Morton index of their finest-level box
// with a histogram pseudo-sort whose order inside a box depends on atomic
// timing (Section 2.1, Algorithm 1). This library needs a deterministic order,
// so it sorts (key, original index) pairs stably: an LSD radix sort with 8-bit
// digits, one single-pass "chained scan" kernel per digit.
#include "device.h"
#include "internal.h"

namespace fmmds {

// ---------------------------------------------------------------------------
// Zero fill (a kernel, so that it can sit inside a captured graph).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void k_zero(uint4* __restrict__ p, size_t n16) {
  const uint4 z = make_uint4(0, 0, 0, 0);
  for (size_t i = blockIdx.x * 256ull + threadIdx.x; i < n16; i += (size_t)gridDim.x * 256)
    p[i] = z;
}

void launch_zero(void* p, size_t bytes, hipStream_t s) {
  // Every region handed to this function is 16-byte aligned and sized.
  const size_t n16 = bytes / 16;
  if (n16 == 0) return;
  const uint32_t grid = (uint32_t)std::min<size_t>(div_up(n16, 256), 4096);
  hipLaunchKernelGGL(k_zero, dim3(grid), dim3(256), 0, s, (uint4*)p, n16);
}

// ---------------------------------------------------------------------------
// K1: Morton key of every point (Section 1.4 box index, Section 2.4
// interleave) plus the digit histograms of every sort pass.
//
// A point (x, y, z) is in the box floor(x * 2^L) per axis; x * 2^L is exact in
// FP32. Coordinates outside [0, 1) (or NaN) raise the range flag; such points
// get box 0 so that later kernels stay in bounds, and the build reports the
// error.
// ---------------------------------------------------------------------------
struct P3 {
  float x, y, z;
};

// Each thread loads kKeyItems points (one 64-point run per wave and item,
// all issued before any is used), so the loads of a block are in flight
// together rather than one per loop trip. Each block writes its digit
// histograms as one row (no atomics: thousands of blocks adding into the same
// 256 bins per pass serialize on those addresses); the digit-offset kernel
// adds the rows.
constexpr int kKeyItems = 8;
constexpr int kKeyChunk = 256 * kKeyItems;
constexpr uint32_t kKeyMaxBlocks = 4096;

template <bool PACKED>
__global__ __launch_bounds__(256) void k_keygen(const P3* __restrict__ xyz, uint32_t n, uint32_t L,
                                                uint64_t* __restrict__ keys,
                                                uint32_t* __restrict__ vals, uint32_t n_pass,
                                                uint32_t* __restrict__ rows,
                                                uint32_t* __restrict__ err) {
  __shared__ uint32_t s_hist[kMaxPasses * 256];
  for (uint32_t i = threadIdx.x; i < n_pass * 256; i += 256) s_hist[i] = 0;
  __syncthreads();
  bool bad = false;
  for (uint64_t base = (uint64_t)blockIdx.x * kKeyChunk; base < n;
       base += (uint64_t)gridDim.x * kKeyChunk) {
    P3 p[kKeyItems];
#pragma unroll
    for (int j = 0; j < kKeyItems; ++j) {
      const uint64_t i = base + (uint64_t)j * 256 + threadIdx.x;
      p[j] = i < n ? xyz[i] : P3{0.f, 0.f, 0.f};
    }
#pragma unroll
    for (int j = 0; j < kKeyItems; ++j) {
      const uint64_t i = base + (uint64_t)j * 256 + threadIdx.x;
      if (i >= n) continue;
      bool ok;
      const uint64_t key = point_key(p[j].x, p[j].y, p[j].z, L, ok);
      bad |= !ok;
      if (PACKED) {
        if (keys) keys[i] = (key << 32) | (uint32_t)i;
      } else {
        keys[i] = key;
        vals[i] = (uint32_t)i;
      }
      for (uint32_t p8 = 0; p8 < n_pass; ++p8)
        atomicAdd(&s_hist[p8 * 256 + ((key >> (8 * p8)) & 0xFF)], 1u);
    }
  }
  if (bad) atomicOr(err, 1u);
  __syncthreads();
  uint32_t* row = rows + (uint64_t)blockIdx.x * n_pass * 256;
  for (uint32_t i = threadIdx.x; i < n_pass * 256; i += 256) row[i] = s_hist[i];
}

uint32_t keygen_blocks(uint32_t n) {
  return std::max<uint32_t>(1, std::min<uint32_t>(div_up(n, kKeyChunk), kKeyMaxBlocks));
}

void launch_keygen(const float* xyz, uint32_t n, uint32_t L, bool packed, uint64_t* keys,
                   uint32_t* vals, uint32_t n_pass, uint32_t* rows, uint32_t* err,
                   hipStream_t s) {
  const uint32_t grid = keygen_blocks(n);
  if (packed)
    hipLaunchKernelGGL(k_keygen<true>, dim3(grid), dim3(256), 0, s, (const P3*)xyz, n, L, keys,
                       vals, n_pass, rows, err);
  else
    hipLaunchKernelGGL(k_keygen<false>, dim3(grid), dim3(256), 0, s, (const P3*)xyz, n, L, keys,
                       vals, n_pass, rows, err);
}

// Keygen's per-block rows added into the zeroed pass histograms: block
// (b, p) adds rows b, b + gridDim.x, ... of pass p, then one atomic per bin
// (a few dozen per address instead of one per keygen block).
constexpr uint32_t kRowReduceBlocks = 64;
__global__ __launch_bounds__(256) void k_reduce_rows(const uint32_t* __restrict__ rows,
                                                     uint32_t n_rows, uint32_t n_pass,
                                                     uint32_t* __restrict__ hist) {
  const uint32_t p = blockIdx.y, d = threadIdx.x, G = gridDim.x;
  uint32_t c = 0, r = blockIdx.x;
  // eight rows' loads in flight per round
  for (; r + 7 * G < n_rows; r += 8 * G) {
    uint32_t v[8];
#pragma unroll
    for (uint32_t t = 0; t < 8; ++t) v[t] = rows[((uint64_t)(r + t * G) * n_pass + p) * 256 + d];
#pragma unroll
    for (uint32_t t = 0; t < 8; ++t) c += v[t];
  }
  for (; r < n_rows; r += G) c += rows[((uint64_t)r * n_pass + p) * 256 + d];
  if (c) atomicAdd(&hist[p * 256 + d], c);
}

void launch_reduce_rows(const uint32_t* rows, uint32_t n_rows, uint32_t* hist, uint32_t n_pass,
                        hipStream_t s) {
  const dim3 grid(std::min(kRowReduceBlocks, n_rows), n_pass);
  hipLaunchKernelGGL(k_reduce_rows, grid, dim3(256), 0, s, rows, n_rows, n_pass, hist);
}

// Exclusive scan of each pass's 256-bin histogram: where digit d starts.
__global__ __launch_bounds__(256) void k_digit_offsets(const uint32_t* __restrict__ hist,
                                                       uint32_t* __restrict__ goff) {
  __shared__ uint32_t s_w[4];
  const uint32_t p = blockIdx.x, d = threadIdx.x, lane = d & 63, w = d >> 6;
  const uint32_t c = hist[p * 256 + d];
  const uint32_t inc = wave_incl_scan(c);
  if (lane == 63) s_w[w] = inc;
  __syncthreads();
  uint32_t base = 0;
  for (uint32_t i = 0; i < w; ++i) base += s_w[i];
  goff[p * 256 + d] = base + inc - c;
}

void launch_digit_offsets(const uint32_t* hist, uint32_t* goff, uint32_t n_pass, hipStream_t s) {
  hipLaunchKernelGGL(k_digit_offsets, dim3(n_pass), dim3(256), 0, s, hist, goff);
}

// The same from keygen's rows where there are few of them: block p adds pass p's
// rows and scans the sums (one launch less; 2048 points a row, so up to 131072).
__global__ __launch_bounds__(256) void k_digit_offsets_rows(const uint32_t* __restrict__ rows,
                                                            uint32_t n_rows, uint32_t n_pass,
                                                            uint32_t* __restrict__ goff) {
  __shared__ uint32_t s_w[4];
  const uint32_t p = blockIdx.x, d = threadIdx.x, lane = d & 63, w = d >> 6;
  uint32_t c = 0;
#pragma unroll 8
  for (uint32_t r = 0; r < n_rows; ++r) c += rows[((uint64_t)r * n_pass + p) * 256 + d];
  const uint32_t inc = wave_incl_scan(c);
  if (lane == 63) s_w[w] = inc;
  __syncthreads();
  uint32_t base = 0;
  for (uint32_t i = 0; i < w; ++i) base += s_w[i];
  goff[p * 256 + d] = base + inc - c;
}

constexpr uint32_t kDigitRows = 64;

void launch_digits(const uint32_t* rows, uint32_t n_rows, uint32_t* hist, uint32_t* goff,
                   uint32_t n_pass, hipStream_t s) {
  if (n_rows <= kDigitRows) {
    hipLaunchKernelGGL(k_digit_offsets_rows, dim3(n_pass), dim3(256), 0, s, rows, n_rows, n_pass,
                       goff);
  } else {
    launch_reduce_rows(rows, n_rows, hist, n_pass, s);
    launch_digit_offsets(hist, goff, n_pass, s);
  }
}

// ---------------------------------------------------------------------------
// K2: one stable LSD pass on the 8-bit digit at `shift`.
//
// A tile of BLOCK * ITEMS elements is split into contiguous 64 * ITEMS-element
// wave segments, loaded 64 at a time (coalesced). Each wave ranks its
// elements by digit with eight ballots per element (lanes whose digit agrees
// on every bit), keeping running per-digit counts in LDS, so ranks follow
// input order. The tile's 256 digit counts are then chained across tiles by
// decoupled look-back (thread d < 256 owns digit d), the tile is staged in
// LDS in digit order, and written out so that consecutive threads store
// consecutive addresses of one digit's run. The look-back chain is what sets
// the pass's length (without it a 4096-element pass over 2^24 elements takes
// ~75 us instead of ~125 us), so each tile publishes its digit counts (LDS
// atomics) before it ranks, large sets take tiles of 8192 elements, which
// halve the chain of 4096-element tiles, and each digit's walk loads four
// predecessors' words at a time.
// ---------------------------------------------------------------------------
// The 8-bit digit at `shift`. A packed element holds the key in its high
// word, and its passes start at shift 32.
template <bool PACKED>
__device__ __forceinline__ uint32_t sort_digit(uint64_t k, uint32_t shift) {
  return PACKED ? __builtin_amdgcn_ubfe((uint32_t)(k >> 32), shift - 32u, 8u)
                : (uint32_t)(k >> shift) & 0xFFu;
}

// Ranks of a wave's items (64 of each i, in order) by the digit at `shift` within
// the wave's own items: item i of this lane is valid while 64 i + lane < lim;
// `hist` (256 words, zeroed) ends with the wave's digit counts.
template <bool PACKED, int ITEMS, typename H>
__device__ __forceinline__ void sort_rank(const uint64_t (&k)[ITEMS], uint32_t shift, uint32_t lim,
                                          uint32_t lane, H* hist, uint32_t (&r)[ITEMS]) {
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const bool valid = 64u * i + lane < lim;
    const uint32_t d = sort_digit<PACKED>(k[i], shift);
    // peers: the valid lanes whose digit equals this lane's. Per bit b, m is
    // all ones where this lane's bit is 0, so that (ballot ^ m) keeps the
    // lanes that agree with it on bit b (one three-input bit op per half).
    const uint64_t vb = __ballot(valid);
    uint32_t plo = (uint32_t)vb, phi = (uint32_t)(vb >> 32);
    const uint32_t nd = ~d;
#pragma unroll
    for (int b = 0; b < 8; ++b) {
      const uint32_t m = (uint32_t)__builtin_amdgcn_sbfe((int)nd, b, 1);
      const uint64_t bal = __ballot(m == 0u);
      plo &= (uint32_t)bal ^ m;
      phi &= (uint32_t)(bal >> 32) ^ m;
    }
    const uint32_t below = __builtin_amdgcn_mbcnt_hi(phi, __builtin_amdgcn_mbcnt_lo(plo, 0u));
    uint32_t prev = 0;
    if (valid) prev = hist[d];
    r[i] = prev + below;
    if (valid && below == 0) hist[d] = (H)(prev + (uint32_t)(__popc(plo) + __popc(phi)));
  }
}

// With SEG, tiles come from a set-aligned table (SegSort): each tile lies in
// one set, a set's first tile starts its own look-back chain, and the digit
// offsets are that set's, so every set is sorted within its own range.
template <bool PACKED, int BLOCK, int ITEMS, bool SEG>
__global__ __launch_bounds__(BLOCK) void k_sort_pass(
    const uint64_t* __restrict__ kin, uint64_t* __restrict__ kout, const uint32_t* __restrict__ vin,
    uint32_t* __restrict__ vout, uint32_t n_host, uint32_t shift, const uint32_t* __restrict__ goff,
    uint64_t* __restrict__ status, uint32_t* __restrict__ tile_counter,
    const uint32_t* __restrict__ n_dev, SegSort sg) {
  static_assert(BLOCK >= 256, "thread d owns digit d");
  constexpr int W = BLOCK / 64;
  constexpr int TILE = BLOCK * ITEMS;
  constexpr int WSEG = 64 * ITEMS;
  __shared__ uint64_t s_key[TILE];
  __shared__ uint32_t s_val[PACKED ? 1 : TILE];
  __shared__ uint32_t s_hist[W][256];
  __shared__ uint32_t s_cnt[256];  // the tile's digit counts, published before the ranking
  __shared__ uint32_t s_lstart[256];
  __shared__ uint32_t s_base[256];
  __shared__ uint32_t s_scan[4];
  __shared__ uint32_t s_tile;

  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) s_tile = atomicAdd(tile_counter, 1u);
  for (uint32_t i = tid; i < W * 256; i += BLOCK) (&s_hist[0][0])[i] = 0;
  if (tid < 256) s_cnt[tid] = 0;
  __syncthreads();
  const uint32_t tile = __builtin_amdgcn_readfirstlane(s_tile);
  uint64_t tbase, tend;
  bool first;
  const uint32_t* __restrict__ go = goff;
  if (SEG) {
    tbase = sg.start[tile];
    tend = sg.start[tile + 1];
    const uint32_t sw = sg.set[tile];
    first = (sw >> 31) != 0;
    go = sg.goff + ((uint64_t)(sw & 0x7FFFFFFFu) * sg.n_pass + sg.pass) * 256;
  } else {
    const uint32_t n = n_dev ? *n_dev : n_host;
    // With the count on the device the grid covers the capacity; tiles past
    // the count exit (tiles only look back at lower tile ids).
    if ((uint64_t)tile * TILE >= n && tile > 0) return;
    tbase = (uint64_t)tile * TILE;
    tend = min(tbase + TILE, (uint64_t)n);
    first = tile == 0;
  }
  const uint64_t wbase = tbase + (uint64_t)w * WSEG;
  // Item i of this lane is element wbase + 64 i + lane, valid while
  // 64 i + lane < lim (32-bit tests; the wave's base pointer is uniform).
  const uint32_t lim = (uint32_t)min((uint64_t)WSEG, tend > wbase ? tend - wbase : 0ull);
  const uint64_t* __restrict__ kw = kin + wbase;
  const uint32_t* __restrict__ vw = PACKED ? nullptr : vin + wbase;

  uint64_t k[ITEMS];
  uint32_t v[ITEMS];
  uint32_t r[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t j = 64u * i + lane;
    k[i] = j < lim ? kw[j] : 0;
    if (!PACKED) v[i] = j < lim ? vw[j] : 0;
  }
  // The tile's digit counts first (LDS atomics), published at once, so that
  // later tiles' look-backs find them while this tile still ranks.
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (64u * i + lane < lim) atomicAdd(&s_cnt[sort_digit<PACKED>(k[i], shift)], 1u);
  __syncthreads();
  if (tid < 256) {
    const uint64_t agg = s_cnt[tid];
    st_status(status + (uint64_t)tile * 256 + tid, (first ? kStInc : kStAgg) | agg);
  }
  sort_rank<PACKED, ITEMS>(k, shift, lim, lane, s_hist[w], r);
  __syncthreads();

  // Thread d < 256 owns digit d: wave-exclusive prefixes, tile count, local
  // start, then the tile's global base by look-back.
  uint32_t cnt = 0, inc = 0;
  if (tid < 256) {
    uint32_t run = 0;
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
      const uint32_t c = s_hist[ww][tid];
      s_hist[ww][tid] = run;
      run += c;
    }
    cnt = run;
    inc = wave_incl_scan(cnt);
    if (lane == 63) s_scan[w] = inc;
  }
  __syncthreads();
  if (tid < 256) {
    const uint32_t d = tid;
    uint32_t wpre = 0;
    for (uint32_t ww = 0; ww < w; ++ww) wpre += s_scan[ww];
    const uint32_t lstart = wpre + inc - cnt;
    s_lstart[d] = lstart;
    const uint64_t excl = first ? 0 : lookback_window<4>(status + d, 256, tile, cnt);
    s_base[d] = go[d] + (uint32_t)excl - lstart;
  }
  __syncthreads();

#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (64u * i + lane < lim) {
      const uint32_t dd = sort_digit<PACKED>(k[i], shift);
      const uint32_t lp = s_lstart[dd] + s_hist[w][dd] + r[i];
      s_key[lp] = k[i];
      if (!PACKED) s_val[lp] = v[i];
    }
  }
  __syncthreads();
  const uint32_t tcount = (uint32_t)(tend - tbase);
  for (uint32_t j = tid; j < tcount; j += BLOCK) {
    const uint64_t kk = s_key[j];
    const uint32_t dd = sort_digit<PACKED>(kk, shift);
    const uint32_t g = s_base[dd] + j;
    kout[g] = kk;
    if (!PACKED) vout[g] = s_val[j];
  }
}

// ---------------------------------------------------------------------------
// Small sets: keys and every pass in one block, which keeps its elements in
// registers and turns them over in LDS between the passes. Key generation, the
// digit counts (two launches) and each pass are launches of their own otherwise,
// a few us apiece whatever their size: 4097 points at level 3 (two passes) took
// 28 us of kernels and four gaps of about 4 us, and take 15 us here. What bounds
// it is the serial chain of each wave's ranks, so that the time grows with the
// items a wave holds; larger sets spread over blocks.
// ---------------------------------------------------------------------------
template <int BLOCK, int ITEMS>
__global__ __launch_bounds__(BLOCK) void k_sort_small(const P3* __restrict__ xyz, uint32_t n,
                                                    uint32_t L, uint32_t n_pass,
                                                    uint64_t* __restrict__ out,
                                                    uint32_t* __restrict__ err) {
  constexpr int W = BLOCK / 64;
  constexpr uint32_t WSEG = 64 * ITEMS;
  __shared__ uint64_t s_key[BLOCK * ITEMS];
  __shared__ uint32_t s_hist[W][256];
  __shared__ uint32_t s_lstart[256];
  __shared__ uint32_t s_scan[4];
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const uint32_t wbase = w * WSEG;
  const uint32_t lim = n > wbase ? min(WSEG, n - wbase) : 0u;
  uint64_t k[ITEMS];
  bool bad = false;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    const uint32_t j = 64u * i + lane;
    k[i] = 0;
    if (j < lim) {
      const P3 p = xyz[wbase + j];
      bool ok;
      k[i] = point_key(p.x, p.y, p.z, L, ok) << 32 | (wbase + j);
      bad |= !ok;
    }
  }
  if (bad) atomicOr(err, 1u);
  for (uint32_t p = 0; p < n_pass; ++p) {
    const uint32_t shift = 32 + 8 * p;
    for (uint32_t i = tid; i < W * 256; i += BLOCK) (&s_hist[0][0])[i] = 0;
    __syncthreads();
    uint32_t r[ITEMS];
    sort_rank<true, ITEMS>(k, shift, lim, lane, s_hist[w], r);
    __syncthreads();
    uint32_t cnt = 0, inc = 0;
    if (tid < 256) {
#pragma unroll
      for (int ww = 0; ww < W; ++ww) {
        const uint32_t c = s_hist[ww][tid];
        s_hist[ww][tid] = cnt;
        cnt += c;
      }
      inc = wave_incl_scan(cnt);
      if (lane == 63) s_scan[w] = inc;
    }
    __syncthreads();
    if (tid < 256) {
      uint32_t wpre = 0;
      for (uint32_t ww = 0; ww < w; ++ww) wpre += s_scan[ww];
      s_lstart[tid] = wpre + inc - cnt;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (64u * i + lane < lim) {
        const uint32_t d = sort_digit<true>(k[i], shift);
        s_key[s_lstart[d] + s_hist[w][d] + r[i]] = k[i];
      }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < ITEMS; ++i)
      if (64u * i + lane < lim) k[i] = s_key[wbase + 64u * i + lane];
    // (the next pass writes s_key after two more barriers)
  }
#pragma unroll
  for (int i = 0; i < ITEMS; ++i)
    if (64u * i + lane < lim) out[wbase + 64u * i + lane] = k[i];
}

void launch_sort_small(const float* xyz, uint32_t n, uint32_t L, uint32_t n_pass, uint64_t* out,
                       uint32_t* err, hipStream_t s) {
#define FMMDS_SMALL(B, I)                                                                        \
  hipLaunchKernelGGL((k_sort_small<B, I>), dim3(1), dim3(B), 0, s, (const P3*)xyz, n, L, n_pass, \
                     out, err)
  if (n <= 2048) FMMDS_SMALL(512, 4);
  else if (n <= 4096) FMMDS_SMALL(1024, 4);
  else FMMDS_SMALL(1024, 8);
#undef FMMDS_SMALL
}

// ---------------------------------------------------------------------------
// Large sets: the passes move the points themselves (coordinates and index, 16
// bytes; the key is computed anew), so that the last one leaves coordinates and
// sorted elements in order. Moving (key, index) alone is half the bytes, but the
// coordinates then have to be gathered by index at the end: 12 random bytes a
// point, a whole line fetched for each (2^24 points at level 8: keys 86 us, three
// passes of 91, tables with the gather 451; here keys 69, passes of 161 on
// average, tables 127). FIRST reads the points as they are given, LAST writes the
// results instead of records. What bounds it is memory: two chains of passes
// together move 3.4 (FIRST) to 3.9 TB/s (a plain copy 4.8). Tiles of 8192 leave
// runs of 512 bytes per digit, one tile a CU; with tiles of 4096 and two tiles a
// CU the build of 2 x 2^24 points took 3835 us, with these 3790 (by elements
// 4005).
// ---------------------------------------------------------------------------
// Builds (us, by records / by elements). Three passes, one set at level 6 of 2^20
// points 249 / 244, 2^21 288 / 297, 2^24 831 / 921; at level 8 2^20 604 / 597, 2^21
// 977 / 993, 2^24 3103 / 3180. Four passes (levels 9 and 10) move so much more that
// one set gains nothing for twice the memory: at level 10 uniform 3 * 2^20 points
// 2871 / 2864, 2^23 6193 / 6218, 2^24 11896 / 11914, clustered 2^23 1741 / 1761, 2^24
// 2571 / 2589. Two sets, whose chains of passes share the chip, gain a little:
// clustered at level 10 2 x 2^22 and a quarter more 1655 / 1647, 2 x 2^23 2183 /
// 2199, 2 x 3 * 2^22 2801 / 2856, 2 x 2^24 3359 / 3450.
constexpr uint32_t kRecMin = 1u << 20, kRecMin4 = 1u << 22;
bool sort_by_records(uint32_t n, uint32_t n_pass, bool two_sets) {
  if (n_pass < 2) return false;
  return n_pass <= 3 ? n > kRecMin : two_sets && n > kRecMin4;
}

constexpr int kRecBlock = 1024, kRecItems = 8, kRecTile = kRecBlock * kRecItems;

__device__ __forceinline__ uint64_t record_key(uint4 q, uint32_t L) {
  bool ok;
  return point_key(__uint_as_float(q.x), __uint_as_float(q.y), __uint_as_float(q.z), L, ok) << 32;
}

template <bool FIRST, bool LAST>
__global__ __launch_bounds__(kRecBlock) void k_sort_records(
    const uint32_t* __restrict__ xyz, const uint4* __restrict__ rin, uint4* __restrict__ rout,
    uint32_t* __restrict__ sorted_xyz, uint64_t* __restrict__ kout, uint32_t n, uint32_t L,
    uint32_t shift, const uint32_t* __restrict__ goff,
    uint64_t* __restrict__ status, uint32_t* __restrict__ tile_counter) {
  constexpr int W = kRecBlock / 64;
  constexpr uint32_t WSEG = 64 * kRecItems;
  __shared__ uint4 s_rec[kRecTile];
  __shared__ uint16_t s_hist[W][256];
  __shared__ uint32_t s_cnt[256], s_lstart[256], s_base[256];
  __shared__ uint32_t s_scan[4];
  __shared__ uint32_t s_tile;
  const uint32_t tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  if (tid == 0) s_tile = atomicAdd(tile_counter, 1u);
  for (uint32_t i = tid; i < W * 128; i += kRecBlock) ((uint32_t*)s_hist)[i] = 0;
  if (tid < 256) s_cnt[tid] = 0;
  __syncthreads();
  const uint32_t tile = __builtin_amdgcn_readfirstlane(s_tile);
  const uint32_t tbase = tile * kRecTile;
  const uint32_t tcount = min((uint32_t)kRecTile, n - tbase);
  const uint32_t wbase = w * WSEG;
  const uint32_t lim = tcount > wbase ? min(WSEG, tcount - wbase) : 0u;

  uint4 q[kRecItems];
  uint64_t k[kRecItems];
  uint32_t r[kRecItems];
#pragma unroll
  for (int i = 0; i < kRecItems; ++i) {
    const uint32_t e = tbase + min(wbase + 64u * i + lane, tcount - 1);  // (past the end: the last)
    if (FIRST) {
      const uint32_t* p = xyz + 3ull * e;
      q[i] = make_uint4(p[0], p[1], p[2], e);
    } else {
      q[i] = rin[e];
    }
  }
#pragma unroll
  for (int i = 0; i < kRecItems; ++i) {
    k[i] = record_key(q[i], L);
    if (64u * i + lane < lim) atomicAdd(&s_cnt[sort_digit<true>(k[i], shift)], 1u);
  }
  __syncthreads();
  if (tid < 256)
    st_status(status + (uint64_t)tile * 256 + tid,
              (tile == 0 ? kStInc : kStAgg) | (uint64_t)s_cnt[tid]);
  sort_rank<true, kRecItems>(k, shift, lim, lane, s_hist[w], r);
  __syncthreads();
  uint32_t cnt = 0, inc = 0;
  if (tid < 256) {
#pragma unroll
    for (int ww = 0; ww < W; ++ww) {
      const uint32_t c = s_hist[ww][tid];
      s_hist[ww][tid] = (uint16_t)cnt;
      cnt += c;
    }
    inc = wave_incl_scan(cnt);
    if (lane == 63) s_scan[w] = inc;
  }
  __syncthreads();
  if (tid < 256) {
    uint32_t wpre = 0;
    for (uint32_t ww = 0; ww < w; ++ww) wpre += s_scan[ww];
    const uint32_t lstart = wpre + inc - cnt;
    s_lstart[tid] = lstart;
    const uint64_t excl = tile == 0 ? 0 : lookback_window<4>(status + tid, 256, tile, cnt);
    s_base[tid] = goff[tid] + (uint32_t)excl - lstart;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kRecItems; ++i) {
    if (64u * i + lane < lim) {
      const uint32_t d = sort_digit<true>(k[i], shift);
      s_rec[s_lstart[d] + s_hist[w][d] + r[i]] = q[i];
    }
  }
  __syncthreads();
#pragma unroll 2
  for (uint32_t j = tid; j < tcount; j += kRecBlock) {
    const uint4 v = s_rec[j];
    const uint64_t key = record_key(v, L);
    const uint32_t g = s_base[sort_digit<true>(key, shift)] + j;
    if (LAST) {
      uint32_t* o = sorted_xyz + 3ull * g;
      o[0] = v.x, o[1] = v.y, o[2] = v.z;
      kout[g] = key | v.w;
    } else {
      rout[g] = v;
    }
  }
}

uint32_t record_tiles(uint32_t n) { return div_up(n, kRecTile); }

void launch_sort_records(const float* xyz, const uint4* rin, uint4* rout, float* sorted_xyz,
                         uint64_t* kout, uint32_t n, uint32_t L, uint32_t shift,
                         const uint32_t* goff, uint64_t* status, uint32_t* tile_counter,
                         hipStream_t s) {
#define FMMDS_REC(A, B)                                                                         \
  hipLaunchKernelGGL((k_sort_records<A, B>), dim3(record_tiles(n)), dim3(kRecBlock), 0, s,      \
                     (const uint32_t*)xyz, rin, rout, (uint32_t*)sorted_xyz, kout, n, L,  \
                     shift, goff, status, tile_counter)
  if (!rin) FMMDS_REC(true, false);
  else if (kout) FMMDS_REC(false, true);
  else FMMDS_REC(false, false);
#undef FMMDS_REC
}

uint32_t sort_tile_elems(int items) { return 256u * (uint32_t)items; }

// Fewer, larger tiles shorten the look-back chain and write longer runs; more
// tiles spread a small set over more CUs (there are 256). us per pass, packed
// elements (tiles of 2048 / 4096 / 8192): 65536 elements 10.1 / 11.2 / 14.7,
// 200000 12.1 / 12.5 / 15.6, 500000 15.8 / 14.9 / 17.5, 10^6 23.2 / 19.0 / 19.8,
// 2 * 10^6 34.2 / 26.0 / 24.0; key and index apart: 65536 10.6 / 11.7 / 14.9,
// 500000 17.0 / 16.2 / 18.2, 10^6 24.5 / 20.3 / 21.0, 4 * 10^6 59 / 43 / 41.
constexpr uint32_t kSortSmallTiles = 1u << 18, kSortMidTiles = 1u << 20;
int sort_items(uint32_t n) {
  return n <= kSortSmallTiles ? 8 : n <= kSortMidTiles ? kSortItemsDefault : kSortWide;
}
uint32_t sort_tiles_max(uint32_t n) {
  uint32_t t = sort_tiles(n, sort_items(n));
  if (n > kSortSmallTiles) t = std::max(t, sort_tiles(kSortSmallTiles, 8));
  if (n > kSortMidTiles) t = std::max(t, sort_tiles(kSortMidTiles, kSortItemsDefault));
  return t;
}

uint32_t sort_tiles(uint32_t n, int items) { return div_up(n, sort_tile_elems(items)); }

template <bool SEG>
void sort_pass_dispatch(bool packed, const uint64_t* kin, uint64_t* kout, const uint32_t* vin,
                        uint32_t* vout, uint32_t n, uint32_t grid, uint32_t shift,
                        const uint32_t* goff, uint64_t* status, uint32_t* tile_counter,
                        hipStream_t s, int items, const uint32_t* n_dev, const SegSort& sg) {
#define FMMDS_SORT(P, B, I)                                                                     \
  hipLaunchKernelGGL((k_sort_pass<P, B, I, SEG>), dim3(grid), dim3(B), 0, s, kin, kout, vin,   \
                     vout, n, shift, goff, status, tile_counter, n_dev, sg)
#define FMMDS_SORT2(B, I)                                                                       \
  do {                                                                                           \
    if (packed) FMMDS_SORT(true, B, I);                                                          \
    else FMMDS_SORT(false, B, I);                                                                \
  } while (0)
  // 1024 threads a tile: a wave ranks its items one after the other, so fewer
  // items a thread are a shorter tile (us per pass with 256 threads: tiles of
  // 2048 14.7 -> 10.1 at 65536 elements, 55.5 -> 54.3 at 4 * 10^6; of 4096 41.1
  // -> 39.2). Large tiles of packed elements stay at 512 threads, whose LDS
  // leaves room for two tiles a CU (2^24 elements: 91 us a pass, 116 with 1024);
  // with the index apart (153 us a pass in tiles of 4096 by 256) there is room
  // for one either way, 137 us.
  if (items == kSortWide && packed) FMMDS_SORT(true, 512, 16);
  else if (items == kSortWide) FMMDS_SORT(false, 1024, 8);
  else if (items == 8) FMMDS_SORT2(1024, 2);
  else if (items == 12) FMMDS_SORT2(1024, 3);
  else FMMDS_SORT2(1024, 4);
#undef FMMDS_SORT2
#undef FMMDS_SORT
}

void launch_sort_pass(bool packed, const uint64_t* kin, uint64_t* kout, const uint32_t* vin,
                      uint32_t* vout, uint32_t n, uint32_t shift, const uint32_t* goff,
                      uint64_t* status, uint32_t* tile_counter, hipStream_t s, int items,
                      const uint32_t* n_dev) {
  sort_pass_dispatch<false>(packed, kin, kout, vin, vout, n, sort_tiles(n, items), shift, goff,
                            status, tile_counter, s, items, n_dev, SegSort{});
}

void launch_sort_pass_seg(bool packed, const uint64_t* kin, uint64_t* kout, const uint32_t* vin,
                          uint32_t* vout, uint32_t shift, const SegSort& sg, uint64_t* status,
                          uint32_t* tile_counter, hipStream_t s, int items) {
  if (sg.n_tiles == 0) return;
  sort_pass_dispatch<true>(packed, kin, kout, vin, vout, 0, sg.n_tiles, shift, nullptr, status,
                           tile_counter, s, items, nullptr, sg);
}

}  // namespace fmmds
