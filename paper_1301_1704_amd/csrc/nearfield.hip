// Near-field sum over the E2 lists: the first consumer of the structures.
//
// For every receiver point y in the box b of the finest level, the source
// points of the E2 boxes of b are exactly the points Algorithm 2 gathers:
// the E2 list names nonempty source boxes by rank, and a source box's points
// are consecutive in the sorted order from its bookmark to the next one. The
// sum here is the Laplace potential phi(y) = sum q_i / |x_i - y| over those
// points (the direct part of the FMM, Section 1.2), in FP32, with pairs at
// distance zero left out; the result goes to y's original position through
// the receiver permutation (the paper keeps RecvPermutationIdx for this).
//
// Layout: the sorted source points and their charges are packed once into
// 16-byte records (x, y, z, q), so each source point is one 16-byte load.
//
// One wave takes W receivers consecutive in Morton order (64, fewer when that
// would leave the chip short of waves) and turns the E2 lists of their boxes
// into runs of consecutive source points in LDS. Then, box by box of the wave:
//   - short lists: 64 / W lanes per receiver, each walking a part of its box's
//     runs; lanes of one box read the same points, and those of neighboring
//     boxes mostly the same lines;
//   - long lists, and boxes that hold the whole wave of receivers (clustered
//     input puts hundreds of points in one box): the wave stages
//     the box's source points in LDS 64 at a time (one coalesced 16-byte load
//     per lane) and every lane sums its receiver against the whole tile. With
//     r < 64 receivers the tile is split over 64 / R lane groups (R = r rounded
//     up to a power of two) whose partial sums are added by shuffles.
#include <mutex>

#include "device.h"
#include "internal.h"

namespace fmmds {

// One term of the sum, q / |x - y|, added to acc; a coincident pair adds nothing
// whatever its charge (infinite or NaN): its charge is replaced by zero and its
// distance by one whose reciprocal is finite.
// Coordinates come scaled by kNearScale (exactly), so that the square of the
// smallest distance whose square FP32 can hold is a normal number, as the
// reciprocal square root instruction needs; the reciprocal is scaled back before
// the charge meets it, so that a term is subnormal or infinite only where q / r
// itself is. A term takes 12 instructions; with the library's rsqrtf, which scales
// its argument each time, it took 16 (3.6M uniform points at 110 per box, bound
// by these: 4406 -> 3252 us).
constexpr float kNearScale = 4096.0f;
constexpr float kNearMin = 1.17549435e-38f;  // the smallest normal number
__device__ __forceinline__ void add_term(float& acc, const float4 x, float yx, float yy, float yz) {
  const float dx = fabsf(x.x) - yx, dy = x.y - yy, dz = x.z - yz;
  const float r2 = dx * dx + dy * dy + dz * dz;
  const float q = r2 >= kNearMin ? x.w : 0.0f;
  acc += q * (kNearScale * __builtin_amdgcn_rsqf(fmaxf(r2, kNearMin)));
}

// The same for charges that near_plain holds for: neither a term nor a sum leaves
// FP32's normal range while it is kNearScale times too small, and zero times the
// charge is zero, so the sum is scaled at its end and the reciprocal selected: 10
// instructions (2^20 sources and receivers at level 2, bound by these: 88.8 -> 78.6
// ms). A record whose charge is another one has a negative x.
__device__ __forceinline__ void add_plain_term(float& acc, const float4 x, float yx, float yy,
                                               float yz) {
  const float dx = fabsf(x.x) - yx, dy = x.y - yy, dz = x.z - yz;
  const float r2 = dx * dx + dy * dy + dz * dz;
  const float inv = __builtin_amdgcn_rsqf(r2);
  acc += x.w * (r2 >= kNearMin ? inv : 0.0f);
}
__device__ __forceinline__ bool near_plain(float q) {
  const float m = fabsf(q);
  return q == 0.0f || (m >= 0x1p-80f && m <= 0x1p60f);
}

// The sources as records, and the box of every T-th receiver (t_log2 = log2 T).
// T is the receivers per wave W, so that each wave finds its first box there, but
// at least 8, so that the table fits the scratch that the header promises (8 bytes
// per 9 receivers): waves of 4 go on from the box starts between, which they load
// anyway.
constexpr uint32_t kNearTable = 8;
__global__ __launch_bounds__(256) void k_pack_sources(
    const float* __restrict__ sxyz, const uint32_t* __restrict__ sperm,
    const float* __restrict__ charges, uint32_t n, float4* __restrict__ out,
    const uint32_t* __restrict__ rbegin, uint32_t n_rbox, uint32_t t_log2,
    uint32_t* __restrict__ wave_box) {
  for (uint64_t i = blockIdx.x * 256ull + threadIdx.x; i < n; i += gridDim.x * 256ull) {
    const float q = charges ? charges[sperm[i]] : 1.0f;
    const float x = kNearScale * fabsf(sxyz[3 * i]);  // (-0.0 is a coordinate too)
    out[i] = make_float4(near_plain(q) ? x : -x, kNearScale * sxyz[3 * i + 1],
                         kNearScale * sxyz[3 * i + 2], q);
  }
  const uint32_t T = 1u << t_log2;
  for (uint64_t b = blockIdx.x * 256ull + threadIdx.x; b < n_rbox; b += gridDim.x * 256ull) {
    const uint32_t k0 = rbegin[b], k1 = rbegin[b + 1];
    for (uint64_t t = ((uint64_t)k0 + T - 1u) >> t_log2; t << t_log2 < k1; ++t)
      wave_box[t] = (uint32_t)b;
  }
}

// Staging: entries of consecutive ranks are consecutive points, so a run costs
// two bookmark loads whatever its length, and every load of 4 x 64 entries is
// in flight at once. Lists that do not fit the LDS are taken in rounds of whole
// boxes.
// Short lists: a lane walks its runs as one sequence of points, four at a time,
// so that a wave makes as many steps as its longest sequence (about 40 points
// on uniform input; a loop per list entry makes the longest box among the lanes
// for each entry in turn, about 110). The next four points are loaded before
// the present ones are summed, into four sums that are added at the end.
//
// Measured, whole sum: 2^24 uniform sources and receivers, level 8: 2230 us with
// a lane per receiver box and its list in batches of eight entries, 1624 us
// now (380 of it the packing, whose charges are a random read each, 350 the
// random writes of phi; the walk itself is bound by the cache's one line a
// cycle: each lane reads its own 16 bytes). 6.0M sources and 5.0M receivers,
// sphere + clusters, level 9: 3250-3800 -> 806-861 us. (Blocks not renumbered so that
// an XCD takes consecutive receivers: the clustered sum takes a quarter longer.)
// 29K sources and 15K receivers at level 3: 97 -> 48 us.
constexpr uint32_t kNearRuns = 512;  // runs staged per wave
constexpr uint32_t kNearChunks = 4;  // list entries staged at a time, in 64s
// Lists of more source points go tile by tile: one lane walking such a list
// alone would outlast its wave (6.0M sources and 5.0M receivers, sphere + clusters,
// level 9, limits of 512 / 1024 / 2048 points: 811 / 806 / 847 us).
constexpr uint32_t kNearLongList = 1024;
// So do boxes of the whole wave, whose lanes all want the same points (boxes of W
// receivers, 36 sources a box, walked / by tiles: W = 64 487 / 324 us, 32 217 /
// 149, 16 124 / 97, 8 77 / 71, 4 52 / 61, so waves of 4 walk). Two boxes in a wave
// are walked at once, but tiled one after the other: with 33 of 64 receivers in
// the first 555 walked, 762 with that one tiled, with 48 521 and 715.
constexpr uint32_t kNearTileMin = 8;

struct NearStage {
  float4 tile[64];
  uint32_t first[kNearRuns], end[kNearRuns];
  uint32_t pre[64];  // inclusive prefix of one box's run lengths
  uint8_t start[64 * kNearChunks];
};

__device__ __forceinline__ void wave_fence() {
  __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
  __builtin_amdgcn_wave_barrier();
}

// The sum over runs [r0, r1) (at most 27) of one box, by the whole wave, for
// the nr receivers whose coordinates lanes f .. f + nr - 1 hold. Lane i of each
// group of R lanes (R = nr rounded up to a power of two) gets receiver i's sum.
__device__ __forceinline__ float tile_sum(NearStage& S, const float4* __restrict__ src,
                                          uint32_t r0, uint32_t r1, uint32_t f, uint32_t nr,
                                          float yx, float yy, float yz, uint32_t& total) {
  const uint32_t lane = threadIdx.x & 63u;
  const uint32_t nrun = r1 - r0;
  const uint32_t cnt = lane < nrun ? S.end[r0 + lane] - S.first[r0 + lane] : 0u;
  const uint32_t pre = wave_incl_scan(cnt);
  total = (uint32_t)__builtin_amdgcn_readlane((int)pre, 63);
  S.pre[lane] = pre;
  uint32_t R = 1;
  while (R < nr) R <<= 1;
  const uint32_t G = 64u / R, r = lane & (R - 1u), g = lane / R;
  const int from = (int)(f + min(r, nr - 1u));
  yx = __shfl(yx, from, 64), yy = __shfl(yy, from, 64), yz = __shfl(yz, from, 64);
  wave_fence();
  float acc = 0.0f, plain = 0.0f;  // plain: to be scaled
  for (uint32_t p = 0; p < total; p += 64) {
    // Stage points p .. p + 63 of the runs' concatenation: point q lies in the
    // first run whose inclusive prefix exceeds q.
    const uint32_t q = p + lane;
    float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
    if (q < total) {
      uint32_t lo = 0, hi = nrun - 1;
      while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (S.pre[mid] > q) hi = mid;
        else lo = mid + 1;
      }
      x = src[S.first[r0 + lo] + (q - (lo ? S.pre[lo - 1] : 0u))];
    }
    const bool all_plain = __ballot(__float_as_int(x.x) < 0) == 0;
    wave_fence();  // the previous tile's reads come before this store
    S.tile[lane] = x;
    wave_fence();
    const uint32_t m = min(64u, total - p);
    uint32_t j = g;
    if (all_plain) {
      for (; j + 3 * G < m; j += 4 * G) {
        const float4 a = S.tile[j], c = S.tile[j + G], d = S.tile[j + 2 * G], e = S.tile[j + 3 * G];
        add_plain_term(plain, a, yx, yy, yz);
        add_plain_term(plain, c, yx, yy, yz);
        add_plain_term(plain, d, yx, yy, yz);
        add_plain_term(plain, e, yx, yy, yz);
      }
      for (; j < m; j += G) add_plain_term(plain, S.tile[j], yx, yy, yz);
    } else {
      for (; j < m; j += G) add_term(acc, S.tile[j], yx, yy, yz);
    }
  }
  wave_fence();
  acc += kNearScale * plain;
  for (uint32_t o = R; o < 64u; o <<= 1) acc += __shfl_xor(acc, (int)o, 64);
  return acc;
}

template <uint32_t W>
__global__ __launch_bounds__(256, 5) void k_near_field(
    uint32_t n_recv, const uint32_t* __restrict__ rbegin, uint32_t n_rbox,
    const float* __restrict__ rxyz, const uint32_t* __restrict__ rperm,
    const uint32_t* __restrict__ e2_off, const uint32_t* __restrict__ e2_ent,
    const uint32_t* __restrict__ sbegin, const float4* __restrict__ src, float* __restrict__ phi,
    unsigned long long* __restrict__ n_pairs, const uint32_t* __restrict__ wave_box) {
  __shared__ NearStage s_stage[4];
  constexpr uint32_t kParts = 64u / W;  // lanes per receiver
  const uint32_t lane = threadIdx.x & 63u, rec = lane & (W - 1u), part = lane / W;
  const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  NearStage& S = s_stage[w];
  // consecutive receivers on one XCD: their sources come into one L2
  const uint64_t t = (uint64_t)xcd_block(blockIdx.x, gridDim.x) * 4 + w;
  const uint64_t k0 = W * t;
  if (k0 >= n_recv) return;  // whole wave
  // Box of each receiver: the wave's first one plus the box starts up to it.
  constexpr uint32_t T = W < kNearTable ? kNearTable : W;
  const uint32_t bt = wave_box[k0 / T];
  S.start[lane] = 0;
  wave_fence();
  uint32_t st = 0;  // box starts past the table's receiver (none: 0, never past k0)
  if (lane < T && bt + 1 + (uint64_t)lane < n_rbox) st = rbegin[bt + 1 + lane];
  const uint32_t b0 = bt + (T > W ? (uint32_t)__popcll(__ballot(st != 0 && st <= k0)) : 0u);
  if (st > k0 && st < k0 + W) S.start[st - (uint32_t)k0] = 1;
  wave_fence();
  const uint64_t starts = __ballot(lane < W && S.start[lane] != 0);
  const uint32_t jb = (uint32_t)__popcll(starts & ((2ull << rec) - 1ull));
  const uint64_t k = k0 + rec;
  const bool mine = k < n_recv;
  float yx = 0.0f, yy = 0.0f, yz = 0.0f;
  uint32_t perm = 0;
  if (mine) {
    yx = kNearScale * rxyz[3 * k], yy = kNearScale * rxyz[3 * k + 1];
    yz = kNearScale * rxyz[3 * k + 2];
    perm = rperm[k];
  }
  const uint32_t n_here = (uint32_t)min((uint64_t)W, n_recv - k0);
  // Lane j < nb: where box b0 + j's list starts; e_end: where the last one ends.
  const uint32_t nb = 1u + (uint32_t)__popcll(starts);
  const uint32_t off = e2_off[min(b0 + lane, n_rbox)];
  const uint32_t e_end = (uint32_t)__builtin_amdgcn_readfirstlane((int)e2_off[b0 + nb]);
  uint64_t pts = 0;
  float acc[4] = {0.0f, 0.0f, 0.0f, 0.0f};
  float whole = 0.0f;  // the receiver's sum, if its box was taken tile by tile
  uint32_t box = 0;  // the first box whose list is not summed yet
  uint32_t e = (uint32_t)__builtin_amdgcn_readfirstlane((int)off);
  while (box < nb) {
    // Stage kNearChunks * 64 entries at a time.
    uint32_t runs = 0, my_run = 0;  // lane j: the first run of box b0 + j
    uint32_t prev = 0;              // the last entry of the chunk before
    uint32_t e0 = e;
    while (e0 < e_end) {
      uint32_t s[kNearChunks];
#pragma unroll
      for (uint32_t c = 0; c < kNearChunks; ++c) {
        s[c] = e2_ent[min(e0 + 64u * c + lane, e_end - 1u)];
        S.start[64u * c + lane] = 0;
      }
      wave_fence();
      const bool here = lane >= box && lane < nb && off >= e0 && off - e0 < 64u * kNearChunks;
      if (here) S.start[off - e0] = 1;
      wave_fence();
      uint64_t m[kNearChunks];
      uint32_t last = prev, total = 0;
#pragma unroll
      for (uint32_t c = 0; c < kNearChunks; ++c) {
        const uint32_t up = (uint32_t)__shfl_up((int)s[c], 1, 64);
        const uint32_t before = lane == 0 ? last : up;
        m[c] = __ballot(e0 + 64u * c + lane < e_end &&
                        (S.start[64u * c + lane] != 0 || s[c] != before + 1u));
        last = (uint32_t)__builtin_amdgcn_readlane((int)s[c], 63);
        total += (uint32_t)__popcll(m[c]);
      }
      if (runs + total > kNearRuns) break;  // (never the first time: kNearChunks * 64 runs fit)
      uint32_t first[kNearChunks], end[kNearChunks], r[kNearChunks];
      bool is_end[kNearChunks];
#pragma unroll
      for (uint32_t c = 0; c < kNearChunks; ++c) {
        const uint32_t i = e0 + 64u * c + lane;
        const bool is_start = (m[c] >> lane) & 1u;
        // the run of this entry (lane 0 of the first chunk starts one)
        r[c] = runs + mbcnt(m[c]) + (is_start ? 1u : 0u) - 1u;
        is_end[c] = i < e_end && (lane == 63u || i + 1u == e_end || ((m[c] >> ((lane + 1u) & 63u)) & 1u));
        if (is_start) first[c] = sbegin[s[c]];
        if (is_end[c]) end[c] = sbegin[s[c] + 1u];
        const uint32_t r_of = (uint32_t)__shfl((int)r[c], (int)(off - e0 - 64u * c) & 63, 64);
        if (here && off < e_end && (off - e0) >> 6 == c) my_run = r_of;
        runs += (uint32_t)__popcll(m[c]);
      }
#pragma unroll
      for (uint32_t c = 0; c < kNearChunks; ++c) {
        if ((m[c] >> lane) & 1u) S.first[r[c]] = first[c];
        if (is_end[c]) S.end[r[c]] = end[c];  // (a run over two chunks: the later one's stays)
      }
      prev = last;
      e0 += 64u * kNearChunks;
    }
    wave_fence();
    // The boxes staged whole: up to the last whose next list starts by e0.
    uint32_t stop = nb;
    if (e0 < e_end) {
      stop = (uint32_t)__popcll(__ballot(lane < nb && off <= e0)) - 1u;  // box `stop` is cut
    }
    if (lane < nb && off >= min(e0, e_end)) my_run = runs;  // lists after them (or empty at the end)
    uint32_t r = (uint32_t)__shfl((int)my_run, (int)jb, 64);
    const uint32_t r_next = (uint32_t)__shfl((int)my_run, (int)min(jb + 1u, 63u), 64);
    const uint32_t r1 = jb + 1u < nb ? r_next : runs;
    const bool now = mine && jb >= box && jb < stop;
    // The points of this lane's list, and whether the box goes tile by tile.
    uint32_t n = 0;
    if (now)
      for (uint32_t i = r; i < r1; ++i) n += S.end[i] - S.first[i];
    const uint64_t heads = starts | 1ull;  // lanes < W: first receiver of each box here
    const uint32_t f = 63u - (uint32_t)__clzll((long long)(heads & ((2ull << rec) - 1ull)));
    const uint64_t above = f >= 63u ? 0ull : heads >> (f + 1u);
    const uint32_t nr = above ? (uint32_t)__ffsll((long long)above) : n_here - f;
    const bool tiled = now && n > 0 && (n > kNearLongList || (W >= kNearTileMin && nr == W));
    uint64_t todo = __ballot(tiled && part == 0u && rec == f);
    while (todo) {
      const int h = __ffsll((long long)todo) - 1;
      todo &= todo - 1;
      const uint32_t hr0 = (uint32_t)__builtin_amdgcn_readlane((int)r, h),
                     hr1 = (uint32_t)__builtin_amdgcn_readlane((int)r1, h),
                     hn = (uint32_t)__builtin_amdgcn_readlane((int)nr, h);
      uint32_t total;
      const float v = tile_sum(S, src, hr0, hr1, (uint32_t)h, hn, yx, yy, yz, total);
      const float mine_v = __shfl(v, (int)((rec - (uint32_t)h) & 63u), 64);
      if (rec >= (uint32_t)h && rec < (uint32_t)h + hn) whole = mine_v;
      if (lane == 0) pts += (uint64_t)total * hn;
    }
    if (now && !tiled && n > 0) {
      // this lane's part of the list: points [skip, skip + left)
      uint32_t skip = 0, left = n;
      if (kParts > 1) {
        skip = n * part / kParts;
        left = n * (part + 1u) / kParts - skip;
      }
      if (left > 0) {
      uint32_t p = S.first[r], p_end = S.end[r];
      if (kParts > 1) {
        while (skip >= p_end - p) {
          skip -= p_end - p;
          ++r;
          p = S.first[r], p_end = S.end[r];
        }
        p += skip;
      }
      pts += left;
      // the next four points; returns the number of them that there are
      auto next4 = [&](float4* x) {
        uint32_t c = 0;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          x[u] = src[p];  // (past the end: the last run's first point)
          if (left > 0) {
            --left;
            ++c;
            if (++p == p_end) {
              r = min(r + 1u, r1 - 1u);
              p = S.first[r], p_end = S.end[r];
            }
          }
        }
        return c;
      };
      auto sum4 = [&](const float4* x, uint32_t c) {
#pragma unroll
        for (int u = 0; u < 4; ++u)
          if ((uint32_t)u < c) add_term(acc[u], x[u], yx, yy, yz);
      };
      float4 xa[4], xb[4];
      uint32_t ca = next4(xa), cb = 0;
      while (true) {
        cb = 0;
        if (left > 0) cb = next4(xb);
        sum4(xa, ca);
        if (cb == 0) break;
        ca = 0;
        if (left > 0) ca = next4(xa);
        sum4(xb, cb);
        if (ca == 0) break;
      }
      }
    }
    box = stop;
    e = (uint32_t)__builtin_amdgcn_readlane((int)off, (int)min(stop, 63u));
    wave_fence();
  }
  float sum = (acc[0] + acc[1]) + (acc[2] + acc[3]);
#pragma unroll
  for (uint32_t o = W; o < 64u; o <<= 1) sum += __shfl_xor(sum, (int)o, 64);
  if (mine && part == 0u) phi[perm] = sum + whole;
  if (n_pairs) {
    const uint64_t all = wave_sum_u64(pts);
    if (lane == 0 && all) atomicAdd(n_pairs, (unsigned long long)all);
  }
}

// log2 of the receivers per wave: 64 when that gives the chip's 8192 wave slots
// a wave each, fewer (and so more lanes per receiver) below, down to 4.
uint32_t near_field_w_log2(uint32_t n_recv) {
  uint32_t l = 6;
  while (l > 2 && ((uint64_t)n_recv >> l) < 8192) --l;
  return l;
}

uint64_t near_field_table(uint32_t n_recv) {
  const uint32_t T = std::max(1u << near_field_w_log2(n_recv), kNearTable);
  return ((uint64_t)n_recv + T - 1u) / T;
}

void launch_near_field(const float* sxyz, const uint32_t* sperm, const float* charges,
                       uint32_t n_src, float4* src, uint32_t n_rbox, uint32_t n_recv,
                       const uint32_t* rbegin, const float* rxyz, const uint32_t* rperm,
                       const uint32_t* e2_off, const uint32_t* e2_ent, const uint32_t* sbegin,
                       float* phi, unsigned long long* n_pairs, uint32_t* wave_box,
                       hipStream_t s) {
  const uint32_t l = near_field_w_log2(n_recv);
  const uint32_t pack = std::max<uint32_t>(
      1, std::min<uint32_t>(div_up(std::max(n_src, n_rbox), 256), 8192));
  hipLaunchKernelGGL(k_pack_sources, dim3(pack), dim3(256), 0, s, sxyz, sperm, charges, n_src, src,
                     rbegin, n_rbox, std::max(l, 3u), wave_box);
  static_assert(kNearTable == 1u << 3, "the table's step");
  const dim3 grid(div_up(n_recv, 4ull << l));
#define FMMDS_NEAR(W)                                                                           \
  hipLaunchKernelGGL(k_near_field<W>, grid, dim3(256), 0, s, n_recv, rbegin, n_rbox, rxyz,      \
                     rperm, e2_off, e2_ent, sbegin, src, phi, n_pairs, wave_box)
  switch (l) {
    case 6: FMMDS_NEAR(64); break;
    case 5: FMMDS_NEAR(32); break;
    case 4: FMMDS_NEAR(16); break;
    case 3: FMMDS_NEAR(8); break;
    default: FMMDS_NEAR(4); break;
  }
#undef FMMDS_NEAR
}

// ---------------------------------------------------------------------------
// Fixed scratch of fmmds_near_field_static, the entry point for callers that
// cannot allocate: the packed sources and the waves' boxes live here instead
// of in memory from the cache. Each GPU holds its own copy of the
// array, at its own address, from the library's load on that GPU until the
// process ends. In host code `scratch` names a host-side stand-in, never the
// device memory: the device address comes from hipGetSymbolAddress, once per
// device, with that device current.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kNearStaticBytes];

fmmds_status near_field_static_scratch(void** out) {
  static std::mutex mu;
  static void* ptr[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return FMMDS_ERR_DEVICE;
  }
  std::lock_guard<std::mutex> g(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || p == nullptr) {
      (void)hipGetLastError();
      return FMMDS_ERR_DEVICE;
    }
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return FMMDS_OK;
}

}  // namespace fmmds
