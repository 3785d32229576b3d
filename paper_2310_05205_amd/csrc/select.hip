// Trajectory selection on gfx950 (GEAR Sec. 1 strategies; Sec. 3.3).
//
// Prioritized (weighted) sampling is a prefix sum over the priorities
// followed by one search per uniform draw (Sec. 3.3, centralized selection).
// Here the prefix sum is split between two kernels so that no workgroup ever
// waits on another:
//
//   scan_kernel    one pass over the priorities.  A workgroup reduces a
//                  chunk of 16 tiles of 256 priorities (64 above 2^22
//                  priorities) and writes each tile's sum and the chunk's
//                  (levels 0 and 1 of the sum tree); above 2^24 priorities it
//                  also adds the chunk's sum into the level-2 node that covers
//                  it.
//   search_kernel  16 lanes (one DPP row) per draw.  Each workgroup forms the
//                  inclusive prefix of the highest level, at most 1024 nodes,
//                  in LDS (its last entry is the total S); a draw r =
//                  floor(u*S/2^64) finds its node there by probing 16 evenly
//                  spaced entries at a time, then its tile among the chunk's
//                  (one or four sums per lane, a row scan) and its slot among the
//                  tile's 256 priorities (16 per lane), r reduced by the prefix
//                  before each choice.  The index found is the smallest i with
//                  C_i > r for the inclusive prefix C over all priorities: the
//                  binary-search answer.
//
// Small tables (N <= kSmallN, B <= kSmallMaxB, sum tree not kept across
// updates) take one launch instead: small_select_kernel, one workgroup,
// forms the inclusive prefix C of all N priorities in LDS with a block scan,
// finds each draw's slot as the smallest i with C_i > r by bisection over
// C, and computes the IS weights, all in one launch.
//
// FIFO, LIFO and uniform selection are one thread per draw.
#include <mutex>

#include "gear_internal.h"
#include "wave.h"

namespace gear {
namespace {

struct Levels {
    uint64_t* level[kMaxLevels];   // level 0: tile sums; level 1: chunk sums; level 2: sums of 256 chunks
    int64_t size[kMaxLevels];
    int nlevels;
    // The top level again (level[nlevels - 1]), so that a search reads it
    // without first waiting for nlevels.
    const uint64_t* top;
    int64_t top_size;
};

// Sets the top-level copy of a search's levels.
inline Levels with_top(Levels lv) {
    lv.top = lv.level[lv.nlevels - 1];
    lv.top_size = lv.size[lv.nlevels - 1];
    return lv;
}

// Inclusive prefix within each row of 16 lanes.
__device__ __forceinline__ uint64_t row_inclusive_scan(uint64_t v) {
    v += dpp_u64<0x111, 0xf>(v);  // row_shr:1
    v += dpp_u64<0x112, 0xf>(v);  // row_shr:2
    v += dpp_u64<0x114, 0xf>(v);  // row_shr:4
    v += dpp_u64<0x118, 0xf>(v);  // row_shr:8
    return v;
}

// Number of lanes of this lane's row for which `b` holds.
__device__ __forceinline__ int row_count(bool b) {
    return __popc((uint32_t)(__ballot(b) >> (threadIdx.x & 48)) & 0xFFFFu);
}

// Among four values, the number whose inclusive prefix is <= r (0 .. 3; the
// fourth is the answer when no earlier one is) and the prefix before it.
__device__ __forceinline__ int pick_of4(uint64_t v0, uint64_t v1, uint64_t v2, uint64_t r, uint64_t& before) {
    const uint64_t c1 = v0 + v1, c2 = c1 + v2;
    const bool b0 = v0 <= r, b1 = c1 <= r, b2 = c2 <= r;
    before = b2 ? c2 : b1 ? c1 : b0 ? v0 : 0;
    return (int)b0 + (int)b1 + (int)b2;
}

__device__ inline void load4_u64(const uint64_t* __restrict__ a, int64_t n, int64_t e, uint64_t& v0, uint64_t& v1,
                                 uint64_t& v2, uint64_t& v3) {
    if (e + 4 <= n) {
        const ulonglong2 p0 = *reinterpret_cast<const ulonglong2*>(a + e);
        const ulonglong2 p1 = *reinterpret_cast<const ulonglong2*>(a + e + 2);
        v0 = p0.x; v1 = p0.y; v2 = p1.x; v3 = p1.y;
    } else {
        v0 = e + 0 < n ? a[e + 0] : 0;
        v1 = e + 1 < n ? a[e + 1] : 0;
        v2 = e + 2 < n ? a[e + 2] : 0;
        v3 = e + 3 < n ? a[e + 3] : 0;
    }
}

__device__ inline void load4_u32(const uint32_t* __restrict__ a, int64_t n, int64_t e, uint32_t& p0, uint32_t& p1,
                                 uint32_t& p2, uint32_t& p3) {
    if (e + 4 <= n) {
        const uint4 v = *reinterpret_cast<const uint4*>(a + e);
        p0 = v.x; p1 = v.y; p2 = v.z; p3 = v.w;
    } else {
        p0 = e + 0 < n ? a[e + 0] : 0u;
        p1 = e + 1 < n ? a[e + 1] : 0u;
        p2 = e + 2 < n ? a[e + 2] : 0u;
        p3 = e + 3 < n ? a[e + 3] : 0u;
    }
}

// Every wave reduces four tiles, four 16-byte loads per lane, all issued before
// any is used: 256 threads per chunk of 16 tiles, so that a table of half a
// million priorities is spread over 123 CUs, and 1024 per chunk of 64.
// Against 256 threads per chunk of 32 tiles and an atomic per chunk: 500000
// priorities behind an update 4.3 -> 3.1 us, 2^22 6.8 -> 5.3.
//
// `upper` is the level-2 copy this scan adds into, or NULL; `clear` the other
// copy, which this scan zeroes for the next one (each node is zeroed by the
// chunk that starts it).  kMin: also write the chunk's smallest non-zero
// priority (only the global IS normalisation needs it).
template <bool kMin, int kTiles>
__global__ __launch_bounds__(kTiles * 16) void scan_kernel(const uint32_t* __restrict__ prio, int64_t N,
                                                           uint64_t* __restrict__ upper,
                                                           uint64_t* __restrict__ clear,
                                                           uint64_t* __restrict__ tile_sums, int64_t ntiles,
                                                           uint64_t* __restrict__ chunk_sums,
                                                           uint32_t* __restrict__ chunk_min) {
    constexpr int kScanWaves = kTiles / 4;
    __shared__ uint64_t tile_sum[kTiles];
    __shared__ uint32_t wave_min[kScanWaves];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int64_t chunk = blockIdx.x;
    constexpr int kTilesPerWave = 4;

    const int64_t tile0 = chunk * kTiles + wave * kTilesPerWave;
    uint32_t x[kTilesPerWave][4];
    if ((tile0 + kTilesPerWave) * kTile <= N) {  // the same branch for the whole wave
#pragma unroll
        for (int q = 0; q < kTilesPerWave; q++) {
            const uint4 v = *reinterpret_cast<const uint4*>(prio + (tile0 + q) * kTile + lane * 4);
            x[q][0] = v.x; x[q][1] = v.y; x[q][2] = v.z; x[q][3] = v.w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < kTilesPerWave; q++)
            load4_u32(prio, N, (tile0 + q) * kTile + lane * 4, x[q][0], x[q][1], x[q][2], x[q][3]);
    }
#pragma unroll
    for (int q = 0; q < kTilesPerWave; q++) {
        const uint64_t s = wave_sum((uint64_t)x[q][0] + x[q][1] + x[q][2] + x[q][3]);
        if (lane == 0) {
            tile_sum[wave * kTilesPerWave + q] = s;
            if (tile0 + q < ntiles) tile_sums[tile0 + q] = s;
        }
    }
    if (kMin) {
        // Smallest non-zero priority of the chunk.
        uint32_t m = 0xFFFFFFFFu;
#pragma unroll
        for (int q = 0; q < kTilesPerWave; q++)
#pragma unroll
            for (int e = 0; e < 4; e++) m = (x[q][e] != 0u && x[q][e] < m) ? x[q][e] : m;
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            const uint32_t o = __shfl_xor(m, d);
            m = o < m ? o : m;
        }
        if (lane == 0) wave_min[wave] = m;
    }
    __syncthreads();
    if (wave != 0) return;
    if (kMin && lane == 0) {
        uint32_t cm = wave_min[0];
        for (int k = 1; k < kScanWaves; k++) cm = wave_min[k] < cm ? wave_min[k] : cm;
        chunk_min[chunk] = cm;
    }
    const uint64_t chunk_sum = wave_sum(lane < kTiles ? tile_sum[lane] : 0);
    if (lane != 0) return;
    chunk_sums[chunk] = chunk_sum;
    if (upper != nullptr) {
        if (chunk_sum != 0) atomicAdd(reinterpret_cast<unsigned long long*>(upper + chunk / kFanout), chunk_sum);
        if (chunk % kFanout == 0) clear[chunk / kFanout] = 0;
    }
}

typedef void (*ScanKernel)(const uint32_t*, int64_t, uint64_t*, uint64_t*, uint64_t*, int64_t, uint64_t*, uint32_t*);

unsigned scan_threads(int64_t N) { return (unsigned)tiles_per_chunk(N) * 16; }

ScanKernel scan_variant(bool min, int64_t N) {
    if (tiles_per_chunk(N) == kSmallChunk) return min ? scan_kernel<true, kSmallChunk> : scan_kernel<false, kSmallChunk>;
    return min ? scan_kernel<true, kLargeChunk> : scan_kernel<false, kLargeChunk>;
}

// One GPU's share of a selection over G shards (the table is shard g).
// With totals == NULL the table is the whole population.
struct Shard {
    const uint64_t* totals;  // the G shard totals, identical on every shard
    int G, g;
    int64_t base;            // added to the local slot of an owned draw
};

// One row of 16 lanes per draw, 16 draws per workgroup.  The search is a chain
// of three dependent loads (highest level, tile sums, priorities); with a whole
// wave per draw and a 64-lane scan at each level it was bound by instruction
// issue instead (8192 waves of about 300): 8192 draws over 2^22 priorities 7.2
// -> 5.7 us, 32768 draws with weights and update 32.5 -> 23.3 us.
constexpr int kSearchThreads = 256;
constexpr int kSearchDraws = kSearchThreads / 16;

template <bool kShard, int kTiles, bool kThree>
__global__ __launch_bounds__(kSearchThreads) void search_kernel(const uint32_t* __restrict__ prio, int64_t N,
                                                                Levels lv, int32_t B, uint64_t span, uint64_t seed,
                                                                int want_min, Shard sh, uint32_t* __restrict__ wg_min,
                                                                uint32_t* status, int64_t* __restrict__ idx,
                                                                int32_t* __restrict__ start,
                                                                uint32_t* __restrict__ sel_prio) {
    __shared__ uint64_t top[kTopMax];  // inclusive prefix of the highest level
    __shared__ uint64_t s_wave[kSearchThreads / 64];
    __shared__ uint32_t s_min[kSearchThreads / 64];
    // The arguments at once, not each where it is first used.
    asm volatile("" ::"s"(prio), "s"(N), "s"(lv.top), "s"(lv.top_size), "s"(lv.level[0]), "s"(lv.size[0]), "s"(B),
                 "s"(span), "s"(seed), "s"(idx), "s"(start), "s"(sel_prio));
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int sub = threadIdx.x & 15;  // lane within the draw's row
    const int n = (int)lv.top_size;
    {
        uint64_t v0, v1, v2, v3;
        load4_u64(lv.top, n, threadIdx.x * 4, v0, v1, v2, v3);
        const uint64_t part = v0 + v1 + v2 + v3;
        const uint64_t incl = wave_inclusive_scan(part);
        if (lane == 63) s_wave[wave] = incl;
        __syncthreads();
        uint64_t c = incl - part;
#pragma unroll
        for (int k = 0; k < kSearchThreads / 64; k++) c += k < wave ? s_wave[k] : 0;
        if ((int)threadIdx.x * 4 < n) {  // entries past n are never read
            top[threadIdx.x * 4] = c += v0;
            top[threadIdx.x * 4 + 1] = c += v1;
            top[threadIdx.x * 4 + 2] = c += v2;
            top[threadIdx.x * 4 + 3] = c += v3;
        }
        __syncthreads();
    }
    const uint64_t S = top[n - 1];
    // Draws are numbers in [0, S_all); this table owns [P, P + S).
    uint64_t S_all = S, P = 0;
    if (kShard) {
        uint64_t all = 0, before = 0;
        for (int h = lane; h < sh.G; h += 64) {
            const uint64_t x = sh.totals[h];
            all += x;
            before += h < sh.g ? x : 0;
        }
        S_all = wave_sum(all);
        P = wave_sum(before);
    }
    uint32_t my_min = 0xFFFFFFFFu;  // smallest priority this row selected

    // Every lane of a row takes the same branches, so row scans, counts and
    // broadcasts see their whole row.
    for (int64_t b = (int64_t)blockIdx.x * kSearchDraws + (threadIdx.x >> 4); b < B;
         b += (int64_t)gridDim.x * kSearchDraws) {
        if (S_all == 0) {
            if (sub == 0) {
                idx[b] = -1;
                start[b] = 0;
                if (want_min) sel_prio[b] = 0u;
                atomicOr(status, GEAR_STATUS_NO_WEIGHT);
            }
            continue;
        }
        uint64_t r = scale_draw(splitmix64_out(seed, 2 * (uint64_t)b), S_all);
        const int32_t st = (int32_t)scale_draw(splitmix64_out(seed, 2 * (uint64_t)b + 1), span);
        if (kShard) {
            if (r < P || r - P >= S) {  // another shard's draw: same window start, no slot
                if (sub == 0) {
                    idx[b] = -1;
                    start[b] = st;
                    if (want_min) sel_prio[b] = 0u;
                }
                continue;
            }
            r -= P;
        }
        // The node: the first prefix above r, which exists as r < S.
        int j = 0;
        if (n > 256) {
            int e = sub * 64 + 63;
            j = row_count(e < n && top[e] <= r) * 64;
            e = j + sub * 4 + 3;
            j += row_count(e < n && top[e] <= r) * 4;
            e = j + sub;
            j += row_count(sub < 4 && e < n && top[e] <= r);
        } else {
            int e = sub * 16 + 15;
            j = row_count(e < n && top[e] <= r) * 16;
            e = j + sub;
            j += row_count(e < n && top[e] <= r);
        }
        if (j > 0) r -= top[j - 1];
        // Below, a row whose sums end at or before r (priorities changed under
        // a running selection) takes the last lane: every index stays in range.
        int64_t chunk = j;
        if (kThree) {  // 256 chunks, 16 per lane
            uint64_t v[16], sum = 0;
#pragma unroll
            for (int q = 0; q < 16; q += 4)
                load4_u64(lv.level[1], lv.size[1], (int64_t)j * kFanout + sub * 16 + q, v[q], v[q + 1], v[q + 2],
                          v[q + 3]);
#pragma unroll
            for (int q = 0; q < 16; q++) sum += v[q];
            const uint64_t incl = row_inclusive_scan(sum);
            uint64_t before = incl - sum, c = before;
            int k = 0;
#pragma unroll
            for (int q = 0; q < 15; q++) {
                c += v[q];
                if (c <= r) {
                    k = q + 1;
                    before = c;
                }
            }
            const int l = row_count(incl <= r);
            const int from = l < 15 ? l : 15;
            r -= __shfl(before, from, 16);
            chunk = (int64_t)j * kFanout + from * 16 + __shfl(k, from, 16);
            if (chunk >= lv.size[1]) chunk = lv.size[1] - 1;
        }
        // The tile among the chunk's.
        int64_t tile;
        if (kTiles == 16) {
            const int64_t e = chunk * kTiles + sub;
            const uint64_t v = e < lv.size[0] ? lv.level[0][e] : 0;
            const uint64_t incl = row_inclusive_scan(v);
            const int l = row_count(incl <= r);
            const int from = l < 15 ? l : 15;
            r -= __shfl(incl - v, from, 16);
            tile = chunk * kTiles + from;
        } else {
            uint64_t v0, v1, v2, v3, before;
            load4_u64(lv.level[0], lv.size[0], chunk * kTiles + sub * 4, v0, v1, v2, v3);
            const uint64_t sum = v0 + v1 + v2 + v3;
            const uint64_t incl = row_inclusive_scan(sum);
            const int k = pick_of4(v0, v1, v2, r - (incl - sum), before);
            const int l = row_count(incl <= r);
            const int from = l < 15 ? l : 15;
            r -= __shfl(incl - sum + before, from, 16);
            tile = chunk * kTiles + from * 4 + __shfl(k, from, 16);
        }
        if (tile >= lv.size[0]) tile = lv.size[0] - 1;
        // The slot among the tile's 256 priorities.
        uint32_t p[16];
        const int64_t e0 = tile * kTile + sub * 16;
        if ((tile + 1) * kTile <= N) {
#pragma unroll
            for (int q = 0; q < 16; q += 4) {
                const uint4 v = *reinterpret_cast<const uint4*>(prio + e0 + q);
                p[q] = v.x; p[q + 1] = v.y; p[q + 2] = v.z; p[q + 3] = v.w;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 16; q += 4) load4_u32(prio, N, e0 + q, p[q], p[q + 1], p[q + 2], p[q + 3]);
        }
        uint64_t s4[4];
#pragma unroll
        for (int q = 0; q < 4; q++) s4[q] = (uint64_t)p[4 * q] + p[4 * q + 1] + p[4 * q + 2] + p[4 * q + 3];
        const uint64_t sum = s4[0] + s4[1] + s4[2] + s4[3];
        const uint64_t incl = row_inclusive_scan(sum);
        const int l = row_count(incl <= r);
        const int from = l < 15 ? l : 15;
        uint64_t rest = r - (incl - sum), before, unused;  // of use in lane `from` only
        const int g = pick_of4(s4[0], s4[1], s4[2], rest, before);
        rest -= before;
        uint32_t a[4];
#pragma unroll
        for (int q = 0; q < 4; q++)
            a[q] = g == 0 ? p[q] : g == 1 ? p[4 + q] : g == 2 ? p[8 + q] : p[12 + q];
        const int k = pick_of4(a[0], a[1], a[2], rest, unused);
        const uint32_t mine = k == 0 ? a[0] : k == 1 ? a[1] : k == 2 ? a[2] : a[3];
        const int at = __shfl(g * 4 + k, from, 16);
        const uint32_t pv = __shfl(mine, from, 16);
        if (sub == 0) {
            int64_t slot = tile * kTile + from * 16 + at;
            if (slot >= N) slot = N - 1;  // only under changing priorities
            idx[b] = (kShard ? sh.base : 0) + slot;
            start[b] = st;
            // The selected priority is kept for the weight kernel in the
            // caller's weight buffer, which that kernel then overwrites.
            if (want_min) sel_prio[b] = pv;
        }
        my_min = pv < my_min ? pv : my_min;
    }
    if (want_min) {
        // One slot per workgroup, no atomics: the weight kernel reduces them.
        uint32_t o = __shfl_xor(my_min, 16);
        my_min = o < my_min ? o : my_min;
        o = __shfl_xor(my_min, 32);
        my_min = o < my_min ? o : my_min;
        if (lane == 0) s_min[wave] = my_min;
        __syncthreads();
        if (threadIdx.x == 0) {
            uint32_t m = s_min[0];
            for (int k = 1; k < kSearchThreads / 64; k++) m = s_min[k] < m ? s_min[k] : m;
            wg_min[blockIdx.x] = m;
        }
    }
}

typedef void (*SearchKernel)(const uint32_t*, int64_t, Levels, int32_t, uint64_t, uint64_t, int, Shard, uint32_t*,
                             uint32_t*, int64_t*, int32_t*, uint32_t*);

SearchKernel search_variant(bool shard, int64_t N, int nlevels) {
    if (tiles_per_chunk(N) == kSmallChunk)
        return shard ? search_kernel<true, kSmallChunk, false> : search_kernel<false, kSmallChunk, false>;
    if (nlevels == 2) return shard ? search_kernel<true, kLargeChunk, false> : search_kernel<false, kLargeChunk, false>;
    return shard ? search_kernel<true, kLargeChunk, true> : search_kernel<false, kLargeChunk, true>;
}

int search_grid(int32_t B) {
    const int64_t g = ((int64_t)B + kSearchDraws - 1) / kSearchDraws;  // one draw per row while the grid allows
    return (int)(g < kSearchMaxGrid ? g : kSearchMaxGrid);
}

// (m / p)^beta for 0 < m, p.  pow and not exp(beta * log(m / p)), which loses the low
// bits of the logarithm (off by up to 65 units of 2^-53 at beta 4, pow by one).
__device__ __forceinline__ float is_weight(uint32_t m, uint32_t p, double beta) {
    return (float)pow((double)m / (double)p, beta);
}

// w_b = (n*P(i_b))^-beta / max_b' (n*P(i_b'))^-beta = (p_min / p_b)^beta,
// p_min the smallest selected priority; fp64, rounded once to fp32.  Every
// workgroup first reduces the search's per-workgroup minima.  The selected
// priority p_b arrives in w[b] itself (as uint32 bits; 0 marks a draw with
// no selectable slot) and is replaced by the weight.
__global__ __launch_bounds__(256) void is_weights_kernel(int32_t B, double beta, const uint32_t* __restrict__ wg_min,
                                                         int search_grid, float* __restrict__ w) {
    __shared__ uint32_t s_min[4];
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    // This draw's priority and the first four minima per thread are loaded
    // together, from indices clamped into their buffers, before any is used:
    // one memory round trip covers the search's largest grid.
    constexpr int kMinPerThread = kSearchMaxGrid / 256;
    const uint32_t pb_raw = reinterpret_cast<const uint32_t*>(w)[b < B ? b : B - 1];
    uint32_t v0[kMinPerThread];
#pragma unroll
    for (int u = 0; u < kMinPerThread; u++) {
        const int k = (int)threadIdx.x + u * (int)blockDim.x;
        v0[u] = wg_min[k < search_grid ? k : 0];
    }
    const uint32_t pb = b < B ? pb_raw : 0u;
    uint32_t m = 0xFFFFFFFFu;
#pragma unroll
    for (int u = 0; u < kMinPerThread; u++) {
        const int k = (int)threadIdx.x + u * (int)blockDim.x;
        m = (k < search_grid && v0[u] < m) ? v0[u] : m;
    }
    // Grids larger than blockDim * kMinPerThread (the table's chunk minima).
    for (int k0 = threadIdx.x + blockDim.x * kMinPerThread; k0 < search_grid; k0 += blockDim.x * kMinPerThread) {
        uint32_t v[kMinPerThread];
#pragma unroll
        for (int u = 0; u < kMinPerThread; u++) {
            const int k = k0 + u * (int)blockDim.x;
            v[u] = k < search_grid ? wg_min[k] : 0xFFFFFFFFu;
        }
#pragma unroll
        for (int u = 0; u < kMinPerThread; u++) m = v[u] < m ? v[u] : m;
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(m, d);
        m = o < m ? o : m;
    }
    if ((threadIdx.x & 63) == 0) s_min[threadIdx.x >> 6] = m;
    __syncthreads();
    m = s_min[0];
    for (int k = 1; k < (int)(blockDim.x >> 6); k++) m = s_min[k] < m ? s_min[k] : m;
    if (b >= B) return;
    w[b] = (pb == 0u || m == 0u) ? 0.0f : is_weight(m, pb, beta);
}

constexpr int kSmallThreads = 1024;
constexpr int kSmallPerThread = (int)(kSmallN / kSmallThreads);  // consecutive priorities per thread
static_assert(kSmallN % (4 * kSmallThreads) == 0, "whole 16-byte loads per thread");

// LDS position of prefix entry e: one pad word after every run of
// kSmallPerThread entries, so that the lanes of a wave, each writing its own
// consecutive run, fall in different banks.
__device__ __forceinline__ int64_t small_pos(int64_t e) { return e + e / kSmallPerThread; }

// want_w: also compute weights (the selected priority waits in w[b] as
// uint32 bits, as in the multi-launch path).  global_min: normalise by the
// smallest non-zero priority of the table instead of the batch's.
__global__ __launch_bounds__(kSmallThreads) void small_select_kernel(const uint32_t* __restrict__ prio, int64_t N,
                                                                     int32_t B, uint64_t span, uint64_t seed,
                                                                     int want_w, int global_min, double beta,
                                                                     uint32_t* status, int64_t* __restrict__ idx,
                                                                     int32_t* __restrict__ start,
                                                                     float* __restrict__ w) {
    __shared__ uint64_t C[kSmallN + kSmallN / kSmallPerThread];
    __shared__ uint64_t s_wave[kSmallThreads / 64];
    __shared__ uint32_t s_min[kSmallThreads / 64];
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int64_t e0 = (int64_t)t * kSmallPerThread;
    uint32_t v[kSmallPerThread];
#pragma unroll
    for (int k = 0; k < kSmallPerThread; k += 4) {
        if (e0 + k + 4 <= N) {
            const uint4 x = *reinterpret_cast<const uint4*>(prio + e0 + k);
            v[k] = x.x; v[k + 1] = x.y; v[k + 2] = x.z; v[k + 3] = x.w;
        } else {
#pragma unroll
            for (int q = 0; q < 4; q++) v[k + q] = e0 + k + q < N ? prio[e0 + k + q] : 0u;
        }
    }
    // Block-wide inclusive scan: this thread's run, then the waves in order.
    uint64_t run = 0;
    uint32_t pmin = 0xFFFFFFFFu;  // smallest non-zero priority of this thread's run
#pragma unroll
    for (int k = 0; k < kSmallPerThread; k++) {
        run += v[k];
        pmin = (v[k] != 0u && v[k] < pmin) ? v[k] : pmin;
    }
    const uint64_t incl = wave_inclusive_scan(run);
    if (lane == 63) s_wave[wave] = incl;
    __syncthreads();
    uint64_t acc = incl - run;
    for (int q = 0; q < wave; q++) acc += s_wave[q];
#pragma unroll
    for (int k = 0; k < kSmallPerThread; k++) {
        acc += v[k];
        if (e0 + k < N) C[small_pos(e0 + k)] = acc;
    }
    __syncthreads();
    const uint64_t S = C[small_pos(N - 1)];
    uint32_t m = 0xFFFFFFFFu;  // smallest selected priority (or of the table)
    for (int64_t b = t; b < B; b += kSmallThreads) {
        if (S == 0) {
            idx[b] = -1;
            start[b] = 0;
            if (want_w) reinterpret_cast<uint32_t*>(w)[b] = 0u;
            if (b == 0) atomicOr(status, GEAR_STATUS_NO_WEIGHT);
            continue;
        }
        const uint64_t r = scale_draw(splitmix64_out(seed, 2 * (uint64_t)b), S);
        int64_t lo = 0, hi = N;  // the smallest i with C_i > r lies in [lo, hi]
        while (lo < hi) {
            const int64_t mid = (lo + hi) >> 1;
            if (C[small_pos(mid)] > r) hi = mid;
            else lo = mid + 1;
        }
        const uint32_t pv = (uint32_t)(C[small_pos(lo)] - (lo > 0 ? C[small_pos(lo - 1)] : 0));
        idx[b] = lo;
        start[b] = (int32_t)scale_draw(splitmix64_out(seed, 2 * (uint64_t)b + 1), span);
        if (want_w) reinterpret_cast<uint32_t*>(w)[b] = pv;
        m = pv < m ? pv : m;
    }
    if (!want_w) return;
    if (global_min) m = pmin;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const uint32_t o = __shfl_xor(m, d);
        m = o < m ? o : m;
    }
    if (lane == 0) s_min[wave] = m;
    __syncthreads();
    m = s_min[0];
    for (int q = 1; q < kSmallThreads / 64; q++) m = s_min[q] < m ? s_min[q] : m;
    for (int64_t b = t; b < B; b += kSmallThreads) {
        const uint32_t pb = reinterpret_cast<const uint32_t*>(w)[b];
        w[b] = (pb == 0u || m == 0u) ? 0.0f : is_weight(m, pb, beta);
    }
}

// FIFO / LIFO: ring arithmetic from the oldest / newest live position.
// Uniform: r = floor(u * n / 2^64) over the n live trajectories.
// A ring table's positions are its slots, and its live slots are [0, n).
// A managed table (index manager) reads the slot at each position of its
// commit-order ring `order`, oldest commit at `oldest`.
__global__ void simple_select_kernel(SimpleDraws d, int32_t B, int64_t* __restrict__ idx,
                                     int32_t* __restrict__ start, float* __restrict__ w) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    idx[b] = simple_slot(d, b);
    start[b] = simple_start(d, b);
    if (w) w[b] = 1.0f;
}

// The tree as the search sees it: of level 2, the copy the last scan filled.
Levels tree(const Table& t) {
    Levels lv{};
    lv.nlevels = t.nlevels;
    for (int l = 0; l < t.nlevels; l++) {
        lv.level[l] = l == 0 ? t.tile_sums : l == 1 ? t.chunk_sums : t.upper[t.tree_parity];
        lv.size[l] = t.level_size[l];
    }
    return with_top(lv);
}

}  // namespace

hipError_t launch_scan(Table& t, hipStream_t s) {
    // The level-2 copy this scan fills was zeroed by the previous scan (or at
    // creation); this scan zeroes the other copy for the next one.
    const int par = 1 - t.tree_parity;
    hipLaunchKernelGGL(scan_variant((t.options & GEAR_OPT_IS_GLOBAL_MIN) != 0, t.N), dim3((unsigned)t.nchunks),
                       dim3(scan_threads(t.N)), 0, s, t.priority, t.N, t.upper[par], t.upper[1 - par], t.tile_sums,
                       t.ntiles, t.chunk_sums, t.chunk_min);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) t.tree_parity = par;
    return e;
}

hipError_t launch_search(Table& t, int32_t B, int32_t L, uint64_t seed, bool want_min, int64_t* idx,
                         int32_t* start, uint32_t* sel_prio, int* grid_out, hipStream_t s,
                         const uint64_t* shard_totals, int G, int g, int64_t base) {
    const int grid = search_grid(B);
    Shard sh;
    sh.totals = shard_totals;
    sh.G = G;
    sh.g = g;
    sh.base = base;
    const SearchKernel kernel = search_variant(shard_totals != nullptr, t.N, t.nlevels);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(kSearchThreads), 0, s, t.priority, t.N, tree(t), B,
                       (uint64_t)(t.T - L + 1), seed, want_min ? 1 : 0, sh, t.wg_min, t.status, idx, start, sel_prio);
    *grid_out = grid;
    return hipGetLastError();
}

hipError_t launch_is_weights(Table& t, int32_t B, float beta, int search_grid, float* w, hipStream_t s,
                             bool global_min) {
    // The minimum comes from the search's per-workgroup minima of the batch,
    // or from the scan's per-chunk minima of the whole table.
    hipLaunchKernelGGL(is_weights_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, B, (double)beta,
                       global_min ? t.chunk_min : t.wg_min, global_min ? (int)t.nchunks : search_grid, w);
    return hipGetLastError();
}

bool small_select_applies(const Table& t, int32_t B) {
    return t.N <= kSmallN && B <= kSmallMaxB && !(t.options & GEAR_OPT_INCREMENTAL_TREE);
}

hipError_t launch_small_select(Table& t, int32_t B, int32_t L, uint64_t seed, float beta, int64_t* idx,
                               int32_t* start, float* w, hipStream_t s) {
    hipLaunchKernelGGL(small_select_kernel, dim3(1), dim3(kSmallThreads), 0, s, t.priority, t.N, B,
                       (uint64_t)(t.T - L + 1), seed, w ? 1 : 0, (t.options & GEAR_OPT_IS_GLOBAL_MIN) ? 1 : 0,
                       (double)beta, t.status, idx, start, w);
    return hipGetLastError();
}

SimpleDraws simple_draws(const Table& t, int32_t strategy, int32_t L, uint64_t seed) {
    SimpleDraws d{};
    d.strategy = strategy;
    d.N = t.N;
    d.live = live_count(t);
    if (t.managed) {
        d.oldest = t.ord_head;
        d.newest = (t.ord_head + d.live - 1) % t.N;
    } else {
        d.oldest = (int64_t)((t.next_seq - (uint64_t)d.live) % (uint64_t)t.N);
        d.newest = (int64_t)((t.next_seq - 1) % (uint64_t)t.N);
    }
    d.order = t.managed ? t.order : nullptr;
    d.span = (uint64_t)(t.T - L + 1);
    d.seed = seed;
    return d;
}

hipError_t launch_simple_select(Table& t, int32_t strategy, int32_t B, int32_t L, uint64_t seed, int64_t* idx,
                                int32_t* start, float* w, hipStream_t s) {
    hipLaunchKernelGGL(simple_select_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s,
                       simple_draws(t, strategy, L, seed), B, idx, start, w);
    return hipGetLastError();
}

}  // namespace gear

using gear::fail;
using gear::hip_fail;

extern "C" int gear_select(gear_table* h, int32_t strategy, int32_t B, int32_t L, uint64_t seed, float beta,
                           int64_t* d_idx, int32_t* d_start, float* d_weights, void* stream) {
    if (h == nullptr) return fail(GEAR_E_INVAL, "gear_select: table is NULL");
    gear::Table* t = reinterpret_cast<gear::Table*>(h);
    if (strategy < GEAR_FIFO || strategy > GEAR_TOPK) return fail(GEAR_E_INVAL, "gear_select: unknown strategy");
    if (strategy == GEAR_TOPK && B > GEAR_MAX_TOPK) return fail(GEAR_E_INVAL, "gear_select: TopK batch above GEAR_MAX_TOPK");
    if (B < 1 || B > GEAR_MAX_BATCH) return fail(GEAR_E_INVAL, "gear_select: B out of range");
    if (L < 1 || L > t->T) return fail(GEAR_E_INVAL, "gear_select: L must lie in [1, T]");
    if (d_idx == nullptr || d_start == nullptr) return fail(GEAR_E_INVAL, "gear_select: output pointer is NULL");
    if (!(beta == beta)) return fail(GEAR_E_INVAL, "gear_select: beta is NaN");
    const int64_t live = gear::live_count(*t);
    if (live == 0) return fail(GEAR_E_EMPTY, "gear_select: nothing inserted");
    if ((strategy == GEAR_FIFO || strategy == GEAR_LIFO) && (int64_t)B > live)
        return fail(GEAR_E_INSUFFICIENT, "gear_select: FIFO/LIFO batch larger than the live count");
    gear::DeviceGuard guard(t->device);
    if (guard.error() != hipSuccess) return hip_fail(guard.error(), "gear_select: hipSetDevice");
    hipStream_t s = static_cast<hipStream_t>(stream);

    if (strategy == GEAR_TOPK) {
        hipError_t e = gear::launch_topk(*t, B, L, seed, d_idx, d_start, d_weights, s);
        return e == hipSuccess ? GEAR_OK : hip_fail(e, "gear_select: TopK launch");
    }
    if (strategy != GEAR_PRIORITIZED) {
        hipError_t e = gear::launch_simple_select(*t, strategy, B, L, seed, d_idx, d_start, d_weights, s);
        return e == hipSuccess ? GEAR_OK : hip_fail(e, "gear_select: launch");
    }
    if (gear::small_select_applies(*t, B)) {
        // One launch; the sum tree is left as it is (still marked for a rescan if stale).
        hipError_t e = gear::launch_small_select(*t, B, L, seed, beta, d_idx, d_start, d_weights, s);
        return e == hipSuccess ? GEAR_OK : hip_fail(e, "gear_select: small-table launch");
    }
    if (t->cdf_dirty) {
        hipError_t e = gear::launch_scan(*t, s);
        if (e != hipSuccess) return hip_fail(e, "gear_select: scan launch");
        t->cdf_dirty = false;
    }
    const bool weights = d_weights != nullptr;
    int grid = 0;
    hipError_t e = gear::launch_search(*t, B, L, seed, weights, d_idx, d_start,
                                       reinterpret_cast<uint32_t*>(d_weights), &grid, s);
    if (e != hipSuccess) return hip_fail(e, "gear_select: search launch");
    if (weights) {
        e = gear::launch_is_weights(*t, B, beta, grid, d_weights, s, (t->options & GEAR_OPT_IS_GLOBAL_MIN) != 0);
        if (e != hipSuccess) return hip_fail(e, "gear_select: weight launch");
    }
    return GEAR_OK;
}

// ---------------------------------------------------------------------------
// Prioritized selection without allocation: the kernels above, run over a
// caller's priority array with the sum tree, the per-workgroup minima and
// the status word in a fixed file-scope device array instead of table
// memory.  For callers that cannot allocate (graph capture, serving loops).
// ---------------------------------------------------------------------------
namespace gear {
namespace {

constexpr int64_t kNaTiles = GEAR_NOALLOC_MAX_N / kTile;   // level 0 entries
constexpr int64_t kNaChunks = kTopMax;                       // level 1 entries (the highest level), at most
static_assert(GEAR_NOALLOC_MAX_N <= (int64_t)kTopMax * kLargeChunk * kTile, "two levels cover every allowed table");
// Layout in 64-bit words: tile sums | chunk sums | wg_min (uint32) | status
// (uint32; set by the kernels, never read).  Every call rewrites what it reads.
constexpr int64_t kNaOffTiles = 0;
constexpr int64_t kNaOffChunks = kNaOffTiles + kNaTiles;
constexpr int64_t kNaOffMin = kNaOffChunks + kNaChunks;
constexpr int64_t kNaOffStatus = kNaOffMin + kSearchMaxGrid / 2;
constexpr int64_t kNaWords = (kNaOffStatus + 1 + 31) / 32 * 32;
static_assert(kNaWords * 8 == GEAR_NOALLOC_SCRATCH_BYTES, "header states the scratch size");

// Holds every call's scratch on each device, until the process ends.
static __device__ __align__(256) uint64_t scratch[kNaWords];

// Device address of `scratch` on each device, looked up once per device
// with that device current (host code must not pass the symbol itself).
constexpr int kNaMaxDevices = 64;
std::mutex g_na_mutex;
uint64_t* g_na_ptr[kNaMaxDevices] = {};

hipError_t noalloc_scratch(int dev, uint64_t** out) {
    std::lock_guard<std::mutex> lock(g_na_mutex);
    if (g_na_ptr[dev] == nullptr) {
        void* p = nullptr;
        hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_na_ptr[dev] = static_cast<uint64_t*>(p);
    }
    *out = g_na_ptr[dev];
    return hipSuccess;
}

}  // namespace
}  // namespace gear

extern "C" int gear_select_prioritized_noalloc(const uint32_t* d_priority, int64_t N, int32_t T, int32_t B,
                                               int32_t L, uint64_t seed, float beta, int64_t* d_idx,
                                               int32_t* d_start, float* d_weights, void* stream) {
    using namespace gear;
    if (d_priority == nullptr || d_idx == nullptr || d_start == nullptr)
        return fail(GEAR_E_INVAL, "gear_select_prioritized_noalloc: NULL pointer argument");
    if (N < 1 || N > GEAR_NOALLOC_MAX_N)
        return fail(GEAR_E_INVAL, "gear_select_prioritized_noalloc: N must lie in [1, GEAR_NOALLOC_MAX_N]");
    if (B < 1 || B > GEAR_MAX_BATCH) return fail(GEAR_E_INVAL, "gear_select_prioritized_noalloc: B out of range");
    if (T < 1 || L < 1 || L > T) return fail(GEAR_E_INVAL, "gear_select_prioritized_noalloc: L must lie in [1, T]");
    if (!(beta == beta)) return fail(GEAR_E_INVAL, "gear_select_prioritized_noalloc: beta is NaN");
    (void)hipGetLastError();  // an error pending from an earlier HIP call is not this call's
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return hip_fail(e, "gear_select_prioritized_noalloc: hipGetDevice");
    if (dev < 0 || dev >= kNaMaxDevices) return fail(GEAR_E_INVAL, "gear_select_prioritized_noalloc: device ordinal above 63");
    uint64_t* base = nullptr;
    e = noalloc_scratch(dev, &base);
    if (e != hipSuccess) return hip_fail(e, "gear_select_prioritized_noalloc: hipGetSymbolAddress");
    uint32_t* status = reinterpret_cast<uint32_t*>(base + kNaOffStatus);
    uint32_t* wg_min = reinterpret_cast<uint32_t*>(base + kNaOffMin);
    hipStream_t s = static_cast<hipStream_t>(stream);
    const uint64_t span = (uint64_t)(T - L + 1);

    if (N <= kSmallN && B <= kSmallMaxB) {
        // One launch, as gear_select takes for a table this small.
        hipLaunchKernelGGL(small_select_kernel, dim3(1), dim3(kSmallThreads), 0, s, d_priority, N, B, span, seed,
                           d_weights ? 1 : 0, 0, (double)beta, status, d_idx, d_start, d_weights);
        e = hipGetLastError();
        return e == hipSuccess ? GEAR_OK : hip_fail(e, "gear_select_prioritized_noalloc: small-table launch");
    }
    const int64_t ntiles = (N + kTile - 1) / kTile;
    const int64_t nchunks = (ntiles + tiles_per_chunk(N) - 1) / tiles_per_chunk(N);
    Levels lv{};
    lv.nlevels = 2;
    lv.level[0] = base + kNaOffTiles;
    lv.size[0] = ntiles;
    lv.level[1] = base + kNaOffChunks;
    lv.size[1] = nchunks;
    const char* what = "gear_select_prioritized_noalloc: scan launch";
    hipLaunchKernelGGL(scan_variant(false, N), dim3((unsigned)nchunks), dim3(scan_threads(N)), 0, s, d_priority, N,
                       static_cast<uint64_t*>(nullptr), static_cast<uint64_t*>(nullptr), lv.level[0], ntiles,
                       lv.level[1], static_cast<uint32_t*>(nullptr));
    e = hipGetLastError();
    const int grid = search_grid(B);
    if (e == hipSuccess) {
        what = "gear_select_prioritized_noalloc: search launch";
        Shard sh{};
        sh.G = 1;
        hipLaunchKernelGGL(search_variant(false, N, 2), dim3(grid), dim3(kSearchThreads), 0, s, d_priority, N,
                           with_top(lv), B, span, seed, d_weights ? 1 : 0, sh, wg_min, status, d_idx, d_start,
                           reinterpret_cast<uint32_t*>(d_weights));
        e = hipGetLastError();
    }
    if (e == hipSuccess && d_weights) {
        what = "gear_select_prioritized_noalloc: weight launch";
        hipLaunchKernelGGL(is_weights_kernel, dim3((unsigned)((B + 255) / 256)), dim3(256), 0, s, B, (double)beta,
                           static_cast<const uint32_t*>(wg_min), grid, d_weights);
        e = hipGetLastError();
    }
    return e == hipSuccess ? GEAR_OK : hip_fail(e, what);
}
