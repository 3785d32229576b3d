// Priority update on gfx950 (GEAR Sec. 3.2: the status table holds the
// priorities, and changes to it are gathered and then applied).
//
// The batch is applied as if in order, so for a slot that appears several
// times the last occurrence's value wins.
//
// Batches of up to 8192 run in one launch of 64 workgroups.  Workgroup g owns
// the slots whose hash falls in partition g: it reads the whole batch, lists
// its draws, and enters each into an open-addressing hash table in LDS, whose
// entry for a slot holds b+1 of the last draw that has it (LDS atomic max);
// after a barrier the draw that its slot's entry names writes the new priority.
// Every occurrence of a slot lands in the same workgroup, so no other
// synchronisation is needed.
//
// Larger batches use two kernels over a table-owned tag array:
//   tag    every draw b raises tag[slot] to b+1 (atomic max), so after the
//          kernel tag[slot] names the last occurrence of that slot;
//   apply  the draw whose b+1 equals tag[slot] writes the new priority and
//          puts the tag back to zero.  Other draws of the same slot see
//          either the winner's tag or zero, never their own, so they never
//          write.  Tags are zero again when the kernel ends.
//
// When the table keeps its selection sum tree up to date across updates,
// each writing draw also adds new - old (mod 2^64) into its tile's sum and
// into the covering node of every upper level.  Exactly one draw writes each
// changed slot, so the tree stays equal to the sums of the priorities.  In
// the one-launch path the upper-level additions of a workgroup are first
// combined per node in LDS (levels of at most 1024 nodes), so each node sees
// at most one global atomic per workgroup.
#include "gear_internal.h"

namespace gear {
namespace {

constexpr int kHashThreads = 1024;
constexpr int kHashMaxBatch = 8 * kHashThreads;     // draws of the one-launch path
constexpr int kAggNodes = 1024;                     // level-1 nodes combined in LDS, when there are no more
constexpr int kLevel2Max = GEAR_MAX_CAPACITY >> 22; // level-2 nodes, always combined in LDS

struct Tree {
    uint64_t* tile_sums;             // level 0
    uint64_t* upper[kMaxLevels];     // levels 1 .. nlevels-1 (of level 2, the copy the last scan filled)
    int64_t size[kMaxLevels];
    int nlevels;
    int chunk_shift;                 // a level-1 node covers 2^chunk_shift slots, a level-2 node 2^22
    int maintain;                    // 0: leave the tree alone
};

__device__ inline void add_u64(uint64_t* p, uint64_t d) {
    atomicAdd(reinterpret_cast<unsigned long long*>(p), (unsigned long long)d);
}

// Adds d into the level-1 and level-2 nodes covering `slot`.  Written out per
// level: from a loop over the levels the compiler formed one induction variable
// for the shift and for the address of tree.upper[l], and read the pointer with
// a scalar load of base + 14 and offset 0x32, whose two lowest address bits the
// hardware drops from each part.
constexpr int kLevel2Shift = 22;
static_assert(kTile * kLargeChunk * kFanout == 1 << kLevel2Shift, "slots per level-2 node");
__device__ __forceinline__ void add_upper(const Tree& tree, int64_t slot, uint64_t d) {
    add_u64(tree.upper[1] + (slot >> tree.chunk_shift), d);
    if (tree.nlevels == 3) add_u64(tree.upper[2] + (slot >> kLevel2Shift), d);
}
static_assert(kMaxLevels == 3, "levels 1 and 2 are written out");
static_assert(kLevel2Max <= kHashThreads, "one thread per level-2 node");

// `live`: indices at or past it are invalid.  `committed` (managed tables
// only, else NULL): an index whose flag is 0 is released or still being
// written; its update is dropped, so it never becomes selectable.
//
// kHashThreads * kPerThread draws at most, in 2^part_bits workgroups.  With one
// draw per thread a thread keeps its own; with more, the draws of the partition
// are listed first, so that the code behind exists once and not per draw: an
// earlier kernel that unrolled all of it over eight draws was bound by fetching
// its instructions and took the same 4.5 us for 1 draw as for 1000.  Replayed
// from a graph, before -> after: 256 draws 4.5 -> 2.4 us, 1000 4.6 -> 2.7, 3001
// 5.0 -> 3.6, 8192 6.4 -> 4.9; keeping the tree, 256 5.3 -> 3.0, 8192 8.3 -> 6.0.
template <int kPerThread>
__global__ __launch_bounds__(kHashThreads) void scatter_lds_kernel(const int64_t* __restrict__ idx,
                                                                   const uint32_t* __restrict__ newp, int32_t B,
                                                                   int64_t live, const uint8_t* __restrict__ committed,
                                                                   uint32_t* __restrict__ prio, uint32_t* status,
                                                                   int part_bits, Tree tree) {
    constexpr int kThreads = kHashThreads;
    constexpr int kMost = kThreads * kPerThread;  // a partition may hold every draw
    constexpr int kSize = 2 * kMost;              // hash entries: load factor <= 1/2
    constexpr int kBits = __builtin_ctz(kSize);
    constexpr bool kList = kPerThread > 1;
    __shared__ __align__(16) uint32_t last[kSize];    // b + 1 of the last draw seen of the entry's slot, 0 if free
    __shared__ uint32_t own_slot[kMost];              // slot of draw b, for draws of this partition
    __shared__ uint16_t own_b[kList ? kMost : 1];     // those draws, in any order
    __shared__ int n_own;
    __shared__ uint64_t agg1[kAggNodes];              // additions to level 1 and level 2
    __shared__ uint64_t agg2[kLevel2Max];
    const bool in_lds = tree.size[1] <= kAggNodes;
    // The batch's loads first, from indices clamped into it: the tables are
    // cleared while they are on their way.
    int64_t slot[kPerThread];
#pragma unroll
    for (int k = 0; k < kPerThread; k++) {
        const int b = threadIdx.x + k * kThreads;
        slot[k] = idx[b < B ? b : B - 1];
    }
    if (kList && threadIdx.x == 0) n_own = 0;
    for (int h = threadIdx.x * 4; h < kSize; h += kThreads * 4)
        *reinterpret_cast<uint4*>(&last[h]) = make_uint4(0u, 0u, 0u, 0u);
    if (tree.maintain) {
        for (int m = threadIdx.x; m < kAggNodes; m += kThreads) agg1[m] = 0;
        if (threadIdx.x < kLevel2Max) agg2[threadIdx.x] = 0;
    }
    if (kList) __syncthreads();
    bool bad = false;
    int n = 0;  // own draws of the workgroup; without a list, 1 for a thread that has one
#pragma unroll
    for (int k = 0; k < kPerThread; k++) {
        const int b = threadIdx.x + k * kThreads;
        const bool valid = slot[k] >= 0 && slot[k] < live;
        bad = bad || !valid;  // a clamped index repeats the batch's last draw
        if (b < B && valid && ((uint32_t)slot[k] * 0x85EBCA6Bu) >> (32 - part_bits) == blockIdx.x) {
            own_slot[b] = (uint32_t)slot[k];
            if (kList) own_b[atomicAdd(&n_own, 1)] = (uint16_t)b;
            else n = (int)threadIdx.x + 1;
        }
    }
    __syncthreads();
    if (kList) n = n_own;
    // Value and old priority of this thread's first own draw (usually the
    // only one), issued before the hash phase and used after it.
    const int i0 = threadIdx.x;
    uint32_t val0 = 0, old0 = 0;
    if (i0 < n) {
        const int b = kList ? own_b[i0] : i0;
        val0 = newp[b];
        old0 = tree.maintain ? prio[own_slot[b]] : 0u;
    }
    for (int i = i0; i < n; i += kThreads) {
        const int b = kList ? own_b[i] : i;
        const uint32_t s = own_slot[b];
        if (committed != nullptr && committed[s] == 0) continue;
        uint32_t h = (s * 2654435761u) >> (32 - kBits);
        while (true) {  // at most kMost < kSize distinct slots, so a free or equal entry is found
            const uint32_t was = atomicCAS(&last[h], 0u, (uint32_t)b + 1);
            if (was == 0) break;
            if (own_slot[was - 1] == s) {  // an entry's slot never changes
                atomicMax(&last[h], (uint32_t)b + 1);
                break;
            }
            h = (h + 1) & (kSize - 1);
        }
    }
    __syncthreads();
    for (int i = i0; i < n; i += kThreads) {
        const int b = kList ? own_b[i] : i;
        const uint32_t s = own_slot[b];
        uint32_t h = (s * 2654435761u) >> (32 - kBits);
        uint32_t e;
        while ((e = last[h]) != 0 && own_slot[e - 1] != s) h = (h + 1) & (kSize - 1);
        if (e != (uint32_t)b + 1) continue;  // a later draw of the slot wins, or the update is dropped
        const uint32_t val = i == i0 ? val0 : newp[b];
        const uint32_t old = i == i0 ? old0 : tree.maintain ? prio[s] : 0u;
        prio[s] = val;
        if (!tree.maintain) continue;
        const uint64_t d = (uint64_t)val - (uint64_t)old;  // mod 2^64
        if (d == 0) continue;
        add_u64(tree.tile_sums + (s >> 8), d);
        if (in_lds) add_u64(&agg1[s >> tree.chunk_shift], d);
        else add_u64(tree.upper[1] + (s >> tree.chunk_shift), d);
        if (tree.nlevels == 3) add_u64(&agg2[s >> kLevel2Shift], d);
    }
    if (bad && blockIdx.x == 0) atomicOr(status, GEAR_STATUS_BAD_INDEX);
    if (!tree.maintain) return;
    __syncthreads();
    if (in_lds)
        for (int m = threadIdx.x; m < tree.size[1]; m += kThreads)
            if (agg1[m] != 0) add_u64(tree.upper[1] + m, agg1[m]);
    if (tree.nlevels == 3 && threadIdx.x < tree.size[2] && agg2[threadIdx.x] != 0)
        add_u64(tree.upper[2] + threadIdx.x, agg2[threadIdx.x]);
}

__global__ void scatter_tag_kernel(const int64_t* __restrict__ idx, int32_t B, int64_t live,
                                   const uint8_t* __restrict__ committed, uint32_t* tag, uint32_t* status) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int64_t i = idx[b];
    if (i < 0 || i >= live) {
        atomicOr(status, GEAR_STATUS_BAD_INDEX);
        return;
    }
    if (committed != nullptr && committed[i] == 0) return;
    atomicMax(tag + i, (uint32_t)(b + 1));
}

__global__ void scatter_apply_kernel(const int64_t* __restrict__ idx, const uint32_t* __restrict__ newp, int32_t B,
                                     int64_t live, uint32_t* tag, uint32_t* __restrict__ prio, Tree tree) {
    const int64_t b = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= B) return;
    const int64_t i = idx[b];
    if (i < 0 || i >= live) return;
    // Dropped updates of uncommitted slots never raised the tag, so it is 0.
    if (tag[i] == (uint32_t)(b + 1)) {
        const uint32_t old = prio[i];
        prio[i] = newp[b];
        tag[i] = 0;
        if (tree.maintain) {
            const uint64_t d = (uint64_t)newp[b] - (uint64_t)old;  // mod 2^64
            if (d != 0) {
                add_u64(tree.tile_sums + (i >> 8), d);
                add_upper(tree, i, d);
            }
        }
    }
}

Tree tree_of(const Table& t, bool maintain) {
    Tree tr{};
    tr.tile_sums = t.tile_sums;
    tr.nlevels = t.nlevels;
    for (int l = 0; l < t.nlevels; l++) {
        tr.upper[l] = l == 0 ? nullptr : l == 1 ? t.chunk_sums : t.upper[t.tree_parity];
        tr.size[l] = t.level_size[l];
    }
    tr.chunk_shift = tiles_per_chunk(t.N) == kSmallChunk ? 12 : 14;
    static_assert(kTile * kSmallChunk == 1 << 12 && kTile * kLargeChunk == 1 << 14, "slots per chunk");
    tr.maintain = maintain ? 1 : 0;
    return tr;
}

}  // namespace

hipError_t launch_scatter(Table& t, const int64_t* idx, const uint32_t* newp, int32_t B, bool maintain_tree,
                          hipStream_t s) {
    // Ring tables: slots [0, live count); managed tables: any slot, updates
    // of uncommitted ones dropped.
    const int64_t live = t.managed ? t.N : live_count(t);
    const uint8_t* committed = t.managed ? t.committed : nullptr;
    const Tree tree = tree_of(t, maintain_tree);
    if (B <= kHashMaxBatch) {
        // 64 workgroups, or 32 where each also adds its nodes' sums into the
        // tree (8192 draws: 64 / 32 workgroups 4.9 / 5.0 us without the tree,
        // 6.3 / 6.0 with it; 128 gain 0.1 us and hold twice as many CUs' LDS).
        const int bits = maintain_tree ? 5 : 6;
        const auto kernel = B <= kHashThreads       ? scatter_lds_kernel<1>
                            : B <= 2 * kHashThreads ? scatter_lds_kernel<2>
                            : B <= 4 * kHashThreads ? scatter_lds_kernel<4>
                                                    : scatter_lds_kernel<8>;
        hipLaunchKernelGGL(kernel, dim3(1u << bits), dim3(kHashThreads), 0, s, idx, newp, B, live, committed,
                           t.priority, t.status, bits, tree);
        return hipGetLastError();
    }
    const unsigned grid = (unsigned)((B + 255) / 256);
    hipLaunchKernelGGL(scatter_tag_kernel, dim3(grid), dim3(256), 0, s, idx, B, live, committed, t.tag, t.status);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(scatter_apply_kernel, dim3(grid), dim3(256), 0, s, idx, newp, B, live, t.tag, t.priority,
                       tree);
    return hipGetLastError();
}

}  // namespace gear

using gear::fail;
using gear::hip_fail;

extern "C" int gear_update_priorities(gear_table* h, const int64_t* d_idx, const uint32_t* d_new_priorities,
                                      int32_t B, void* stream) {
    if (h == nullptr) return fail(GEAR_E_INVAL, "gear_update_priorities: table is NULL");
    gear::Table* t = reinterpret_cast<gear::Table*>(h);
    if (B < 0 || B > GEAR_MAX_BATCH) return fail(GEAR_E_INVAL, "gear_update_priorities: B out of range");
    if (B == 0) return GEAR_OK;
    if (d_idx == nullptr || d_new_priorities == nullptr)
        return fail(GEAR_E_INVAL, "gear_update_priorities: NULL pointer argument");
    gear::DeviceGuard guard(t->device);
    if (guard.error() != hipSuccess) return hip_fail(guard.error(), "gear_update_priorities: hipSetDevice");
    // Keep the tree current only if it is current now; otherwise the next
    // prioritized select rescans anyway.
    // Under global IS normalisation the next select rescans anyway, for the
    // chunk minima, so the tree is not maintained.
    const bool maintain = (t->options & GEAR_OPT_INCREMENTAL_TREE) && !(t->options & GEAR_OPT_IS_GLOBAL_MIN) &&
                          !t->cdf_dirty;
    hipError_t e = gear::launch_scatter(*t, d_idx, d_new_priorities, B, maintain, static_cast<hipStream_t>(stream));
    if (e != hipSuccess) return hip_fail(e, "gear_update_priorities: launch");
    if (!maintain) t->cdf_dirty = true;
    return GEAR_OK;
}
