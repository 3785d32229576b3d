// Window collection on gfx950 (GEAR Sec. 3.2 storage format; Sec. 3.4).
//
// For draw b, step t < L and requested column j:
//     out_j[b][t][:] = column c_j, block idx[b], step start[b] + t
// Each window is one contiguous byte range of its column,
//     base_c + (idx[b]*T + start[b]) * E_c,  length W_c = L * E_c,
// and each column's batch [B][L][E_c] is one contiguous range, so the copy
// is driven by the output: a workgroup owns a contiguous piece of one
// column's output.  Wide columns (a window at least a piece long) are cut
// into equal pieces of the whole batch, so a piece may run from the end of
// one window into the start of the next (never further); a launch of a few
// hundred MB then runs in equal pieces instead of ending on the short last
// pieces of every window.  Narrow windows are packed several to a piece with
// their source offsets staged in LDS.  All requested columns run in one
// launch.  A column table in pinned host memory is read by the same kernel
// through its mapped address, so the loads go over the host link without a
// CPU copy.
//
// gear_select_collect runs the same kernel for FIFO, LIFO or uniform draws
// (Sec. 3.3): instead of reading idx[b] and start[b], each piece computes its
// windows' draws from the ring state and the seed, and the piece holding a
// window's first element in the first requested column writes the draw's
// slot, start and weight.  A step then needs no separate selection launch.
//
// Element width per column.  Only the output decides it: window sources may
// start at any byte, since global loads on gfx950 take any address, and an
// unaligned wave load touches one cache line more than an aligned one.
//   16 bytes  when the batch is 16-byte aligned and a window is whole elements,
//             or holds at least kThreads * unroll * 16 / (kThreads - 2) bytes:
//             then some elements straddle two windows (copy_straddle);
//   4 bytes   when the batch and the window are multiples of 4;
//   1 byte    otherwise (small windows of odd size, unaligned batches).
// When sources had to be aligned too, steps of 147, 1, 2 and 1 bytes were
// gathered byte by byte: 3001 windows of 13 steps (5.9 MB) took 29.7 us, now
// 7.8.  512 windows of 20 steps of 68, 24, 4 and 4 bytes (4-byte elements
// before, 16-byte ones now) stayed at 5.7 us: they are bound by latency.
#include "gear_internal.h"

namespace gear {
namespace {

constexpr int kThreads = 256;
// Elements in flight per thread (U), so a piece is kThreads * U elements.
// HBM tables: 2, 8 KiB pieces of 16-byte elements, for every batch size.
// Measured on gfx950 in one process, variants alternating on one table and one
// set of output buffers (us, U = 2 / 4 / 8): windows of 32 steps of 1060 bytes,
// 2.2 MB 3.5 / 3.7 / 4.4, 68 MB 25.9 / 26.5 / 27.0, 278 MB 94.8 / 97.2 / 98.4;
// whole 100 KB trajectories, 51 MB 20.6 / 21.1 / 21.7, 205 MB 71.0 / 73.0 /
// 77.5 (before the lookups were batched, window_offsets, 278 MB took 103.6 us
// with 2 and 96.0 with 8).  Pinned host tables: 4 (8 was 4% slower over the
// host link; 2 no faster).
constexpr int kUnroll = 2;
constexpr int kUnrollHost = 4;
// A launch that mostly moves wide columns reserves LDS that it does not use,
// so that 7 of its workgroups share a CU (160 KiB) instead of 8: 278 MB 93.7
// instead of 94.8 us, 51 MB of whole trajectories 20.2 instead of 20.6, 34 MB
// 14.5 instead of 14.9; 6 per CU are slower again (94.5), and straddling or
// narrow columns want all 8 (93 MB of 147-byte steps 38.7 against 39.5, 33 MB
// of 1360-byte windows 17.5 against 17.8).  It also leaves room for kernels of
// other streams: with the next steps' selection beside it, the 278 MB step
// takes 99.6 us over 100 steps (101.0 with 32 KiB pieces, four per CU).
constexpr unsigned kWideLds = 19 * 1024;
// GEAR_OPT_GATHER_SHARE_CU makes long gathers run with 4 elements per thread
// and two workgroups per CU.  Beside such a gather selection and update take
// about half as long, while the gather takes 98.3 instead of 93.3 us (278 MB):
// worth it only while another stream has to catch up, as at the start of a
// pipeline (20 steps, the first three gathers like this: 104.6 us per step
// against 105.3).
constexpr unsigned kShareLds = 64 * 1024;
constexpr int kUnrollShare = kUnrollHost;
constexpr int64_t kLongBatch = 64ll << 20;
constexpr int kMaxLaunchCols = 16;  // columns per launch (more take several launches)

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

// How a column's batch is cut into pieces.
enum : int32_t {
    kNarrow = 0,    // several whole windows per piece
    kWide = 1,      // equal pieces of the batch, each within one or two windows of whole elements
    kStraddle = 2,  // equal pieces of the batch, an element may cover the end of one window and the start of the next
};

// One column's task: one 64-byte line of the kernel arguments.
struct alignas(64) ColTask {
    const uint8_t* src;   // device-visible column base
    uint8_t* out;         // batch output [B][W]
    int64_t W;            // window bytes, L*E
    int64_t n;            // elements per window, W / width
    uint64_t recip;       // floor((2^64 - 1) / n) (wide) or / W (straddle), for quotient()
    int32_t E;            // bytes per step
    uint32_t epw;         // elements per window (narrow)
    uint32_t magic;       // narrow: ceil(2^32 / epw) for epw > 1; straddle: ceil(2^32 / W), or 0 when a
                          // window holds at least a piece: exact quotient for operands < 2^16
    uint16_t wpp;         // windows per piece (narrow)
    uint8_t width;        // element bytes: 16, 4 or 1
    uint8_t layout : 4;   // kNarrow, kWide or kStraddle
    uint8_t draws_out : 4;  // 1: this column's pieces write the selected slots, starts and weights
    int64_t pad;
};
static_assert(sizeof(ColTask) == 64, "one line per column");

// A gather that selects its own windows (FIFO, LIFO or uniform draws): a
// kernel argument of its own, beside CollectArgs.
struct DrawArgs {
    SimpleDraws draws;      // the windows, computed per piece
    int64_t* idx_out;       // the draws, written by the pieces of a draws_out column
    int32_t* start_out;
    float* w_out;           // ... and weight 1 per draw, when not NULL
};

// A workgroup finds its column from the first line alone and then reads that
// column's line: two rounds of scalar loads before its window offsets, where a
// walk over the columns took one round per column (the two together with
// kernels that hold only the code their columns need: 512 windows of 20 steps
// of 68, 24, 4 and 4 bytes 4.3 -> 3.6 us).
struct CollectArgs {
    int32_t task0[kMaxLaunchCols];  // first task of each column, counted from the launch's first (negative in
                                    // the later launches of a batch cut over several); INT32_MAX past the last
    const int64_t* idx;     // the caller's draws, unless the pieces compute them
    const int32_t* start;
    uint32_t* status;
    int64_t N;
    int32_t B;
    int32_t T;
    int32_t L;
    ColTask col[kMaxLaunchCols];
};

// floor(x / n) for x < 2^63 from recip = floor((2^64 - 1) / n): the high word of
// the product is at most one short.
__device__ __forceinline__ int64_t quotient(int64_t x, int64_t n, uint64_t recip) {
    const int64_t q = (int64_t)__umul64hi((uint64_t)x, recip);
    return x - q * n >= n ? q + 1 : q;
}

// Element types: `type` in the batch (aligned), `src` in a column (any address).
template <int WIDTH>
struct Elem;
template <>
struct Elem<16> {
    typedef u32x4 type;
    typedef u32x4 src __attribute__((aligned(1)));
};
template <>
struct Elem<4> {
    typedef uint32_t type;
    typedef uint32_t src __attribute__((aligned(1)));
};
template <>
struct Elem<1> {
    typedef uint8_t type;
    typedef uint8_t src;
};

// Table bytes are read once per collection and the batch is written once:
// loads and stores are both non-temporal.  Measured on gfx950 with the
// MAT-shaped batch (278 MB each way) and output buffers that alternate, so
// that no batch line is still cached from an earlier launch: 89.8 us with
// non-temporal stores against 94.8 us with plain ones, level with a plain
// copy of the same bytes.  Plain stores win (81 us) only when the same
// output buffer is rewritten while the last-level cache still holds it.
template <int WIDTH>
__device__ inline typename Elem<WIDTH>::type load_stream(const uint8_t* p) {
    return __builtin_nontemporal_load(reinterpret_cast<const typename Elem<WIDTH>::src*>(p));
}

template <int WIDTH>
__device__ inline void store_stream(typename Elem<WIDTH>::type* p, typename Elem<WIDTH>::type v) {
    __builtin_nontemporal_store(v, p);
}

template <int WIDTH>
__device__ inline typename Elem<WIDTH>::type zero_elem() {
    return typename Elem<WIDTH>::type(0);
}

// Element k (< U) of this thread within its piece of kThreads * U elements.
// Each wave owns 64 * U consecutive elements and its k-th load covers the
// k-th 64 of them, so every wave reads and writes one contiguous run instead
// of the four waves interleaving every 64 elements.  On gfx950 a 278 MB copy
// with 4 KiB per wave took 88.5-88.9 us, against 96.4-96.9 us with 32 KiB
// pieces interleaved that way.  In the gather it is worth less: the MAT
// batch with 8 elements per thread 91.1-96.0 us against 91.2-96.7
// interleaved (two machines), and no difference next to another stream's
// selection; the DT-shaped batch with 2, 20.6 against 20.9 us.
template <int U>
__device__ __forceinline__ int64_t lane_elem(int k) {
    return (int64_t)(threadIdx.x >> 6) * (64 * U) + k * 64 + (threadIdx.x & 63);
}

// Source byte offset of window b's first step; kNoWindow for index -1 (a
// draw with no trajectory: a missing TopK entry, a draw another shard
// owns), kBadWindow for an index or start out of range.  Both read as zeros.
constexpr int64_t kNoWindow = -1;
constexpr int64_t kBadWindow = -2;

__device__ __forceinline__ int64_t draw_offset(const CollectArgs& a, const ColTask& c, int64_t i, int32_t s) {
    // Unsigned: an invalid index may wrap, and its product is not used.
    const int64_t off = (int64_t)(((uint64_t)i * (uint64_t)a.T + (uint64_t)s) * (uint64_t)c.E);
    const bool ok = (i >= 0) & (i < a.N) & (s >= 0) & (s <= a.T - a.L);
    return ok ? off : i == -1 ? kNoWindow : kBadWindow;
}

// Offsets of windows b and b2 (one lane's, or the workgroup's).  The draws'
// loads are all issued before any is used: left to the compiler, a start's
// load stood behind the test of its index, and the second window's behind the
// first's, a memory round trip each (512 windows of 20 steps of 68, 24, 4 and 4
// bytes: 3.5 instead of 3.6 us; 3001 of 13 steps of 147, 1, 2 and 1: 6.3
// instead of 6.7).
template <bool DRAWS>
__device__ __forceinline__ void window_offsets(const CollectArgs& a, const DrawArgs& g, const ColTask& c, int64_t b,
                                               int64_t b2, int64_t& off, int64_t& off2) {
    if (DRAWS) {
        off = (simple_slot(g.draws, b) * a.T + simple_start(g.draws, b)) * c.E;
        off2 = (simple_slot(g.draws, b2) * a.T + simple_start(g.draws, b2)) * c.E;
        return;
    }
    const int64_t i = a.idx[b], i2 = a.idx[b2];
    const int32_t s = a.start[b], s2 = a.start[b2];
    asm volatile("" ::"v"(i), "v"(i2), "v"(s), "v"(s2));
    off = draw_offset(a, c, i, s);
    off2 = draw_offset(a, c, i2, s2);
}

template <bool DRAWS>
__device__ __forceinline__ int64_t window_offset(const CollectArgs& a, const DrawArgs& g, const ColTask& c,
                                                 int64_t b) {
    if (DRAWS) return (simple_slot(g.draws, b) * a.T + simple_start(g.draws, b)) * c.E;
    const int64_t i = a.idx[b];
    const int32_t s = a.start[b];
    asm volatile("" ::"v"(i), "v"(s));
    return draw_offset(a, c, i, s);
}

// A gather that selects its own windows writes draw b's slot, start and
// weight once: from the piece of the draws_out column that holds the
// window's first element.
__device__ __forceinline__ void write_draw(const DrawArgs& g, int64_t b) {
    g.idx_out[b] = simple_slot(g.draws, b);
    g.start_out[b] = simple_start(g.draws, b);
    if (g.w_out) g.w_out[b] = 1.0f;
}

// Piece q of a wide column: output elements [q*P, q*P + m) of the column's
// batch, P = kThreads * U, m = P except in the batch's last piece.  A
// window has n >= P elements, so the piece lies in window w0 from element r0
// on and, if r0 + m > n, runs into window w0 + 1.
template <int WIDTH, int U, bool DRAWS>
__device__ void copy_wide(const CollectArgs& a, const DrawArgs& g, const ColTask& c, int64_t q) {
    typedef typename Elem<WIDTH>::type V;
    constexpr int64_t P = (int64_t)kThreads * U;
    const int64_t o0 = q * P;
    const int64_t w0 = quotient(o0, c.n, c.recip);
    const int64_t r0 = o0 - w0 * c.n;
    const int64_t total = (int64_t)a.B * c.n;
    const int64_t m = (total - o0) < P ? (total - o0) : P;
    const bool two = r0 + m > c.n;
    int64_t so0, so1 = kNoWindow;
    if (two) window_offsets<DRAWS>(a, g, c, w0, w0 + 1, so0, so1);
    else so0 = window_offset<DRAWS>(a, g, c, w0);
    if (threadIdx.x == 0 && (so0 == kBadWindow || so1 == kBadWindow)) atomicOr(a.status, GEAR_STATUS_BAD_INDEX);
    if (DRAWS && c.draws_out && threadIdx.x == 0) {  // a piece holds at most one window's first element
        if (r0 == 0) write_draw(g, w0);
        else if (two) write_draw(g, w0 + 1);
    }
    V* dst = reinterpret_cast<V*>(c.out) + o0;
    // Byte offsets of the two windows' sources, shifted so that element r of
    // the piece (r = r0 + e) reads base + r * WIDTH in either window.
    const int64_t b0 = so0, b1 = so1 - c.W;
    V v[U];
    if (m == P && so0 >= 0 && (!two || so1 >= 0)) {
        // Every element valid: the loads go out unconditionally, all in flight.
#pragma unroll
        for (int k = 0; k < U; k++) {
            const int64_t r = r0 + lane_elem<U>(k);
            v[k] = load_stream<WIDTH>(c.src + (r < c.n ? b0 : b1) + r * WIDTH);
        }
#pragma unroll
        for (int k = 0; k < U; k++) store_stream<WIDTH>(dst + lane_elem<U>(k), v[k]);
        return;
    }
    // The batch's last piece, or a piece touching a missing or invalid
    // window (whose elements are zero).
#pragma unroll
    for (int k = 0; k < U; k++) {
        const int64_t e = lane_elem<U>(k);
        const int64_t r = r0 + e;
        const bool second = r >= c.n;
        v[k] = zero_elem<WIDTH>();
        if (e < m && (second ? so1 : so0) >= 0) v[k] = load_stream<WIDTH>(c.src + (second ? b1 : b0) + r * WIDTH);
    }
#pragma unroll
    for (int k = 0; k < U; k++) {
        const int64_t e = lane_elem<U>(k);
        if (e < m) store_stream<WIDTH>(dst + e, v[k]);
    }
}

// The windows of a narrow or straddling piece, shared by the workgroup.  One
// object for every kind of piece, so that the kernel's LDS stays at 2 KB and
// kWideLds, kShareLds alone set how many workgroups share a CU.
struct Staged {
    int64_t off[kThreads];         // source byte offset per window, negative if it reads as zeros
    uint32_t flags[kThreads / 64];  // per wave: kStagedBad, kStagedZeros
};
constexpr uint32_t kStagedBad = 1;    // a window is invalid
constexpr uint32_t kStagedZeros = 2;  // a window reads as zeros

// Stages windows b0 .. b0 + n - 1, one per thread, behind one barrier; returns
// the flags of all of them.  Window k writes its draw when k >= first_draw.
template <bool DRAWS>
__device__ __forceinline__ uint32_t stage_windows(const CollectArgs& a, const DrawArgs& g, const ColTask& c, int64_t b0,
                                                  int n, int first_draw, Staged& st) {
    int64_t so = 0;
    if ((int)threadIdx.x < n) {
        so = window_offset<DRAWS>(a, g, c, b0 + threadIdx.x);
        st.off[threadIdx.x] = so;
        if (DRAWS && c.draws_out && (int)threadIdx.x >= first_draw) write_draw(g, b0 + threadIdx.x);
    }
    const uint32_t mine = (__ballot(so == kBadWindow) ? kStagedBad : 0u) | (__ballot(so < 0) ? kStagedZeros : 0u);
    if ((threadIdx.x & 63) == 0) st.flags[threadIdx.x >> 6] = mine;
    __syncthreads();
    const uint32_t all = __builtin_amdgcn_readfirstlane(st.flags[0] | st.flags[1] | st.flags[2] | st.flags[3]);
    if (threadIdx.x == 0 && (all & kStagedBad)) atomicOr(a.status, GEAR_STATUS_BAD_INDEX);
    return all;
}
static_assert(kThreads == 256, "four waves' flags");

template <int WIDTH, int U, bool DRAWS>
__device__ void copy_narrow(const CollectArgs& a, const DrawArgs& g, const ColTask& c, int64_t q, Staged& st) {
    typedef typename Elem<WIDTH>::type V;
    const int64_t b0 = q * c.wpp;
    const int nb = (int)((a.B - b0) < c.wpp ? (a.B - b0) : c.wpp);
    stage_windows<DRAWS>(a, g, c, b0, nb, 0, st);
    const uint32_t total = (uint32_t)nb * c.epw;
    V* dst = reinterpret_cast<V*>(c.out) + b0 * (int64_t)c.epw;
    V v[U];
#pragma unroll
    for (int k = 0; k < U; k++) {
        const uint32_t e = (uint32_t)lane_elem<U>(k);
        v[k] = zero_elem<WIDTH>();
        if (e < total) {
            const uint32_t w = c.epw == 1 ? e : __umulhi(e, c.magic);
            const int64_t so = st.off[w];
            if (so >= 0) v[k] = load_stream<WIDTH>(c.src + so + (int64_t)(e - w * c.epw) * WIDTH);
        }
    }
#pragma unroll
    for (int k = 0; k < U; k++) {
        const uint32_t e = (uint32_t)lane_elem<U>(k);
        if (e < total) store_stream<WIDTH>(dst + e, v[k]);
    }
}

// Bytes s .. s + 15 (1 <= s <= 15) of the 32 bytes of a followed by b.
__device__ __forceinline__ u32x4 join16(u32x4 a, u32x4 b, uint32_t s) {
    const uint64_t a0 = ((uint64_t)a.y << 32) | a.x, a1 = ((uint64_t)a.w << 32) | a.z;
    const uint64_t b0 = ((uint64_t)b.y << 32) | b.x, b1 = ((uint64_t)b.w << 32) | b.z;
    const bool high = s >= 8;
    const uint64_t x = high ? a1 : a0, y = high ? b0 : a1, z = high ? b1 : b0;
    const uint32_t bits = (s & 7) * 8;
    const uint64_t lo = bits ? (x >> bits) | (y << (64 - bits)) : x;
    const uint64_t hi = bits ? (y >> bits) | (z << (64 - bits)) : y;
    u32x4 r;
    r.x = (uint32_t)lo;
    r.y = (uint32_t)(lo >> 32);
    r.z = (uint32_t)hi;
    r.w = (uint32_t)(hi >> 32);
    return r;
}

// Piece q of a column whose windows are not whole 16-byte elements: batch
// bytes [q*P, q*P + m), P = kThreads * U * 16.  A window holds at least 16
// bytes and a piece touches at most kThreads windows (the host's rule), so an
// element lies in one window, or covers the last bytes of one and the first of
// the next: then its two sources are the last 16 bytes of the one and the
// first 16 of the other, both inside their windows, and the element is 16
// consecutive bytes of the two together.  All first sources are loaded
// together; the second ones, on few lanes unless windows are short, follow.
template <int U, bool DRAWS>
__device__ void copy_straddle(const CollectArgs& a, const DrawArgs& g, const ColTask& c, int64_t q, Staged& st) {
    constexpr int64_t P = (int64_t)kThreads * U * 16;
    const int64_t o0 = q * P;
    const int64_t w0 = quotient(o0, c.W, c.recip);
    const int64_t total = (int64_t)a.B * c.W;
    const int32_t m = (int32_t)((total - o0) < P ? (total - o0) : P);
    const int64_t r0 = o0 - w0 * c.W;
    // Windows touched; with W >= P the piece may reach into a second one only.
    const int nw = c.magic ? (int)(((uint32_t)r0 + (uint32_t)m + (uint32_t)c.W - 1) / (uint32_t)c.W)
                           : (r0 + m > c.W ? 2 : 1);
    // Every touched window but the first starts inside the piece, and the first
    // does when the piece begins with it: those write their draws.
    const bool valid = !(stage_windows<DRAWS>(a, g, c, w0, nw, r0 == 0 ? 0 : 1, st) & kStagedZeros);
    const int32_t n16 = m / 16;  // whole elements; the batch's last bytes may be fewer
    u32x4* dst = reinterpret_cast<u32x4*>(c.out + o0);
    if (n16 > 0) {
        u32x4 v[U];
        int64_t at[U];               // offset of the first source, negative for zeros
        uint32_t win[U], cut[U];     // window; bytes of the first source that are skipped (0: no straddle)
#pragma unroll
        for (int k = 0; k < U; k++) {
            int32_t e = (int32_t)lane_elem<U>(k);
            e = e < n16 ? e : n16 - 1;
            const int64_t t = r0 + (int64_t)e * 16;
            win[k] = c.magic ? __umulhi((uint32_t)t, c.magic) : (t >= c.W ? 1u : 0u);
            const int64_t r = t - (int64_t)win[k] * c.W;
            const int64_t last = c.W - 16;
            cut[k] = r > last ? (uint32_t)(r - last) : 0u;
            const int64_t so = st.off[win[k]];
            at[k] = so < 0 ? so : so + (r > last ? last : r);
        }
        if (valid) {  // the loads go out unconditionally, all in flight
#pragma unroll
            for (int k = 0; k < U; k++) v[k] = load_stream<16>(c.src + at[k]);
        } else {
#pragma unroll
            for (int k = 0; k < U; k++) {
                v[k] = zero_elem<16>();
                if (at[k] >= 0) v[k] = load_stream<16>(c.src + at[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < U; k++) {
            if (cut[k]) {
                const int64_t so = st.off[win[k] + 1];
                v[k] = join16(v[k], so >= 0 ? load_stream<16>(c.src + so) : zero_elem<16>(), cut[k]);
            }
        }
#pragma unroll
        for (int k = 0; k < U; k++) {
            const int32_t e = (int32_t)lane_elem<U>(k);
            if (e < n16) store_stream<16>(dst + e, v[k]);
        }
    }
    const int32_t t = n16 * 16 + (int32_t)threadIdx.x;
    if (t < m) {  // fewer than 16 bytes, in the batch's last window
        const int64_t p = r0 + t;
        const uint32_t w = c.magic ? __umulhi((uint32_t)p, c.magic) : (p >= c.W ? 1u : 0u);
        const int64_t so = st.off[w];
        c.out[o0 + t] = so >= 0 ? c.src[so + (p - (int64_t)w * c.W)] : (uint8_t)0;
    }
}

// ANY: columns of every layout and width; otherwise only 16-byte elements in
// kWide and kNarrow columns.  DRAWS: the pieces compute their windows.
template <int U, bool DRAWS, bool ANY>
__global__ __launch_bounds__(kThreads) void collect_kernel(CollectArgs a, DrawArgs g) {
    __shared__ Staged st;
    const int32_t task = (int32_t)blockIdx.x;
    int j = 0, first = a.task0[0];
#pragma unroll
    for (int k0 = 0; k0 < kMaxLaunchCols; k0 += 4) {
#pragma unroll
        for (int k = k0 + 1; k <= k0 + 3; k++) {
            const bool past = a.task0[k] <= task;
            j = past ? k : j;
            first = past ? a.task0[k] : first;
        }
        if (k0 + 4 == kMaxLaunchCols || a.task0[k0 + 4 < kMaxLaunchCols ? k0 + 4 : 0] > task) break;
        j = k0 + 4;
        first = a.task0[k0 + 4 < kMaxLaunchCols ? k0 + 4 : 0];
    }
    // The whole line and the shared arguments at once; left to the compiler,
    // each field's load stands where the field is first used.
    const ColTask c = a.col[j];
    asm volatile("" ::"s"(c.src), "s"(c.out), "s"(c.W), "s"(c.n), "s"(c.recip), "s"(c.E), "s"(c.epw), "s"(c.magic),
                 "s"(a.idx), "s"(a.start), "s"(a.N), "s"(a.B), "s"(a.T), "s"(a.L));
    const int64_t q = task - first;
    if (ANY && c.layout == kStraddle) {
        copy_straddle<U, DRAWS>(a, g, c, q, st);
    } else if (c.layout == kWide) {
        if (!ANY || c.width == 16) copy_wide<16, U, DRAWS>(a, g, c, q);
        else if (c.width == 4) copy_wide<4, U, DRAWS>(a, g, c, q);
        else copy_wide<1, U, DRAWS>(a, g, c, q);
    } else {
        if (!ANY || c.width == 16) copy_narrow<16, U, DRAWS>(a, g, c, q, st);
        else if (c.width == 4) copy_narrow<4, U, DRAWS>(a, g, c, q, st);
        else copy_narrow<1, U, DRAWS>(a, g, c, q, st);
    }
}

typedef void (*CollectKernel)(CollectArgs, DrawArgs);

template <int U>
CollectKernel collect_variant(bool draws, bool any) {
    if (draws) return any ? collect_kernel<U, true, true> : collect_kernel<U, true, false>;
    return any ? collect_kernel<U, false, true> : collect_kernel<U, false, false>;
}

// How column c's batch of B windows of L steps is cut into pieces; returns their
// number.
int64_t plan_column(const Table& t, int32_t c, void* out, int32_t B, int32_t L, int unroll, ColTask& ct) {
    ct.src = t.col_dev[c];
    ct.out = static_cast<uint8_t*>(out);
    ct.E = (int32_t)t.elem_bytes[c];  // at most 2^30
    ct.W = (int64_t)L * ct.E;
    const uintptr_t oa = reinterpret_cast<uintptr_t>(ct.out);
    const int64_t elems = (int64_t)kThreads * unroll;  // per piece
    // A straddling piece stages its windows' offsets, one per thread.
    const bool straddle = oa % 16 == 0 && ct.W % 16 != 0 && ct.W >= 16 && ct.W * (kThreads - 2) >= elems * 16;
    if (straddle || (oa % 16 == 0 && ct.W % 16 == 0)) ct.width = 16;
    else if (oa % 4 == 0 && ct.W % 4 == 0) ct.width = 4;
    else ct.width = 1;
    const int64_t piece = elems * ct.width;
    ct.n = ct.W / ct.width;
    ct.layout = straddle ? kStraddle : ct.W >= piece ? kWide : kNarrow;
    if (ct.layout == kStraddle) {
        ct.recip = ~0ull / (uint64_t)ct.W;
        ct.magic = ct.W < piece ? (uint32_t)(((1ull << 32) + ct.W - 1) / ct.W) : 0u;
        return ((int64_t)B * ct.W + piece - 1) / piece;
    }
    if (ct.layout == kWide) {
        ct.recip = ~0ull / (uint64_t)ct.n;
        return ((int64_t)B * ct.n + elems - 1) / elems;
    }
    int64_t wpp = piece / ct.W;
    if (wpp > kThreads) wpp = kThreads;
    ct.wpp = (uint16_t)wpp;
    ct.epw = (uint32_t)(ct.W / ct.width);
    ct.magic = ct.epw > 1 ? (uint32_t)(((1ull << 32) + ct.epw - 1) / ct.epw) : 0u;
    return (B + wpp - 1) / wpp;
}

// The collect launches over ncols requested columns (kMaxLaunchCols per
// launch).  With `draws`, the windows are those FIFO, LIFO or uniform draws,
// computed in the kernel, and the first launch's first column writes them to
// idx_out, start_out and w_out; otherwise they come from idx and start.
int launch_collect(Table* t, const int64_t* d_idx, const int32_t* d_start, const SimpleDraws* draws,
                   int64_t* idx_out, int32_t* start_out, float* w_out, int32_t B, int32_t L,
                   const int32_t* col_ids, int32_t ncols, void* const* d_out, hipStream_t s, const char* who) {
    const bool pinned = t->residency == GEAR_HOST_PINNED;
    int64_t batch_bytes = 0;
    for (int j = 0; j < ncols; j++) batch_bytes += (int64_t)B * L * t->elem_bytes[col_ids ? col_ids[j] : j];
    const bool share = !pinned && batch_bytes >= kLongBatch && (t->options & GEAR_OPT_GATHER_SHARE_CU);
    const int unroll = pinned ? kUnrollHost : share ? kUnrollShare : kUnroll;

    // A batch that is refused launches nothing: with several groups of columns,
    // every group's pieces are counted before the first launch.
    for (int j0 = 0; j0 < ncols && ncols > kMaxLaunchCols; j0 += kMaxLaunchCols) {
        int64_t tasks = 0;
        for (int j = j0; j < ncols && j < j0 + kMaxLaunchCols; j++) {
            ColTask ct{};
            tasks += plan_column(*t, col_ids ? col_ids[j] : j, d_out[j], B, L, unroll, ct);
        }
        if (tasks > INT32_MAX) return fail(GEAR_E_INVAL, std::string(who) + ": batch too large for one call");
    }

    for (int j0 = 0; j0 < ncols; j0 += kMaxLaunchCols) {
        CollectArgs a{};
        a.idx = d_idx;
        a.start = d_start;
        DrawArgs g{};
        if (draws) {
            g.draws = *draws;
            g.idx_out = idx_out;
            g.start_out = start_out;
            g.w_out = w_out;
        }
        a.B = B;
        a.T = t->T;
        a.L = L;
        a.N = t->N;
        a.status = t->status;
        int64_t tasks = 0, wide_tasks = 0;
        int launch_cols = 0;
        bool any = false;  // a column needs more than 16-byte elements of whole windows
        for (int k = 0; k < kMaxLaunchCols; k++) a.task0[k] = INT32_MAX;
        // Tasks are numbered from the last requested column to the first:
        // the wide columns, listed first in the common layouts, then end
        // the launch with full pieces instead of small packed ones
        // (measured 1.6% faster on whole 68 KB trajectories).
        const int jend = ncols < j0 + kMaxLaunchCols ? ncols : j0 + kMaxLaunchCols;
        for (int j = jend - 1; j >= j0; j--) {
            if (tasks > INT32_MAX) break;  // refused below
            a.task0[launch_cols] = (int32_t)tasks;
            ColTask& ct = a.col[launch_cols++];
            const int64_t k = plan_column(*t, col_ids ? col_ids[j] : j, d_out[j], B, L, unroll, ct);
            ct.draws_out = draws != nullptr && j == 0;
            any = any || ct.layout == kStraddle || ct.width != 16;
            tasks += k;
            wide_tasks += ct.layout == kWide ? k : 0;
        }
        if (tasks > INT32_MAX) return fail(GEAR_E_INVAL, std::string(who) + ": batch too large for one call");
        const unsigned lds = share ? kShareLds : !pinned && wide_tasks * 2 > tasks ? kWideLds : 0u;
        const CollectKernel kernel = unroll == kUnroll ? collect_variant<kUnroll>(draws != nullptr, any)
                                                       : collect_variant<kUnrollHost>(draws != nullptr, any);
        // One launch, unless the batch has more pieces than a launch may have
        // workgroups (128 GiB in elements of 16 bytes).
        const int64_t most = t->max_items / kThreads;
        for (int64_t done = 0; done < tasks; done += most) {
            const int64_t grid = tasks - done < most ? tasks - done : most;
            hipLaunchKernelGGL(kernel, dim3((unsigned)grid), dim3(kThreads), lds, s, a, g);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return hip_fail(e, (std::string(who) + ": launch").c_str());
            for (int k = 0; k < launch_cols; k++) a.task0[k] -= (int32_t)grid;
        }
    }
    return GEAR_OK;
}

// Argument checks shared by gear_collect and gear_select_collect.
int check_columns(const Table* t, const int32_t* col_ids, int32_t ncols, void* const* d_out, const char* who) {
    if (d_out == nullptr) return fail(GEAR_E_INVAL, std::string(who) + ": NULL pointer argument");
    if (col_ids == nullptr && ncols != t->ncols)
        return fail(GEAR_E_INVAL, std::string(who) + ": ncols must equal the table's column count when col_ids is NULL");
    if (ncols < 1 || ncols > GEAR_MAX_COLUMNS) return fail(GEAR_E_INVAL, std::string(who) + ": ncols out of range");
    for (int j = 0; j < ncols; j++) {
        const int c = col_ids ? col_ids[j] : j;
        if (c < 0 || c >= t->ncols) return fail(GEAR_E_INVAL, std::string(who) + ": no such column");
        if (d_out[j] == nullptr) return fail(GEAR_E_INVAL, std::string(who) + ": output pointer is NULL");
    }
    return GEAR_OK;
}

}  // namespace
}  // namespace gear

using gear::fail;
using gear::hip_fail;

extern "C" int gear_collect(gear_table* h, const int64_t* d_idx, const int32_t* d_start, int32_t B, int32_t L,
                            const int32_t* col_ids, int32_t ncols, void* const* d_out, void* stream) {
    if (h == nullptr) return fail(GEAR_E_INVAL, "gear_collect: table is NULL");
    gear::Table* t = reinterpret_cast<gear::Table*>(h);
    if (B < 1 || B > GEAR_MAX_BATCH) return fail(GEAR_E_INVAL, "gear_collect: B out of range");
    if (L < 1 || L > t->T) return fail(GEAR_E_INVAL, "gear_collect: L must lie in [1, T]");
    if (d_idx == nullptr || d_start == nullptr) return fail(GEAR_E_INVAL, "gear_collect: NULL pointer argument");
    int rc = gear::check_columns(t, col_ids, ncols, d_out, "gear_collect");
    if (rc != GEAR_OK) return rc;
    gear::DeviceGuard guard(t->device);
    if (guard.error() != hipSuccess) return hip_fail(guard.error(), "gear_collect: hipSetDevice");
    return gear::launch_collect(t, d_idx, d_start, nullptr, nullptr, nullptr, nullptr, B, L, col_ids, ncols, d_out,
                                static_cast<hipStream_t>(stream), "gear_collect");
}

extern "C" int gear_select_collect(gear_table* h, int32_t strategy, int32_t B, int32_t L, uint64_t seed,
                                   int64_t* d_idx, int32_t* d_start, float* d_weights, const int32_t* col_ids,
                                   int32_t ncols, void* const* d_out, void* stream) {
    if (h == nullptr) return fail(GEAR_E_INVAL, "gear_select_collect: table is NULL");
    gear::Table* t = reinterpret_cast<gear::Table*>(h);
    if (strategy != GEAR_FIFO && strategy != GEAR_LIFO && strategy != GEAR_UNIFORM)
        return fail(GEAR_E_INVAL, "gear_select_collect: strategy must be GEAR_FIFO, GEAR_LIFO or GEAR_UNIFORM");
    if (B < 1 || B > GEAR_MAX_BATCH) return fail(GEAR_E_INVAL, "gear_select_collect: B out of range");
    if (L < 1 || L > t->T) return fail(GEAR_E_INVAL, "gear_select_collect: L must lie in [1, T]");
    if (d_idx == nullptr || d_start == nullptr)
        return fail(GEAR_E_INVAL, "gear_select_collect: NULL pointer argument");
    int rc = gear::check_columns(t, col_ids, ncols, d_out, "gear_select_collect");
    if (rc != GEAR_OK) return rc;
    const int64_t live = gear::live_count(*t);
    if (live == 0) return fail(GEAR_E_EMPTY, "gear_select_collect: nothing inserted");
    if ((strategy == GEAR_FIFO || strategy == GEAR_LIFO) && (int64_t)B > live)
        return fail(GEAR_E_INSUFFICIENT, "gear_select_collect: FIFO/LIFO batch larger than the live count");
    gear::DeviceGuard guard(t->device);
    if (guard.error() != hipSuccess) return hip_fail(guard.error(), "gear_select_collect: hipSetDevice");
    const gear::SimpleDraws d = gear::simple_draws(*t, strategy, L, seed);
    return gear::launch_collect(t, nullptr, nullptr, &d, d_idx, d_start, d_weights, B, L, col_ids, ncols, d_out,
                                static_cast<hipStream_t>(stream), "gear_select_collect");
}
