// GREM over a stream of edge chunks, two partitions, for gfx950 (Armada paper, Sec. 4.1, Alg. 1
// "GREM Bipartite Graph Partitioning" with the helpers of Alg. 2, in the stream model the paper
// states them in: an edge list in random order, a chunk is c_size consecutive edges, the chunk's
// nodes are the distinct endpoints of its edges and each is (re)evaluated from the chunk's edges).
//
// Chunk-synchronous form: every decision of a chunk reads labels and sizes as of the chunk's start;
// moves are admitted in ascending node id while the target has room; rejected refined nodes stay;
// rejected new nodes are placed one by one, ascending id, in the currently smaller partition.
//
// One run works on several groups of nodes side by side, each with its own edges, chunk length, capacity
// and sizes: a plain call is a run of one group, a level of the recursive bisection one of all its groups
// (chunk i of every group in the same launches).  In the run's state a group's nodes are consecutive and
// padded to whole blocks, a block of nodes being what one workgroup of the per-node kernels owns.
//
// Data layout (device memory, by node of the state)
//   Lw    uint64 per 32 nodes: low half = nodes that have a label, high half = those of partition 1 (no label: 0).  A quarter
//                   of a byte per node is what the random look-ups go to; the per-node kernels take 64 nodes' labels in
//                   one load and relabel them with a few bit operations
//   est   double[2] Alg. 1's nbr_counts; on large graphs 8 bytes per node hold them while they fit (es_blend_packed)
//   mv0, mv1, nw    bitmaps: nodes asking to move to partition 0 / 1, and those of them that have no label
//                   yet.  Bitmaps are ordered sets: bit order is id order, so ranks by id are prefix
//                   pop-counts.
//   mark            bitmap: v is an endpoint of a chunk edge whose other end has no label
// The chunk's fresh counts (Alg. 2 cnt_nbrs) come in one of three ways, the same integers any way:
//   in memory (small graphs)  hc, uint64 per node: low half = neighbours in partition 0, high half = in
//                   partition 1; k_es_count adds one 64-bit atomic per edge end, k_es_score reads and clears.
//   binned (large graphs)     k_es_bin (k_es_bin4, k_es_bin8: of four and eight edges per thread instead of two) looks the other end's label
//                   up for every edge end and sorts the (node, label) pairs by ranges of nodes; k_es_score_bins counts a block's pairs in LDS
//   asked (larger ones)       where the labels outgrow the L2s, k_es_ask and k_es_answer do k_es_bin's work with labels in LDS
// Per chunk: count or bin -> score (blend, assign, mover ballots) -> k_es_admit (ranks = movers of the earlier
// blocks + pop-count prefix; admitted moves relabel; closed-form target of the j-th rejected node; sizes).  The
// sizes live in two copies that take turns from chunk to chunk.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "grem.h"
#include "grem_es_estimate.hip.h"

namespace {

typedef unsigned long long u64;

constexpr int kBlock = 1024;                 // per-node kernels: 16 waves
constexpr int kWaves = kBlock / 64;
constexpr int kMaxWaveWords = 64;            // most bitmap words a wave of the per-node kernels owns
constexpr int kMaxAdmitWords = 128;          // ... of k_es_admit
constexpr uint32_t kNone = 2u;               // label of a node that has none
constexpr int kCountBlock = 256;
constexpr int kTurn = 4;                     // bitmap words a wave has in flight

// One group of a run.
struct EsGroup {
    int64_t e_lo, m, c_size;                 // its edges in the list, edges per chunk
    long long P;                             // capacity of a partition
    int64_t v_lo;                            // its first node in the caller's arrays
    uint32_t node0, nv;                      // its first node in the state, its nodes
    uint32_t blk0, nblk;                     // its blocks of nodes
    uint32_t tile0, id;                      // bisection: its first tile of edges, its number in the level
};

// What the kernels of a run share.
struct EsRun {
    const EsGroup* groups;
    const uint32_t* blk_group;               // group of a block
    u64* S;                                  // [2][groups][2]: sizes, two copies
    u64* Lw;
    double2* est;                            // the estimates, a node's at its own place, or those of `packed` that have outgrown it
    u64* packed;                             // binned, where there is memory for it: the estimates in 8 bytes each
    uint32_t* wide;                          // ... and per block how many have outgrown them
    u64 *mark, *mv0, *mv1, *nw;
    uint4* bs;                               // per block: movers to 0, to 1, those of either without a label
    uint32_t* flags;                         // [0] an endpoint out of range, [1] a bad seed
    uint32_t ngroups;
    int wpw;                                 // bitmap words per wave: a block is kBlock * wpw nodes
    int awpw;                                // the same in k_es_admit, a multiple of wpw
    EsGroup only;                            // a run of one group: that group (groups and blk_group are not looked at: two loads
                                             // less, one after the other, at the head of every launch)
};
__device__ __forceinline__ uint32_t es_group_of(const EsRun& st, uint32_t block) { return st.ngroups == 1u ? 0u : st.blk_group[block]; }
__device__ __forceinline__ EsGroup es_group(const EsRun& st, uint32_t gi)
{
    if (st.ngroups == 1u) return st.only;
    return st.groups[gi];
}

// label of node v: 0, 1 or kNone
__device__ __forceinline__ uint32_t es_label(u64 word, uint32_t v)
{
    const u64 x = word >> (v & 31u);
    return (x & 1ull) ? (uint32_t)(x >> 32) & 1u : kNone;
}

// the labels of 64 nodes (bitmap word w): who has one, who is in partition 1
struct EsLabels { u64 has, one; };
__device__ __forceinline__ EsLabels es_load_labels(const EsRun& st, size_t w)
{
    const ulonglong2 x = reinterpret_cast<const ulonglong2*>(st.Lw)[w];
    return {(x.x & 0xFFFFFFFFull) | x.y << 32, x.x >> 32 | (x.y & ~0xFFFFFFFFull)};
}
__device__ __forceinline__ void es_store_labels(const EsRun& st, size_t w, EsLabels l)
{
    reinterpret_cast<ulonglong2*>(st.Lw)[w] =
        make_ulonglong2((l.has & 0xFFFFFFFFull) | l.one << 32, l.has >> 32 | (l.one & ~0xFFFFFFFFull));
}

// first and last edge of the group's chunk (an empty range past its last chunk)
__device__ __forceinline__ void es_chunk(const EsGroup& g, int64_t chunk, int64_t& lo, int64_t& hi)
{
    const int64_t a = chunk * g.c_size < g.m ? chunk * g.c_size : g.m;
    const int64_t b = a + g.c_size < g.m ? a + g.c_size : g.m;
    lo = g.e_lo + a;
    hi = g.e_lo + b;
}

__global__ __launch_bounds__(256) void k_es_fill64(u64* p, size_t count, u64 value)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = value;
}

// several arrays at once: a run of 20,000 nodes spent some 4 us on each launch of its own
struct EsClears {
    static constexpr int kMost = 8;
    u64* p[kMost];
    size_t words[kMost];
    int n = 0;
    void add(void* at, size_t bytes) { p[n] = (u64*)at; words[n++] = bytes / 8; }
};
__global__ __launch_bounds__(256) void k_es_clear(EsClears c)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (int k = 0; k < c.n; ++k)
        for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < c.words[k]; i += stride) c.p[k][i] = 0ull;
}

__global__ __launch_bounds__(256) void k_es_blk_groups(const EsGroup* __restrict__ groups, uint32_t* blk_group)
{
    const EsGroup g = groups[blockIdx.x];
    for (uint32_t b = threadIdx.x; b < g.nblk; b += 256) blk_group[g.blk0 + b] = blockIdx.x;
}

// flags[0] = 1 if any endpoint lies outside [0, n)
__global__ __launch_bounds__(256) void k_es_check(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                  int64_t m, uint32_t n, uint32_t* flags)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += stride)
        bad |= ((uint32_t)src[e] >= n) | ((uint32_t)dst[e] >= n);
    if (bad) flags[0] = 1u;
}

// c_nodes of the first chunk as a bitmap (Alg. 1: unique_nodes_in_edges).  Runs before the range check has
// been read back: ends out of range are passed over.  Most ends find their bit set already: a plain look
// spares them the atomic (a stale word only costs one).
__device__ __forceinline__ void es_mark_ends(const EsRun& st, const EsGroup& g, uint32_t s, uint32_t d)
{
    const uint32_t end[2] = {s, d};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        if (end[i] >= g.nv) continue;
        const uint32_t v = g.node0 + end[i];
        const u64 bit = 1ull << (v & 63u);
        if (!(__hip_atomic_load(&st.mark[v >> 6], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) & bit))
            atomicOr(&st.mark[v >> 6], bit);
    }
}
__global__ __launch_bounds__(kCountBlock) void k_es_mark(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                         EsRun st)
{
    const EsGroup g = es_group(st, blockIdx.y);
    int64_t lo, hi;
    es_chunk(g, 0, lo, hi);
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < hi; e += stride) es_mark_ends(st, g, (uint32_t)src[e], (uint32_t)dst[e]);
}

// both for a run of one group: all of its edges checked, the first chunk's ends marked
__global__ __launch_bounds__(kCountBlock) void k_es_check_mark(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, EsRun st)
{
    const EsGroup g = st.only;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    bool bad = false;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < g.m; e += stride) {
        const uint32_t s = (uint32_t)src[e], d = (uint32_t)dst[e];
        bad |= (s >= g.nv) | (d >= g.nv);
        if (e < g.c_size) es_mark_ends(st, g, s, d);
    }
    if (bad) st.flags[0] = 1u;
}

// The two-partition choice of Alg. 2, on sizes from which the node itself has been taken out: the
// side that holds strictly more of the node's neighbours wins when it still has room; with no such
// side (equal estimates, or the richer side full) the smaller partition takes the node, 0 on a tie.
// lean: +1 where side 1 holds more, -1 where side 0 does, 0: neither
__device__ __forceinline__ int es_assign(int lean, long long s0, long long s1, long long P)
{
    if (lean != 0) {
        const int p = lean > 0;
        if ((p ? s1 : s0) < P) return p;
    }
    return s1 < s0;
}

// Alg. 1's blend of a packed estimate with the fresh counts (es_blend), stored; the comparison of the two sides.
__device__ __forceinline__ int es_blend_packed(const EsRun& st, size_t node, uint2 word, double2 doubles, bool blend, uint32_t h0, uint32_t h1,
                                               size_t first_wide, uint32_t* wide)
{
    uint2* const packed = reinterpret_cast<uint2*>(st.packed) + node;
    const EsBlended now = es_blend(word, doubles, blend, h0, h1);
    if (now.fits) {
        *packed = now.word;
    } else if (es_is_wide(word)) {
        st.est[es_wide_place(word)] = now.sums;
    } else {
        const size_t at = first_wide + atomicAdd(wide, 1u);
        st.est[at] = now.sums;
        *packed = es_wide_word(at);
    }
    return now.lean;
}

// value of x in lane i, i uniform over the wave
__device__ __forceinline__ u64 es_bcast(u64 x, int i)
{
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)x, i);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)(x >> 32), i);
    return ((u64)hi << 32) | lo;
}

// x + the value of x that the cross-lane move CTRL brings (0 where it brings none, or where ROWS leaves the row out)
template <int CTRL, int ROWS> __device__ __forceinline__ uint32_t es_dpp_add(uint32_t x)
{
    return x + (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, ROWS, 0xF, false);
}
// inclusive prefix sum over the lanes of each row of 16 (row_shr by 1, 2, 4, 8), and over all 64 (row_bcast 15 and 31)
__device__ __forceinline__ uint32_t es_row_inclusive(uint32_t x)
{
    x = es_dpp_add<0x111, 0xF>(x);
    x = es_dpp_add<0x112, 0xF>(x);
    x = es_dpp_add<0x114, 0xF>(x);
    return es_dpp_add<0x118, 0xF>(x);
}
__device__ __forceinline__ uint32_t es_wave_inclusive(uint32_t x)
{
    return es_dpp_add<0x143, 0xC>(es_dpp_add<0x142, 0xA>(es_row_inclusive(x)));
}
__device__ __forceinline__ uint32_t es_lane(uint32_t x, int i) { return (uint32_t)__builtin_amdgcn_readlane((int)x, i); }
__device__ __forceinline__ uint32_t es_wave_sum(uint32_t x) { return es_lane(es_wave_inclusive(x), 63); }
__device__ __forceinline__ int es_wave() { return __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// sums over the workgroup (kBlock threads, all of them call it); every sum is below 2^32
template <int N> __device__ __forceinline__ void es_block_sums(uint32_t (&x)[N])
{
    __shared__ uint32_t part[N][kWaves];
    static_assert(kWaves == 16, "a row of lanes holds the waves' sums");
    const int lane = threadIdx.x & 63, wave = es_wave();
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const uint32_t sum = es_wave_sum(x[i]);
        if (lane == 0) part[i][wave] = sum;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = es_lane(es_row_inclusive(part[i][lane & 15]), 15);
}

// exclusive prefix of x over the workgroup's threads and the sum over all of them; wsum: kWaves words of LDS
__device__ __forceinline__ uint32_t es_block_exclusive(uint32_t x, uint32_t* wsum, uint32_t* total = nullptr)
{
    const int lane = threadIdx.x & 63, wave = es_wave();
    const uint32_t incl = es_wave_inclusive(x);
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    const uint32_t waves = es_row_inclusive(wsum[lane & 15]);
    if (total) *total = es_lane(waves, 15);
    return incl - x + (wave ? es_lane(waves, wave - 1) : 0u);
}

// Alg. 1, first chunk: the chunk's nodes take seed_algo's labels; sizes are counted.
// flags[1] = 1 if a node of the chunk has a seed label other than 0 or 1.
__global__ __launch_bounds__(kBlock) void k_es_seed(EsRun st, const int32_t* __restrict__ seed)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t gi = es_group_of(st, blockIdx.x);
    const EsGroup g = es_group(st, gi);
    const uint32_t word0 = ((uint32_t)blockIdx.x * kWaves + wave) * st.wpw;
    const u64 mine = lane < st.wpw ? st.mark[word0 + lane] : 0ull;
    EsLabels labels{0ull, 0ull};
    for (int i0 = 0; i0 < st.wpw; i0 += kTurn) {
        int s[kTurn];
        bool on[kTurn];
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            on[u] = i0 + u < st.wpw && ((es_bcast(mine, (i0 + u) & 63) >> lane) & 1ull);
            s[u] = on[u] ? seed[g.v_lo + ((word0 + i0 + u) * 64u + lane - g.node0)] : -1;
        }
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            if (on[u] && s[u] != 0 && s[u] != 1) st.flags[1] = 1u;
            const u64 zeros = __ballot(on[u] && s[u] == 0), ones = __ballot(on[u] && s[u] == 1);
            if (lane == i0 + u) labels = {zeros | ones, ones};
        }
    }
    if (mine) es_store_labels(st, word0 + lane, labels);           // (no label before)
    uint32_t sizes[2] = {(uint32_t)__popcll(labels.has & ~labels.one), (uint32_t)__popcll(labels.one)};
    es_block_sums(sizes);
    if (threadIdx.x < 2 && sizes[threadIdx.x]) atomicAdd(&st.S[2 * gi + threadIdx.x], (u64)sizes[threadIdx.x]);
}

// flags[1] = 1 if the seeds fill a partition beyond its capacity
__global__ __launch_bounds__(256) void k_es_seed_sizes(EsRun st)
{
    const uint32_t gi = blockIdx.x * blockDim.x + threadIdx.x;
    if (gi >= st.ngroups) return;
    const long long P = es_group(st, gi).P;
    if ((long long)st.S[2 * gi] > P || (long long)st.S[2 * gi + 1] > P) st.flags[1] = 1u;
}

// cnt_nbrs (Alg. 2) for every node of the chunk at once, in memory: each edge adds one to the count its two
// ends keep for the partition of the other end (a loop counts once, for the node itself).  An
// unassigned other end adds nothing; the node's bit in `mark` is set instead, so that a node of the
// chunk is known by a non-zero count or its bit: one atomic per edge end either way.
// Random look-ups and atomics, 39 G/s of them together once labels and hc outgrow the L2 (then the ends are binned).
// An edge per thread: with four in flight each, nothing was faster at chunks of 2,000 to 100M edges, and those of 6,000 took
// 7.1 us for 3.8.
__global__ __launch_bounds__(kCountBlock) void k_es_count(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                          EsRun st, int64_t chunk, u64* hc)
{
    const EsGroup g = es_group(st, blockIdx.y);
    int64_t lo, hi;
    es_chunk(g, chunk, lo, hi);
    const u64* __restrict__ Lw = st.Lw + (g.node0 >> 5);           // (a group starts at a whole block)
    hc += g.node0;
    u64* mark = st.mark + (g.node0 >> 6);
    const int64_t threads = (int64_t)gridDim.x * blockDim.x;
    for (int64_t e = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < hi; e += threads) {
        const uint32_t s = (uint32_t)src[e], d = (uint32_t)dst[e];
        const u64 ws = Lw[s >> 5], wd = Lw[d >> 5];
        const uint32_t ls = es_label(ws, s), ld = es_label(wd, d);
        if (ld != kNone) atomicAdd(&hc[s], ld ? (1ull << 32) : 1ull);
        else atomicOr(&mark[s >> 6], 1ull << (s & 63u));
        if (d == s) continue;
        if (ls != kNone) atomicAdd(&hc[d], ls ? (1ull << 32) : 1ull);
        else atomicOr(&mark[d >> 6], 1ull << (d & 63u));
    }
}

// ---- the chunk's edge ends binned by ranges of nodes -------------------------------------------------------
//
// A bin is 2^cb nodes of the state, at most kBins of them (nb: how many, a multiple of kBlock).  All chunks' bin sizes are counted
// beforehand (k_es_hist, with the range check of the endpoints).  Where a chunk has many tiles, a bin's room is split among eight
// classes of tiles (neighbours; ends[chunk][class][bin]): workgroups go to the XCDs in turn, so that what the tiles of a class
// write one after the other meets in one L2, and a run need not fill a line.  (Nothing but the time depends on where they go.)
// ends[] holds first the sizes, then the starts (k_es_hist_scan), which k_es_bin moves on to the ends.
constexpr int kBins = 4096;
constexpr int kBinTile = 8192;               // most edges per workgroup: 64 KB of pairs, two workgroups per CU
constexpr int kBinPer = kBinTile / kBlock;

struct EsBins {
    uint32_t* ends;
    uint32_t nb;
    int cb, classes;
    // the pairs of a bin once they are all there
    __device__ __forceinline__ void range(int64_t chunk, uint32_t bin, uint32_t& p0, uint32_t& p1) const
    {
        const uint32_t* row = ends + ((size_t)chunk * classes + (classes - 1)) * nb;
        p0 = bin ? row[bin - 1u] : 0u;
        p1 = row[bin];
    }
};

// (gridDim.x is a multiple of the classes; tile: edges of a workgroup of k_es_bin or k_es_ask; hist: a word per bin or, where
// labels are asked for, per bin and class.  kBinTile is a multiple of the tile, the tile of kBlock.)
__global__ __launch_bounds__(kBlock) void k_es_hist(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                    EsRun st, EsBins bins, EsBins ranges, int tile)
{
    extern __shared__ uint32_t hist[];
    const EsGroup g = es_group(st, blockIdx.y);
    int64_t lo, hi;
    es_chunk(g, blockIdx.z, lo, hi);
    if (lo + (int64_t)blockIdx.x * tile >= hi) return;
    const bool asked = ranges.ends != nullptr;
    const uint32_t per = asked ? (uint32_t)bins.classes : 1u, cells = bins.nb * per;
    for (uint32_t i = threadIdx.x; i < cells; i += kBlock) hist[i] = 0u;
    __syncthreads();
    bool bad = false;
    // (as many of its tiles at a time as make kBinTile edges)
    const int64_t step = (int64_t)gridDim.x * tile;
    for (int64_t t = lo + (int64_t)blockIdx.x * tile; t < hi; t += kBinTile / tile * step) {
        uint32_t s[kBinPer], d[kBinPer];
#pragma unroll
        for (int u = 0; u < kBinPer; ++u) {
            const int64_t e = t + u * kBlock / tile * step + u * kBlock % tile + threadIdx.x;
            s[u] = e < hi ? (uint32_t)src[e] : g.nv;
            d[u] = e < hi ? (uint32_t)dst[e] : g.nv;
            bad |= e < hi && (s[u] >= g.nv || d[u] >= g.nv);
        }
#pragma unroll
        for (int u = 0; u < kBinPer; ++u) {
            if (s[u] >= g.nv || d[u] >= g.nv) continue;
            const uint32_t x = g.node0 + s[u], y = g.node0 + d[u];
            atomicAdd(&hist[asked ? (y >> ranges.cb) % per * bins.nb + (x >> bins.cb) : x >> bins.cb], 1u);
            if (x != y) atomicAdd(&hist[asked ? (x >> ranges.cb) % per * bins.nb + (y >> bins.cb) : y >> bins.cb], 1u);
        }
    }
    if (bad) st.flags[0] = 1u;
    __syncthreads();
    uint32_t* table = bins.ends + (size_t)blockIdx.z * bins.nb * bins.classes;
    const int own = (int)(blockIdx.x % (unsigned)bins.classes);
    for (uint32_t i = threadIdx.x; i < cells; i += kBlock)
        if (hist[i]) atomicAdd(&table[asked ? i : own * bins.nb + i], hist[i]);
    if (!asked) return;
    const uint32_t each = 1u << (ranges.cb - bins.cb);             // (a range asks as often as it is asked: every edge has two ends)
    for (uint32_t i = threadIdx.x; i < bins.nb / each; i += kBlock) {
        uint32_t c = 0;
        for (uint32_t j = 0; j < each * per; ++j) c += hist[j / each * bins.nb + i * each + j % each];
        if (c) atomicAdd(&ranges.ends[((size_t)blockIdx.z * ranges.classes + own) * ranges.nb + i], c);
    }
}

// The bins of more than `limit` pairs in a chunk, which no workgroup should count alone (k_es_crowd).
struct EsCrowd {
    uint16_t* place;                         // [chunk][bin]: 0, or 1 + the bin's place among the chunk's crowded ones
    uint32_t* bins;                          // [chunk]: how many there are
    u64* hc;                                 // [place][node of the bin]: counts as in EsMemory::hc, zero between chunks
    uint32_t* seen;                          // ... and a bit per node
    uint32_t limit;
};

// sizes -> starts (one workgroup per chunk, neighbouring bins a thread's)
__global__ __launch_bounds__(kBlock) void k_es_hist_scan(EsBins bins, EsCrowd crowd, uint32_t* totals)
{
    __shared__ uint32_t wsum[kWaves];
    const uint32_t own = bins.nb / kBlock, first = threadIdx.x * own;
    uint32_t* row = bins.ends + (size_t)blockIdx.x * bins.nb * bins.classes + first;
    uint32_t sum = 0, crowded = 0;
    for (uint32_t i = 0; i < own; ++i) {
        uint32_t c = 0;
        for (int k = 0; k < bins.classes; ++k) c += row[(size_t)k * bins.nb + i];
        sum += c;
        crowded += crowd.place && c > crowd.limit ? 1u : 0u;
    }
    uint32_t at = es_block_exclusive(sum, wsum);
    __syncthreads();
    uint32_t place = es_block_exclusive(crowded, wsum);
    for (uint32_t i = 0; i < own; ++i) {
        const uint32_t start = at;
        for (int k = 0; k < bins.classes; ++k) {
            const uint32_t c = row[(size_t)k * bins.nb + i];
            row[(size_t)k * bins.nb + i] = at;
            at += c;
        }
        if (totals && threadIdx.x == kBlock - 1 && i + 1u == own) totals[blockIdx.x] = at;
        if (!crowd.place) continue;
        const bool is = at - start > crowd.limit;
        crowd.place[(size_t)blockIdx.x * bins.nb + first + i] = is ? (uint16_t)(++place) : (uint16_t)0;
    }
    if (crowd.place && threadIdx.x == kBlock - 1) crowd.bins[blockIdx.x] = place;
}

// LDS of a tile's sorting: its items, per bin a word (how many, then where they go) and 16 bits (where they start)
inline size_t es_sort_lds(size_t items, size_t item_bytes, uint32_t nb) { return items * item_bytes + (size_t)nb * 6; }

// The bins' counts of a tile become starts in the sorted order and places in memory (minus the start): from hist[] to at[] (the
// same array) and start[]; returns the number of items.  cursors: the tile's class of the chunk's row.  (Bins kBlock apart are a
// thread's and neighbours in the order: a wave's atomics go to neighbouring words.)
__device__ __forceinline__ uint32_t es_sort_scan(uint32_t* at, uint16_t* start, const EsBins& bins, uint32_t* cursors, uint32_t* wsum)
{
    uint32_t c[kBins / kBlock], sum = 0, total;
#pragma unroll
    for (int i = 0; i < kBins / kBlock; ++i) {
        const uint32_t bin = i * kBlock + threadIdx.x;
        c[i] = bin < bins.nb ? at[bin] : 0u;
        sum += c[i];
    }
    uint32_t place[kBins / kBlock];
#pragma unroll
    for (int i = 0; i < kBins / kBlock; ++i)
        if (c[i]) place[i] = atomicAdd(&cursors[i * kBlock + threadIdx.x], c[i]);
    uint32_t excl = es_block_exclusive(sum, wsum, &total);
#pragma unroll
    for (int i = 0; i < kBins / kBlock; ++i) {
        const uint32_t bin = i * kBlock + threadIdx.x;
        if (bin >= bins.nb) continue;
        start[bin] = (uint16_t)excl;
        if (c[i]) at[bin] = place[i] - excl;
        excl += c[i];
    }
    __syncthreads();
    return total;
}

// cnt_nbrs, first half: for every edge end the label of the other end, the pairs sorted by bin.  A pair is the
// node's place in its bin and 0, 1 or 2 (no label) above it.  What bounds it is the look-up of the labels (59 G/s
// in the 28 MB of 111M nodes, which outgrow the L2); the pairs cost 4 bytes written and read where an atomic on the node's counts costs a
// read and a write of 64.  A tile's pairs are collected in LDS bin by bin and written in runs.
// 32M edge ends of 111M nodes: 1.61 ms with an atomic per end and a byte per label, 0.62 so sorted, 0.55 with two bits per label.
template <int PER>
__device__ __forceinline__ void es_bin_tile(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                            const EsRun& st, int64_t chunk, const EsBins& bins, uint32_t* __restrict__ pairs)
{
    extern __shared__ uint32_t items[];            // 2 * PER * kBlock, then at[], start[]
    __shared__ uint32_t wsum[kWaves];
    uint32_t* at = items + 2 * PER * kBlock;
    uint16_t* start = reinterpret_cast<uint16_t*>(at + bins.nb);
    const EsGroup g = es_group(st, blockIdx.y);
    int64_t lo, hi;
    es_chunk(g, chunk, lo, hi);
    lo += (int64_t)blockIdx.x * (PER * kBlock);
    if (lo >= hi) return;
    const int tid = threadIdx.x, cb = bins.cb;
    for (uint32_t i = tid; i < bins.nb; i += kBlock) at[i] = 0u;
    constexpr uint32_t kNothing = 0xFFFFFFFFu;
    uint32_t a[PER], b[PER];                       // node of the state | label code << 30 (fewer than 2^30 nodes)
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int64_t e = lo + u * kBlock + tid;
        a[u] = e < hi ? g.node0 + (uint32_t)src[e] : kNothing;
        b[u] = e < hi ? g.node0 + (uint32_t)dst[e] : kNothing;
    }
    u64 la[PER], lb[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        la[u] = a[u] != kNothing ? st.Lw[a[u] >> 5] : 0ull;
        lb[u] = a[u] != kNothing ? st.Lw[b[u] >> 5] : 0ull;
    }
    __syncthreads();
    uint32_t ra[PER], rb[PER];                     // rank among the tile's pairs of the same bin
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (a[u] == kNothing) continue;
        ra[u] = atomicAdd(&at[a[u] >> cb], 1u);
        const bool loop = a[u] == b[u];
        if (!loop) rb[u] = atomicAdd(&at[b[u] >> cb], 1u);
        const uint32_t of_a = es_label(la[u], a[u]), of_b = es_label(lb[u], b[u]);
        a[u] |= of_b << 30;
        b[u] = loop ? kNothing : b[u] | of_a << 30;
    }
    __syncthreads();
    const uint32_t total = es_sort_scan(at, start, bins, bins.ends + ((size_t)chunk * bins.classes + blockIdx.x % (unsigned)bins.classes) * bins.nb, wsum);
    auto place = [&](uint32_t x, uint32_t rank) {
        const uint32_t node = x & 0x3FFFFFFFu, bin = node >> cb;
        items[start[bin] + rank] = (node & ((1u << cb) - 1u)) | (x >> 30) << cb | bin << (cb + 2);      // (cb <= 18, 4096 bins)
    };
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        if (a[u] != kNothing) place(a[u], ra[u]);
        if (b[u] != kNothing) place(b[u], rb[u]);
    }
    __syncthreads();
    for (uint32_t i = tid; i < total; i += kBlock) {
        const uint32_t x = items[i];
        pairs[at[x >> (cb + 2)] + i] = x & ((1u << (cb + 2)) - 1u);
    }
}
__global__ __launch_bounds__(kBlock, 8) void k_es_bin4(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, EsRun st, int64_t chunk,
                                                      EsBins bins, uint32_t* __restrict__ pairs)
{
    es_bin_tile<4>(src, dst, st, chunk, bins, pairs);
}
__global__ __launch_bounds__(kBlock, 8) void k_es_bin(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, EsRun st, int64_t chunk,
                                                       EsBins bins, uint32_t* __restrict__ pairs)
{
    es_bin_tile<2>(src, dst, st, chunk, bins, pairs);
}
__global__ __launch_bounds__(kBlock, 8) void k_es_bin8(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, EsRun st, int64_t chunk,
                                                       EsBins bins, uint32_t* __restrict__ pairs)
{
    es_bin_tile<8>(src, dst, st, chunk, bins, pairs);
}

// ---- labels looked up in LDS --------------------------------------------------------------------------------
//
// Where the labels outgrow the L2s, look-ups run at 59 G/s (28 MB, 111M nodes) and each reads a line of 128 bytes.  Then an edge
// end asks for the other's label: k_es_ask sorts the asks (asked node, asking node) by ranges of asked nodes, and
// k_es_answer, which has a range's labels in LDS, sorts the answers into the bins.  32M ends of 111M nodes: 129 + 175 us instead of k_es_bin's 544, and the bins
// can be a block's nodes each (848 bins that four blocks read were as many as k_es_bin could serve: 700 us with 3392).

// The ranges' numbers class by class: 0, 8, 16, ..., 1, 9, ...  (as for the tiles of edges, a class's tiles go to one XCD)
__device__ __forceinline__ uint32_t es_ask_range(const EsBins& ranges, uint32_t i)
{
    const uint32_t each = ranges.nb / ranges.classes;
    return i % each * ranges.classes + i / each;
}
// A tile is kAskTile asks of a range or fewer; first[chunk][i]: tiles of the ranges before the i-th (one workgroup per chunk; the
// ranges' starts are known, the last one ends where the bins do).
constexpr int kAskTile = 16384;
__global__ __launch_bounds__(kBlock) void k_es_ask_tiles(EsBins ranges, const uint32_t* __restrict__ totals, uint32_t* first)
{
    __shared__ uint32_t wsum[kWaves];
    const uint32_t own = ranges.nb / kBlock, at = threadIdx.x * own;
    const uint32_t* row = ranges.ends + (size_t)blockIdx.x * ranges.nb * ranges.classes;
    auto tiles = [&](uint32_t i) {
        const uint32_t range = es_ask_range(ranges, i);
        const uint32_t end = range + 1u < ranges.nb ? row[range + 1u] : totals[blockIdx.x];
        return (end - row[range] + kAskTile - 1u) / kAskTile;
    };
    uint32_t sum = 0, total;
    for (uint32_t i = 0; i < own; ++i) sum += tiles(at + i);
    uint32_t before = es_block_exclusive(sum, wsum, &total);
    uint32_t* out = first + (size_t)blockIdx.x * (ranges.nb + 1u);
    for (uint32_t i = 0; i < own; ++i) {
        out[at + i] = before;
        before += tiles(at + i);
    }
    if (threadIdx.x == kBlock - 1) out[ranges.nb] = total;
}

// The ends' asks sorted by range: tile after tile of a class, the next one's edges on their way while a tile is written.
// (A word per range and tile is moved on in memory, neighbouring words by a wave: with the classes' words next to each other those
// atomics, a line each, were most of the time here and in k_es_answer, which took 451 us for 204 at 111M nodes.)
constexpr int kAskPer = 4, kAskEdges = kAskPer * kBlock;
__global__ __launch_bounds__(kBlock, 8) void k_es_ask(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                      EsRun st, int64_t chunk, EsBins ranges, uint2* __restrict__ asks)
{
    extern __shared__ uint32_t items[];            // 2 * kAskEdges of two words, then at[], start[]
    __shared__ uint32_t wsum[kWaves];
    uint2* sorted = reinterpret_cast<uint2*>(items);
    uint32_t* at = items + 4 * kAskEdges;
    uint16_t* start = reinterpret_cast<uint16_t*>(at + ranges.nb);
    const EsGroup g = es_group(st, blockIdx.y);
    int64_t lo, hi;
    es_chunk(g, chunk, lo, hi);
    lo += (int64_t)blockIdx.x * kAskEdges;
    const int tid = threadIdx.x, cb = ranges.cb;
    constexpr uint32_t kNothing = 0xFFFFFFFFu;
    uint32_t* const cursors = ranges.ends + ((size_t)chunk * ranges.classes + blockIdx.x % (unsigned)ranges.classes) * ranges.nb;
    uint32_t a[kAskPer], b[kAskPer];
    auto request = [&] {
#pragma unroll
        for (int u = 0; u < kAskPer; ++u) {
            const int64_t e = lo + u * kBlock + tid;
            a[u] = e < hi ? g.node0 + (uint32_t)src[e] : kNothing;
            b[u] = e < hi ? g.node0 + (uint32_t)dst[e] : kNothing;
        }
    };
    request();
    for (; lo < hi;) {
        for (uint32_t i = tid; i < ranges.nb; i += kBlock) at[i] = 0u;
        __syncthreads();
        uint32_t ra[kAskPer], rb[kAskPer];         // rank among the tile's asks of the same range
#pragma unroll
        for (int u = 0; u < kAskPer; ++u) {
            if (a[u] == kNothing) continue;
            ra[u] = atomicAdd(&at[a[u] >> cb], 1u);
            if (a[u] != b[u]) rb[u] = atomicAdd(&at[b[u] >> cb], 1u);
        }
        __syncthreads();
        const uint32_t total = es_sort_scan(at, start, ranges, cursors, wsum);
#pragma unroll
        for (int u = 0; u < kAskPer; ++u) {
            if (a[u] == kNothing) continue;
            sorted[start[a[u] >> cb] + ra[u]] = make_uint2(a[u], b[u]);
            if (a[u] != b[u]) sorted[start[b[u] >> cb] + rb[u]] = make_uint2(b[u], a[u]);
        }
        lo += (int64_t)gridDim.x * kAskEdges;
        request();
        __syncthreads();
        for (uint32_t i = tid; i < total; i += kBlock) {
            const uint2 x = sorted[i];
            asks[at[x.x >> cb] + i] = x;
        }
        __syncthreads();
    }
}

// A workgroup answers a tile of a range's asks after another, the next one's asks on their way while it writes.
__global__ __launch_bounds__(kBlock) void k_es_answer(EsRun st, int64_t chunk, EsBins ranges, const uint32_t* __restrict__ first,
                                                      const uint2* __restrict__ asks, EsBins bins, uint32_t nodes, uint32_t* __restrict__ pairs)
{
    extern __shared__ uint32_t items[];            // kAskTile, then the range's labels, at[], start[]
    __shared__ uint32_t wsum[kWaves];
    constexpr int PER = kAskTile / kBlock;
    const int tid = threadIdx.x, lane = tid & 63, cb = bins.cb;
    const uint32_t words = 1u << (ranges.cb - 5);
    u64* labels = reinterpret_cast<u64*>(items + kAskTile);
    uint32_t* at = items + kAskTile + 2 * words;
    uint16_t* start = reinterpret_cast<uint16_t*>(at + bins.nb);
    const uint32_t own = blockIdx.x % (unsigned)ranges.classes, each = ranges.nb / ranges.classes;
    const uint32_t* row = first + (size_t)chunk * (ranges.nb + 1) + own * each;
    const uint32_t tile1 = row[each], step = gridDim.x / (unsigned)ranges.classes;
    uint32_t* const cursors = bins.ends + ((size_t)chunk * bins.classes + own) * bins.nb;
    uint32_t tile = row[0] + blockIdx.x / (unsigned)ranges.classes, range = 0, p0 = 0, count = 0;
    uint2 ask[PER];
    auto request = [&] {                           // the tile's place, and its asks on their way
        if (tile >= tile1) return;
        uint32_t i = 0;                            // the last range that begins at the tile or before it
        for (uint32_t j = 0; j < each; j += 64) i += (uint32_t)__popcll(__ballot(j + lane < each && row[j + lane] <= tile));
        --i;
        const uint32_t t0 = row[i], tiles = row[i + 1u] - t0;
        range = es_ask_range(ranges, own * each + i);
        uint32_t p1;
        ranges.range(chunk, range, p0, p1);
        const uint32_t per = (p1 - p0 + tiles - 1u) / tiles;       // (kAskTile or fewer)
        p0 += (tile - t0) * per;
        count = p0 >= p1 ? 0u : p1 - p0 < per ? p1 - p0 : per;
#pragma unroll
        for (int u = 0; u < PER; ++u)
            if ((uint32_t)(u * kBlock + tid) < count) ask[u] = asks[p0 + u * kBlock + tid];
    };
    request();
    for (; tile < tile1;) {
        const ulonglong2* from = reinterpret_cast<const ulonglong2*>(st.Lw + (size_t)range * words);
        const uint32_t held = nodes / 32u - range * words < words ? nodes / 32u - range * words : words;       // (a range asked for begins inside)
        for (uint32_t i = tid; i < held / 2; i += kBlock) reinterpret_cast<ulonglong2*>(labels)[i] = from[i];
        for (uint32_t i = tid; i < bins.nb; i += kBlock) at[i] = 0u;
        __syncthreads();
        uint32_t rank[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if ((uint32_t)(u * kBlock + tid) >= count) continue;
            const uint32_t asked = ask[u].x & ((1u << ranges.cb) - 1u);
            ask[u].x = es_label(labels[asked >> 5], asked);
            rank[u] = atomicAdd(&at[ask[u].y >> cb], 1u);
        }
        __syncthreads();
        const uint32_t total = es_sort_scan(at, start, bins, cursors, wsum);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if ((uint32_t)(u * kBlock + tid) >= count) continue;
            const uint32_t node = ask[u].y, bin = node >> cb;
            items[start[bin] + rank[u]] = (node & ((1u << cb) - 1u)) | ask[u].x << cb | bin << (cb + 2);
        }
        tile += step;
        request();
        __syncthreads();
        for (uint32_t i = tid; i < total; i += kBlock) {
            const uint32_t x = items[i];
            pairs[at[x >> (cb + 2)] + i] = x & ((1u << (cb + 2)) - 1u);
        }
        __syncthreads();
    }
}

// ---- the per-node kernels: a wave owns wpw consecutive bitmap words (lane i holds word i), a block of 16 waves
// kBlock * wpw nodes ----------------------------------------------------------------------------------------------

// Alg. 1 for the nodes of up to kTurn bitmap words, one lane per node and word: blend the stored estimate with
// the fresh counts h when the node has a label, store the estimate, ask `assign` for a partition.  Sets the words of
// nodes that want to move (lane i0 + u keeps word i0 + u).  labels: lane i0 + u has those of word i0 + u.  on: the node belongs
// to the chunk.
__device__ __forceinline__ void es_score_words(const EsRun& st, uint32_t word0, int i0, const EsLabels& labels, const bool (&on)[kTurn],
                                               const uint32_t (&h0)[kTurn], const uint32_t (&h1)[kTurn], int first, int fixed,
                                               long long P, long long S0, long long S1, u64& out0, u64& out1)
{
    const int lane = threadIdx.x & 63;
    uint32_t old[kTurn];
    double2 prev[kTurn];
    bool blend[kTurn];
#pragma unroll
    for (int u = 0; u < kTurn; ++u) {
        const u64 has = es_bcast(labels.has, (i0 + u) & 63), one = es_bcast(labels.one, (i0 + u) & 63);
        old[u] = ((has >> lane) & 1ull) ? (uint32_t)(one >> lane) & 1u : kNone;
        blend[u] = on[u] && !first && old[u] != kNone && !fixed;
        if (blend[u]) prev[u] = st.est[(size_t)(word0 + i0 + u) * 64 + lane];
    }
#pragma unroll
    for (int u = 0; u < kTurn; ++u) {
        int want = -1;
        if (on[u] && (first || !(fixed && old[u] != kNone))) {
            double nbrs0 = (double)h0[u], nbrs1 = (double)h1[u];
            if (blend[u]) {
                nbrs0 = (prev[u].x + nbrs0) * 0.5;
                nbrs1 = (prev[u].y + nbrs1) * 0.5;
            }
            st.est[(size_t)(word0 + i0 + u) * 64 + lane] = make_double2(nbrs0, nbrs1);
            if (!first) {
                const int t = es_assign((nbrs1 > nbrs0) - (nbrs0 > nbrs1), S0 - (old[u] == 0u), S1 - (old[u] == 1u), P);
                if ((uint32_t)t != old[u]) want = t;
            }
        }
        const u64 m0 = __ballot(want == 0), m1 = __ballot(want == 1);
        if (lane == i0 + u) { out0 = m0; out1 = m1; }
    }
}

// a lane's word of movers: stored, and their numbers added to the lane's (to 0, to 1, those of either without a label)
__device__ __forceinline__ void es_store_words(const EsRun& st, uint32_t word, u64 out0, u64 out1, const EsLabels& labels, uint32_t (&m)[4])
{
    const u64 fresh = (out0 | out1) & ~labels.has;
    st.mv0[word] = out0;
    st.mv1[word] = out1;
    st.nw[word] = fresh;
    m[0] += (uint32_t)__popcll(out0);
    m[1] += (uint32_t)__popcll(out1);
    m[2] += (uint32_t)__popcll(out0 & fresh);
    m[3] += (uint32_t)__popcll(out1 & fresh);
}
__device__ __forceinline__ void es_store_movers(const EsRun& st, uint32_t (&m)[4], uint32_t block)
{
    es_block_sums(m);
    if (threadIdx.x == 0) st.bs[block] = make_uint4(m[0], m[1], m[2], m[3]);
}

// The pairs of the chunk's crowded bins, counted before the scoring by all workgroups: a piece of a bin's pairs and one of
// its blocks at a time, in LDS, added to the counts in memory that k_es_score_bins then reads instead of the pairs.  Ids in
// order of degree put a quarter of all ends in one bin, whose four blocks each walked 8M pairs twice: a chunk of 16M
// edges of 111M nodes took 4.7 ms in k_es_score_bins, 0.75 on permuted ids.
constexpr uint32_t kCrowdPiece = 65535;            // pairs per turn: the two counts of a node fit 16 bits each
__global__ __launch_bounds__(kBlock) void k_es_crowd(int64_t chunk, EsBins tab, uint32_t bn, uint32_t nblocks,
                                                     const uint32_t* __restrict__ pairs, EsCrowd crowd)
{
    extern __shared__ uint32_t cnt[];              // bn words, then as many bits
    __shared__ uint32_t wsum[kWaves], first[kBins + 1];
    __shared__ uint16_t bin_of[kBins];
    uint32_t* seen = cnt + bn;
    const int tid = threadIdx.x, cb = tab.cb;
    const uint32_t bins = crowd.bins[chunk], blocks = (1u << cb) / bn;
    const uint32_t own = tab.nb / kBlock;          // neighbouring places of a thread
    for (uint32_t i = tid; i < tab.nb; i += kBlock) {
        const uint32_t place = crowd.place[(size_t)chunk * tab.nb + i];
        if (place) bin_of[place - 1u] = (uint16_t)i;
    }
    __syncthreads();
    auto turns = [&](uint32_t at) {
        if (at >= bins) return 0u;
        uint32_t p0, p1;
        tab.range(chunk, bin_of[at], p0, p1);
        return (p1 - p0 + kCrowdPiece - 1u) / kCrowdPiece * blocks;
    };
    uint32_t items = 0;
    for (uint32_t i = 0; i < own; ++i) items += turns(tid * own + i);
    uint32_t excl = es_block_exclusive(items, wsum);
    for (uint32_t i = 0; i < own; ++i) {
        first[tid * own + i] = excl;
        excl += turns(tid * own + i);
    }
    if (tid == kBlock - 1) first[tab.nb] = excl;
    __syncthreads();
    uint32_t at = 0;                               // the crowded bin of the item
    for (uint32_t item = blockIdx.x; item < first[tab.nb]; item += gridDim.x) {
        while (item >= first[at + 1u]) ++at;
        const uint32_t bin = bin_of[at], part = item - first[at], low = part % blocks * bn;
        if (((bin << cb) + low) / bn >= nblocks) continue;                   // (past the last block; the same for all threads)
        uint32_t p0, p1;
        tab.range(chunk, bin, p0, p1);
        p0 += part / blocks * kCrowdPiece;
        if (p1 - p0 > kCrowdPiece) p1 = p0 + kCrowdPiece;
        for (uint32_t i = tid; i < bn; i += kBlock) cnt[i] = 0u;
        for (uint32_t i = tid; i < bn / 32; i += kBlock) seen[i] = 0u;
        __syncthreads();
        constexpr int U = 8;
        for (uint32_t i = p0 + tid; i < p1; i += kBlock * U) {
            uint32_t x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = p1 - i > (uint32_t)(u * kBlock) ? pairs[i + u * kBlock] : 0xFFFFFFFFu;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t rel = (x[u] & ((1u << cb) - 1u)) - low, code = x[u] >> cb;
                if (x[u] == 0xFFFFFFFFu || rel >= bn) continue;
                if (code >= 2u) atomicOr(&seen[rel >> 5], 1u << (rel & 31u));
                else atomicAdd(&cnt[rel], code ? 65536u : 1u);
            }
            if (p1 - i <= (uint32_t)(kBlock * U)) break;
        }
        __syncthreads();
        const size_t node = ((size_t)at << cb) + low;
        for (uint32_t i = tid; i < bn; i += kBlock) {
            const uint32_t c = cnt[i];
            if (c) atomicAdd(&crowd.hc[node + i], (u64)(c & 0xFFFFu) | (u64)(c >> 16) << 32);
        }
        for (uint32_t i = tid; i < bn / 32; i += kBlock)
            if (seen[i]) atomicOr(&crowd.seen[node / 32 + i], seen[i]);
        __syncthreads();
    }
}

// From the counts in memory; clears what it consumed (hc, mark).  first: the seeded first chunk (estimates only).
// fixed: fixed greedy decisions (a node that has a label is left alone).
// A wave has the counts of kTurn words in flight, and blocks are as small as it takes to fill the chip (es_shape):
// when every wave walked 64 words one load at a time this took 54 us for 20,000 nodes, 5.3 now.
__global__ __launch_bounds__(kBlock) void k_es_score(EsRun st, int par, int first, int fixed, u64* hc)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t gi = es_group_of(st, blockIdx.x);
    const long long P = es_group(st, gi).P;
    const long long S0 = (long long)st.S[2 * (par * st.ngroups + gi)], S1 = (long long)st.S[2 * (par * st.ngroups + gi) + 1];
    const uint32_t word0 = ((uint32_t)blockIdx.x * kWaves + wave) * st.wpw;
    const bool mine = lane < st.wpw;
    const u64 myword = mine ? st.mark[word0 + lane] : 0ull;
    const EsLabels labels = mine ? es_load_labels(st, word0 + lane) : EsLabels{0ull, 0ull};
    u64 out0 = 0ull, out1 = 0ull;
    for (int i0 = 0; i0 < st.wpw; i0 += kTurn) {
        u64 h[kTurn];
        bool on[kTurn];
        uint32_t h0[kTurn], h1[kTurn];
#pragma unroll
        for (int u = 0; u < kTurn; ++u) h[u] = i0 + u < st.wpw ? hc[(size_t)(word0 + i0 + u) * 64 + lane] : 0ull;
#pragma unroll
        for (int u = 0; u < kTurn; ++u) {
            const u64 word = i0 + u < st.wpw ? es_bcast(myword, (i0 + u) & 63) : 0ull;
            on[u] = h[u] != 0ull || ((word >> lane) & 1ull);
            if (h[u]) hc[(size_t)(word0 + i0 + u) * 64 + lane] = 0ull;
            h0[u] = (uint32_t)h[u];
            h1[u] = (uint32_t)(h[u] >> 32);
        }
        es_score_words(st, word0, i0, labels, on, h0, h1, first, fixed, P, S0, S1, out0, out1);
    }
    uint32_t movers[4] = {0u, 0u, 0u, 0u};
    if (mine) {
        es_store_words(st, word0 + lane, out0, out1, labels, movers);
        if (myword) st.mark[word0 + lane] = 0ull;
    }
    es_store_movers(st, movers, blockIdx.x);
}

// LDS of k_es_score_bins: two words per 32 nodes, and six bytes for each of `room` nodes of the chunk or, where a count is kept
// for every node, four and a bit per node
inline size_t es_bins_lds(int64_t bn, int64_t room) { return (size_t)bn / 4 + (size_t)room * 6; }

// The pairs [p0, p1), four at a time from the last whole four before them on (the list's end is padded), U fours per lane
// and turn, the next turn's on their way.
struct EsPairs {
    static constexpr int U = 2;
    const uint4* fours;
    uint32_t p0, p1, q1, q;
    uint4 x[U];
    __device__ __forceinline__ void request()
    {
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (q + u * kBlock < q1) x[u] = fours[q + u * kBlock];
    }
    __device__ __forceinline__ void start() { q = (p0 >> 2) + threadIdx.x; request(); }
    template <typename F> __device__ __forceinline__ void each(F&& f)
    {
        for (; q < q1;) {
            uint4 y[U];
            const uint32_t at = q;
#pragma unroll
            for (int u = 0; u < U; ++u) y[u] = x[u];
            q += U * kBlock;
            request();
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = 4u * (at + u * kBlock);
                if (i >= p0 && i + 4u <= p1) {
                    f(y[u].x); f(y[u].y); f(y[u].z); f(y[u].w);
                } else {                           // the list's ends
                    if (i - p0 < p1 - p0) f(y[u].x);
                    if (i + 1u - p0 < p1 - p0) f(y[u].y);
                    if (i + 2u - p0 < p1 - p0) f(y[u].z);
                    if (i + 3u - p0 < p1 - p0) f(y[u].w);
                }
            }
        }
    }
};

// cnt_nbrs, second half, from the binned pairs: a block counts the pairs of its bin that are its own in LDS, then scores its nodes.
// One node in eight belongs to a chunk of one per cent: a bitmap of the chunk's nodes, ranked, gives each of them a place in a
// list and in the counts, so that the LDS holds six bytes for a node of the chunk instead of four for every node, two workgroups
// share a CU, and a lane has a node of the chunk each time.  Where chunks hold most nodes (`sparse` is not set) and in a bin with more of them
// than there is `room` for, every node has its count (`direct`; of 32 bits in a bin of more than 65,535 pairs), in
// rounds of as many nodes as fit; those of a crowded bin come from memory (k_es_crowd).  In an order of degree such blocks are what a
// launch waits for: labels and estimates are asked for before the counts are looked at, crowded bins take one round, and neighbours go to
// different XCDs (14M nodes by degree, 4M ends: 85 -> 66 us).
// What bounds it is the estimates: the 64-byte pieces that hold one of the chunk's nodes are written (8 bytes per node: 450 MB at 111M
// nodes and 32M ends, 14M nodes of the chunk), and 128-byte lines read (1 GB).  With doubles, 16 bytes per node, stores alone were 225 us of 555; now 410.
// 14M nodes, 4M ends: 65 -> 42 us.  Nontemporal loads or stores of the estimates were slower, or no faster; four nodes per lane in flight spill.
constexpr int kScoreTurn = 2;                      // nodes a lane has in flight
constexpr int kPlaceTurn = 2;                      // ... whose counts come from memory
constexpr uint32_t kListPairs = 4;                 // a block whose bin has more pairs than so many times `room` (50,000: a count fits 16 bits) does not try a list
                                                   // (14M nodes, four partitions by degree, sixteen permuted: 2 30.7 and 39.6 ms, 3 30.8 and 36.6, 4 30.6 and
                                                   // 33.5, any 31.5 and 34.0: a dense group's bins have many pairs of few nodes)
__global__ __launch_bounds__(kBlock, 8) void k_es_score_bins(EsRun st, int par, int first, int fixed, int64_t chunk, EsBins tab,
                                                             uint32_t nblocks, uint32_t room, int sparse,
                                                             const uint32_t* __restrict__ pairs, EsCrowd crowd)
{
    extern __shared__ uint32_t bits[];             // list: the chunk's nodes among the block's
    __shared__ uint32_t wsum[kWaves], wide;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, cb = tab.cb;
    const uint32_t bn = (uint32_t)(kBlock * st.wpw);
    // Workgroups go to the XCDs in turn.  Neighbouring blocks, which in an order of degree or a sorted list are alike, to different ones, unless
    // they read the same bin.
    const uint32_t block = bn >> cb ? blockIdx.x : (blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
    if (block >= nblocks) return;
    const uint32_t node0 = block * bn;
    const uint32_t bin = node0 >> cb, in_bin = node0 & ((1u << cb) - 1u);
    uint32_t p0, p1;
    tab.range(chunk, bin, p0, p1);
    const uint32_t place = crowd.place[(size_t)chunk * tab.nb + bin];                // not 0: counted by k_es_crowd
    if (place) p1 = p0;
    EsPairs list{reinterpret_cast<const uint4*>(pairs), p0, p1, (p1 + 3u) >> 2, 0u, {}};
    list.start();
    const uint32_t gi = es_group_of(st, block);
    const long long P = es_group(st, gi).P, S0 = (long long)st.S[2 * (par * st.ngroups + gi)], S1 = (long long)st.S[2 * (par * st.ngroups + gi) + 1];
    // what `assign` answers, by label and lean: bit 3 * label + lean + 1
    const uint32_t answers = (uint32_t)__ballot(lane < 9 && es_assign(lane % 3 - 1, S0 - (lane < 3), S1 - (lane >= 3 && lane < 6), P));
    const uint32_t words = bn / 32;
    uint32_t *mv0 = bits, *mv1 = bits + words, *base = mv1;                          // base: the chunk's nodes before a word
    uint32_t* cnt = bits + 2 * words;
    uint16_t* nodes = reinterpret_cast<uint16_t*>(cnt + room);
    const bool whole = st.packed == nullptr;                                         // the estimates are all doubles
    if (tid == 0 && !whole) wide = st.wide[block];

    // the score of a node of the chunk: its label's word, its estimate as stored (if any is looked at) and its counts
    const bool stored = !first && !fixed && !whole;
    auto settle = [&](uint32_t rel, u64 labels, uint2 est, uint32_t h0, uint32_t h1) {
        const uint32_t old = es_label(labels, rel);                // (a block starts at a whole word)
        if (fixed && !first && old != kNone) return;
        const bool blend = !first && !fixed && old != kNone;
        double2 doubles = make_double2(0.0, 0.0);
        if (!blend) est = make_uint2(0u, 0u);
        if (whole) est = es_wide_word(node0 + rel);
        if (blend && es_is_wide(est)) doubles = st.est[es_wide_place(est)];
        const int lean = es_blend_packed(st, node0 + rel, est, doubles, blend, h0, h1, node0, &wide);
        if (first) return;
        const uint32_t t = answers >> (3u * old + (uint32_t)(lean + 1)) & 1u;
        if (t != old) atomicOr(&(t ? mv1 : mv0)[rel >> 5], 1u << (rel & 31u));
    };
    // counts of `count` nodes from `low` on (or, listed, of those in nodes[]) are there: their scores
    auto score = [&](uint32_t count, uint32_t low, bool listed, bool narrow, const uint32_t* seen) {
        for (uint32_t i0 = tid; i0 < count; i0 += kBlock * kScoreTurn) {
            uint32_t rel[kScoreTurn], h0[kScoreTurn], h1[kScoreTurn];
            uint2 est[kScoreTurn];
            u64 labels[kScoreTurn];
            bool on[kScoreTurn];
#pragma unroll
            for (int u = 0; u < kScoreTurn; ++u) {
                const uint32_t i = i0 + u * kBlock;
                on[u] = i < count;
                const uint32_t at = on[u] ? i : 0u;
                rel[u] = listed ? nodes[at] : low + at;
                if (narrow) {
                    h0[u] = cnt[at] & 0xFFFFu;
                    h1[u] = cnt[at] >> 16;
                } else {
                    h0[u] = cnt[2u * at];
                    h1[u] = cnt[2u * at + 1u];
                }
                if (!listed) on[u] &= (h0[u] | h1[u]) != 0u || ((seen[at >> 5] >> (at & 31u)) & 1u);
                est[u] = make_uint2(0u, 0u);
                labels[u] = 0ull;
                if (on[u] || !listed) labels[u] = st.Lw[(node0 + rel[u]) >> 5];
                if ((on[u] || !listed) && stored) est[u] = reinterpret_cast<const uint2*>(st.packed)[node0 + rel[u]];
            }
#pragma unroll
            for (int u = 0; u < kScoreTurn; ++u)
                if (on[u]) settle(rel[u], labels[u], est[u], h0[u], h1[u]);
        }
    };

    if (place) {
        // counted in memory, where what is taken is cleared; most of its nodes belong to the chunk, and everything is asked for at once
        u64* hc = crowd.hc + (((size_t)place - 1) << cb) + in_bin;
        uint32_t* was_seen = crowd.seen + ((((size_t)place - 1) << cb) + in_bin) / 32;
        for (uint32_t i = tid; i < words; i += kBlock) mv0[i] = mv1[i] = 0u;
        __syncthreads();
        for (uint32_t i0 = tid; i0 < bn; i0 += kBlock * kPlaceTurn) {             // (bn is a multiple of it)
            u64 h[kPlaceTurn], labels[kPlaceTurn];
            uint32_t seen[kPlaceTurn];
            uint2 est[kPlaceTurn];
#pragma unroll
            for (int u = 0; u < kPlaceTurn; ++u) {
                const uint32_t rel = i0 + u * kBlock;
                h[u] = hc[rel];
                seen[u] = was_seen[rel >> 5];
                labels[u] = st.Lw[(node0 + rel) >> 5];
                est[u] = stored ? reinterpret_cast<const uint2*>(st.packed)[node0 + rel] : make_uint2(0u, 0u);
            }
#pragma unroll
            for (int u = 0; u < kPlaceTurn; ++u) {
                const uint32_t rel = i0 + u * kBlock;
                if (h[u]) hc[rel] = 0ull;
                if (seen[u] && (rel & 31u) == 0u) was_seen[rel >> 5] = 0u;       // (read by this wave alone)
                if (h[u] || ((seen[u] >> (rel & 31u)) & 1u)) settle(rel, labels[u], est[u], (uint32_t)h[u], (uint32_t)(h[u] >> 32));
            }
        }
    }
    bool direct = !sparse || p1 - p0 > kListPairs * room;
    if (!direct && !place) {
        for (uint32_t i = tid; i < words; i += kBlock) bits[i] = 0u;
        __syncthreads();
        list.each([&](uint32_t pair) {
            const uint32_t rel = (pair & ((1u << cb) - 1u)) - in_bin;
            if (rel < bn) atomicOr(&bits[rel >> 5], 1u << (rel & 31u));
        });
        list.start();
        __syncthreads();
        const uint32_t own = words > (uint32_t)kBlock ? words / kBlock : 1u;       // neighbouring words of a thread
        uint32_t in_own = 0, total;
        for (uint32_t i = 0; i < own; ++i) in_own += tid * own + i < words ? (uint32_t)__popc(bits[tid * own + i]) : 0u;
        uint32_t before = es_block_exclusive(in_own, wsum, &total);
        direct = total > room;
        if (!direct) {
            for (uint32_t i = 0; i < own && tid * own + i < words; ++i) {
                const uint32_t w = tid * own + i;
                base[w] = before;
                for (uint32_t rest = bits[w]; rest; rest &= rest - 1u) nodes[before++] = (uint16_t)(w * 32u + (uint32_t)__builtin_ctz(rest));
            }
            for (uint32_t i = tid; i < total; i += kBlock) cnt[i] = 0u;
            __syncthreads();
            list.each([&](uint32_t pair) {
                const uint32_t rel = (pair & ((1u << cb) - 1u)) - in_bin, code = pair >> cb;
                if (rel >= bn) return;
                const uint32_t at = base[rel >> 5] + (uint32_t)__popc(bits[rel >> 5] & ((1u << (rel & 31u)) - 1u));
                if (code < 2u) atomicAdd(&cnt[at], code ? 65536u : 1u);
            });
            __syncthreads();
            for (uint32_t i = tid; i < words; i += kBlock) mv0[i] = mv1[i] = 0u;
            __syncthreads();
            score(total, 0u, true, true, nullptr);
        } else {
            __syncthreads();                       // (bits are read no more)
        }
    }
    if (direct && !place) {
        // counts for every node, in rounds of as many as there is room for
        const bool narrow = p1 - p0 <= 65535u;
        uint32_t sub = bn;
        while ((narrow ? sub : 2u * sub) + sub / 32u > room + room / 2u) sub /= 2u;
        uint32_t* seen = cnt + (narrow ? sub : 2u * sub);
        for (uint32_t i = tid; i < words; i += kBlock) mv0[i] = mv1[i] = 0u;
        for (uint32_t low = 0; low < bn; low += sub) {
            list.start();
            for (uint32_t i = tid; i < (narrow ? sub : 2u * sub) + sub / 32u; i += kBlock) cnt[i] = 0u;
            __syncthreads();
            list.each([&](uint32_t pair) {
                const uint32_t rel = (pair & ((1u << cb) - 1u)) - in_bin - low, code = pair >> cb;
                if (rel >= sub) return;
                if (code >= 2u) atomicOr(&seen[rel >> 5], 1u << (rel & 31u));
                else if (narrow) atomicAdd(&cnt[rel], code ? 65536u : 1u);
                else atomicAdd(&cnt[2u * rel + code], 1u);
            });
            __syncthreads();
            score(sub, low, false, narrow, seen);
            __syncthreads();
        }
    }
    __syncthreads();
    uint32_t movers[4] = {0u, 0u, 0u, 0u};
    const int nw = st.wpw;
    const uint32_t word0 = node0 / 64 + wave * nw;
    if (lane < nw)
        es_store_words(st, word0 + lane, reinterpret_cast<const u64*>(mv0)[wave * nw + lane], reinterpret_cast<const u64*>(mv1)[wave * nw + lane],
                       es_load_labels(st, word0 + lane), movers);
    es_store_movers(st, movers, block);
    if (tid == 0 && !whole) st.wide[block] = wide;
}

// the first c set bits of x (c <= their number).  Between "none" and "all" there is one word per partition and chunk.
__device__ __forceinline__ u64 es_first_bits(u64 x, long long c)
{
    if (c >= (long long)__popcll(x)) return x;
    u64 rest = x;
    for (; c > 0; --c) rest &= rest - 1ull;
    return x ^ rest;
}

// The rejected new nodes of the group that asked for partition p (more movers ask for it than `room`), in blocks before
// `own` and in all: every block's movers are in order, so all after the room-th of them are rejected; the block in
// which the room runs out is looked at word by word.
__device__ __forceinline__ void es_rejected(const EsRun& st, uint32_t blk0, uint32_t nblk, int p, long long room, uint32_t own, uint32_t& before, uint32_t& all)
{
    __shared__ uint32_t wsum[kWaves], s_block, s_first;
    const u64* __restrict__ mv = p ? st.mv1 : st.mv0;
    const uint32_t last = (uint32_t)room;          // rank of the first that is rejected
    uint32_t carry = 0, out[2] = {0u, 0u};         // before own, in all
    for (uint32_t base = blk0; base < blk0 + nblk; base += kBlock) {
        const uint32_t b = base + threadIdx.x;
        uint4 q = make_uint4(0u, 0u, 0u, 0u);
        if (b < blk0 + nblk) q = st.bs[b];
        const uint32_t x = p ? q.y : q.x, fresh = p ? q.w : q.z;
        uint32_t turn;
        const uint32_t first = carry + es_block_exclusive(x, wsum, &turn);
        if (last >= first && last - first < x) { s_block = b; s_first = first; }
        if (first > last) {                        // all of its movers are rejected
            out[1] += fresh;
            if (b < own) out[0] += fresh;
        }
        carry += turn;
        __syncthreads();
    }
    // the block itself: a thread per word
    const uint32_t block = s_block, words = (uint32_t)(kWaves * st.wpw), word = block * words + threadIdx.x;
    const u64 m = threadIdx.x < words ? mv[word] : 0ull, fresh = threadIdx.x < words ? st.nw[word] : 0ull;       // (words <= kBlock)
    const long long rank = (long long)s_first + es_block_exclusive((uint32_t)__popcll(m), wsum);
    const uint32_t here = (uint32_t)__popcll((m & ~es_first_bits(m, room - rank)) & fresh);
    out[1] += here;
    if (block < own) out[0] += here;
    es_block_sums(out);
    before = out[0];
    all = out[1];
    __syncthreads();
}

// Admission: a mover whose rank among the chunk's requests for its target (ascending id) is below
// the room the target had when the chunk started is relabelled (fix_sizes, Alg. 2).  Rejected new nodes are placed one by
// one, ascending id, in the smaller partition (0 on a tie), in closed form: the first |difference| go to the smaller one,
// the rest alternate 0,1,...  Every block adds up its group's movers itself, and where a partition has not room for all of
// them also the rejected ones of the blocks before it; the group's first block writes the sizes after the chunk to
// their other copy.
// A lane takes W neighbouring words of 64 nodes (awpw = 64 * W words per wave, or fewer with W = 1): the admitted movers
// of a word are its first bits, as many as there is room for, the alternation over rejected ones is a prefix parity, and labels
// change in a few bit operations.  W and awpw: so many that 256 blocks or fewer do it up to 33M nodes in one group, as each adds up
// all blocks' counts; beyond that a block takes 131,072 nodes, 848 of them 111M (es_shape; with twice as many, and 92 registers, 52 us for 43).  In two
// launches (admission, spill), with labels of a byte each and movers taken one by one: 103 us per chunk at 111M nodes, 13 at 20,000; so 43 and 6.
template <int W>
__global__ __launch_bounds__(kBlock) void k_es_admit(EsRun st, int par)
{
    __shared__ uint32_t c0[kWaves], c1[kWaves], co[kWaves];
    const int lane = threadIdx.x & 63, wave = es_wave(), awpw = st.awpw;
    const uint32_t own = (uint32_t)blockIdx.x * (uint32_t)(awpw / st.wpw);            // its first block of the scoring
    const uint32_t gi = es_group_of(st, own);
    const EsGroup g = es_group(st, gi);
    const uint32_t blk0 = g.blk0, nblk = g.nblk;
    const uint32_t word0 = ((uint32_t)blockIdx.x * kWaves + wave) * awpw + lane * W;
    const bool mine = lane * W < awpw;
    u64 my0[W], my1[W], fresh[W];
    EsLabels old[W];
    uint32_t n0 = 0, n1 = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        my0[i] = mine ? st.mv0[word0 + i] : 0ull;
        my1[i] = mine ? st.mv1[word0 + i] : 0ull;
        fresh[i] = mine ? st.nw[word0 + i] : 0ull;
        old[i] = mine ? es_load_labels(st, word0 + i) : EsLabels{0ull, 0ull};
    }
    uint32_t sums[6] = {0u, 0u, 0u, 0u, 0u, 0u};   // movers to 0 and 1: in earlier blocks, in all; those of all without a label
    for (uint32_t b = blk0 + threadIdx.x; b < blk0 + nblk; b += kBlock) {
        const uint4 q = st.bs[b];
        if (b < own) { sums[0] += q.x; sums[1] += q.y; }
        sums[2] += q.x; sums[3] += q.y;
        sums[4] += q.z; sums[5] += q.w;
    }
#pragma unroll
    for (int i = 0; i < W; ++i) { n0 += (uint32_t)__popcll(my0[i]); n1 += (uint32_t)__popcll(my1[i]); }
    es_block_sums(sums);
    const long long P = g.P;
    const long long S0 = (long long)st.S[2 * (par * st.ngroups + gi)], S1 = (long long)st.S[2 * (par * st.ngroups + gi) + 1];
    const long long room0 = P - S0 > 0 ? P - S0 : 0, room1 = P - S1 > 0 ? P - S1 : 0;
    long long rank0 = (long long)(sums[0] + es_block_exclusive(n0, c0)), rank1 = (long long)(sums[1] + es_block_exclusive(n1, c1));
    const long long all0 = (long long)sums[2], all1 = (long long)sums[3];
    // rejected new nodes: in earlier blocks, in all, by what they asked for
    uint32_t out_before = 0, out0 = 0, out1 = 0;
    if (all0 > room0) es_rejected(st, blk0, nblk, 0, room0, own, out_before, out0);
    if (all1 > room1) { uint32_t more; es_rejected(st, blk0, nblk, 1, room1, own, more, out1); out_before += more; }
    const long long adm0 = all0 < room0 ? all0 : room0, adm1 = all1 < room1 ? all1 : room1;
    const long long new0 = (long long)(sums[4] - out0), new1 = (long long)(sums[5] - out1);      // admitted
    const long long a = S0 + adm0 - (adm1 - new1), b = S1 + adm1 - (adm0 - new0);                // sizes after the admissions
    const long long gap = a <= b ? b - a : a - b, total = (long long)out0 + (long long)out1;
    if (own == blk0 && threadIdx.x == 0) {
        const long long lead = total < gap ? total : gap, rest = total - lead;
        u64* next = st.S + 2 * ((par ^ 1) * st.ngroups + gi);
        next[0] = (u64)(a + (a <= b ? lead : 0) + (rest + 1) / 2);
        next[1] = (u64)(b + (a <= b ? 0 : lead) + rest / 2);
    }
    u64 to0[W], to1[W];
    uint32_t outs = 0;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        to0[i] = es_first_bits(my0[i], room0 - rank0);
        to1[i] = es_first_bits(my1[i], room1 - rank1);
        rank0 += __popcll(my0[i]);
        rank1 += __popcll(my1[i]);
        fresh[i] &= (my0[i] | my1[i]) & ~(to0[i] | to1[i]);                          // rejected
        outs += (uint32_t)__popcll(fresh[i]);
    }
    long long j = (long long)out_before;                                             // placements before the lane's
    if (total) j += (long long)es_block_exclusive(outs, co);
#pragma unroll
    for (int i = 0; i < W; ++i) {
        if (!(to0[i] | to1[i] | fresh[i])) continue;
        const u64 lead = es_first_bits(fresh[i], gap - j), rest = fresh[i] ^ lead;
        u64 odd = rest;                                                              // bit x: an odd number of bits of rest up to x
        if (rest)
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) odd ^= odd << o;
        const long long first = j + __popcll(lead) - gap;                            // of rest, among those that alternate
        const u64 ones = to1[i] | (a <= b ? 0ull : lead) | (rest & ((first & 1) ? odd : ~odd));
        es_store_labels(st, word0 + i, {old[i].has | to0[i] | to1[i] | fresh[i], (old[i].one & ~to0[i]) | ones});
        j += __popcll(fresh[i]);
    }
}

__global__ __launch_bounds__(256) void k_es_expand(int64_t n, const u64* __restrict__ Lw, int32_t* parts,
                                                   const u64* S, int64_t* sizes_out)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const uint32_t l = es_label(Lw[v >> 5], (uint32_t)v);
        parts[v] = l == kNone ? -1 : (int32_t)l;
    }
    if (sizes_out && blockIdx.x == 0 && threadIdx.x < 2) sizes_out[threadIdx.x] = (int64_t)S[threadIdx.x];
}

// nbr_counts_out of a run that kept its estimates in 8 bytes
__global__ __launch_bounds__(256) void k_es_expand_packed(int64_t n, EsRun st, double2* out)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const uint2 word = reinterpret_cast<const uint2*>(st.packed)[v];
        out[v] = es_is_wide(word) ? st.est[es_wide_place(word)] : es_unpack(word);
    }
}

// listed edges whose ends carry different labels (Sec. 1)
__global__ __launch_bounds__(256) void k_es_cut(const int32_t* __restrict__ src, const int32_t* __restrict__ dst, int64_t m,
                                                const int32_t* __restrict__ parts, u64* cut)
{
    __shared__ u64 wsum[4];
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    u64 c = 0;
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < m; e += stride)
        c += parts[src[e]] != parts[dst[e]];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) c += __shfl_down(c, o);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) {
        const u64 t = wsum[0] + wsum[1] + wsum[2] + wsum[3];
        if (t) atomicAdd(cut, t);
    }
}

// ---- recursive bisection (Sec. 4.1: more than two partitions by splitting every part in two) ------
//
// Per level the edges that still lie inside a group are kept grouped by group, in stream order, and
// already written in the group's own node numbers (0..nv-1 in ascending id), so that a group's
// segment is the input of the two-partition run as it stands.  Per level and group there is also
// the list of its nodes' ids (and their seed bits) in that numbering.  When the groups have been split,
// every node gets its number inside its half (its rank among the nodes of the same half), the
// halves' node lists are written, and the groups' edges are rewritten in those numbers while they
// are sorted into "both ends in half 0", "both ends in half 1" and "ends part" (dropped).

constexpr int kSelBlock = 1024;     // stable selection of edges: a thread owns kSelPer consecutive edges
constexpr int kSelPer = 4;
constexpr int kSelTile = kSelBlock * kSelPer;

// per block: its nodes with label 0 and its nodes without a label
__global__ __launch_bounds__(kBlock) void k_rb_count(EsRun st)
{
    const EsGroup g = es_group(st, es_group_of(st, blockIdx.x));
    const uint32_t bw = (uint32_t)(kWaves * st.wpw), word = blockIdx.x * bw + threadIdx.x, v = word * 64u - g.node0;   // (a thread per word)
    uint32_t n[2] = {0u, 0u};
    if (threadIdx.x < bw && v < g.nv) {
        const EsLabels l = es_load_labels(st, word);
        const u64 in = g.nv - v < 64u ? (1ull << (g.nv - v)) - 1ull : ~0ull;
        n[0] = (uint32_t)__popcll(l.has & ~l.one);
        n[1] = (uint32_t)__popcll(in & ~l.has);
    }
    es_block_sums(n);
    if (threadIdx.x == 0) st.bs[blockIdx.x] = make_uint4(n[0], n[1], 0u, 0u);
}

// Nodes the two-partition run left without a label (no edge inside the group) are placed one by one, ascending id,
// in the currently smaller half (0 on a tie): the first |difference| of them go to the smaller half, the rest
// alternate 0,1,... .  So the node of half 0 with z labelled zeros and j unlabelled nodes before it is number
// z + (zeros among the first j placements) of its half, and nothing but the two counts per block is needed.
// halves[]: per 32 nodes of the state the nodes of half 1 (low half) and how many of the group's nodes before them are of half
// 0 (high half), from which a node's number inside its half follows: a quarter of a byte per node, which every L2 holds up to
// some 16M nodes (28 MB at 111M), is what the edges' ends are looked up in.  The halves' node lists (ids and next level's seed bits) are written, half 0 first.  At the
// last level the labels 2 * group + half go out instead.  gof == nullptr: node i has id i.  nodes0[group]: nodes of half 0.
__global__ __launch_bounds__(kBlock) void k_rb_children(EsRun st, int par, const int32_t* __restrict__ gof,
                                                        const int32_t* __restrict__ next_bits, u64* halves,
                                                        int32_t* gof_next, int32_t* seed_next, int32_t* labels_out,
                                                        long long* nodes0)
{
    __shared__ uint32_t cz[kWaves], cn[kWaves];
    const int lane = threadIdx.x & 63, wave = es_wave(), wpw = st.wpw;
    const uint32_t gi = es_group_of(st, blockIdx.x);
    const EsGroup g = es_group(st, gi);
    uint32_t sums[4] = {0u, 0u, 0u, 0u};          // zeros and nodes without a label: in earlier blocks, in all
    for (uint32_t b = g.blk0 + threadIdx.x; b < g.blk0 + g.nblk; b += kBlock) {
        const uint32_t z = st.bs[b].x, e = st.bs[b].y;
        sums[2] += z; sums[3] += e;
        if (b < blockIdx.x) { sums[0] += z; sums[1] += e; }
    }
    es_block_sums(sums);
    const uint32_t zeros_all = sums[2], nones_all = sums[3];
    const long long S0 = (long long)st.S[2 * (par * st.ngroups + gi)], S1 = (long long)st.S[2 * (par * st.ngroups + gi) + 1];
    const long long gap = S0 <= S1 ? S1 - S0 : S0 - S1;
    const bool lead0 = S0 <= S1;
    auto placed0 = [&](long long j) {                 // zeros among the first j placements
        const long long lead = j < gap ? j : gap;
        return (lead0 ? lead : 0ll) + (j - lead + 1) / 2;
    };
    const long long count0 = (long long)zeros_all + placed0((long long)nones_all);
    if (blockIdx.x == g.blk0 && threadIdx.x == 0) nodes0[g.id] = count0;
    // a wave's nodes: its words one after the other; their counts of zeros and of nodes without a label
    const uint32_t first = ((uint32_t)blockIdx.x * kWaves + wave) * wpw * 64u;
    const uint32_t own0 = first - g.node0 + lane * 64u;          // first node of the lane's word
    EsLabels mine{0ull, 0ull};
    if (lane < wpw) mine = es_load_labels(st, first / 64u + lane);
    const u64 nodes = lane >= wpw || own0 >= g.nv ? 0ull : g.nv - own0 < 64u ? (1ull << (g.nv - own0)) - 1ull : ~0ull;
    const u64 my_zeros = mine.has & ~mine.one, my_nones = nodes & ~mine.has;
    uint32_t zeros = sums[0] + es_lane(es_block_exclusive((uint32_t)__popcll(my_zeros), cz), 0);          // before the wave's
    uint32_t nones = sums[1] + es_lane(es_block_exclusive((uint32_t)__popcll(my_nones), cn), 0);
    const u64 below = (1ull << lane) - 1ull;
    u64 ones = 0ull;                                  // lane i: the nodes of half 1 of the wave's word i, and the group's nodes
    uint32_t before = 0;                              // of half 0 before it
    for (int i = 0; i < wpw; ++i) {
        const uint32_t v = first + i * 64u + lane;
        const bool in = v - g.node0 < g.nv;
        const u64 bz = es_bcast(my_zeros, i), bn = es_bcast(my_nones, i);
        const uint32_t l = ((bz >> lane) & 1ull) ? 0u : ((bn >> lane) & 1ull) ? kNone : 1u;
        const long long z = (long long)zeros + __popcll(bz & below), j = (long long)nones + __popcll(bn & below);
        const uint32_t half = l != kNone ? l : j < gap ? (lead0 ? 0u : 1u) : (uint32_t)((j - gap) & 1);
        const u64 word = __ballot(in && half == 1u);
        if (lane == i) { ones = word; before = zeros + (uint32_t)placed0((long long)nones); }
        zeros += __popcll(bz);
        nones += __popcll(bn);
        if (!in) continue;
        const int64_t own = (int64_t)(v - g.node0);
        const int32_t id = gof ? gof[g.v_lo + own] : (int32_t)own;
        if (labels_out) { labels_out[id] = 2 * (int32_t)g.id + (int32_t)half; continue; }
        const long long r0 = z + placed0(j);          // nodes of half 0 before this one
        const long long num = half == 0u ? r0 : own - r0;
        const int64_t at = g.v_lo + (half == 0u ? num : count0 + num);
        gof_next[at] = id;
        seed_next[at] = next_bits[id];
    }
    // (of a word that ends inside, only the nodes that there are get looked up)
    if (!labels_out && lane < wpw) {
        const uint32_t next = before + 32u - (uint32_t)__popc((uint32_t)ones);
        reinterpret_cast<ulonglong2*>(halves)[first / 64u + lane] =
            make_ulonglong2((ones & 0xFFFFFFFFull) | (u64)before << 32, ones >> 32 | (u64)next << 32);
    }
}

// half of the node in bit 31, its number inside the half below it
__device__ __forceinline__ uint32_t rb_number(u64 word, uint32_t v)
{
    const uint32_t ones = (uint32_t)word, bit = 1u << (v & 31u);
    const uint32_t zeros = (uint32_t)(word >> 32) + (uint32_t)__popc(~ones & (bit - 1u));
    return ones & bit ? (v - zeros) | 0x80000000u : zeros;
}

// An edge of a group goes to the half both its ends are in (key 0 / 1) or is dropped (key 2); its
// ends are rewritten in the halves' node numbers (tmp_s, tmp_d) for the scatter.  The random look-ups bound it: three levels of
// 200M edges and 14M nodes took 15.5 ms from a table of 4 bytes per node, 3.4 from the 3.5 MB of `halves`.
__global__ __launch_bounds__(kSelBlock) void k_rb_split_count(const EsGroup* __restrict__ groups, const int32_t* __restrict__ src,
                                                              const int32_t* __restrict__ dst, const u64* __restrict__ halves,
                                                              uint8_t* __restrict__ key, int32_t* __restrict__ tmp_s,
                                                              int32_t* __restrict__ tmp_d, uint32_t* bc0, uint32_t* bc1)
{
    __shared__ uint32_t c0[kSelBlock / 64], c1[kSelBlock / 64];
    const EsGroup g = groups[blockIdx.y];
    if ((int64_t)blockIdx.x * kSelTile >= g.m) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u64* __restrict__ own = halves + (g.node0 >> 5);           // (a group starts at a whole block)
    const int64_t end = g.e_lo + g.m;
    const int64_t e0 = g.e_lo + (int64_t)blockIdx.x * kSelTile + threadIdx.x;
    uint32_t n0 = 0, n1 = 0, s[kSelPer], d[kSelPer];
    u64 a[kSelPer], b[kSelPer];
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
        const int64_t e = e0 + u * kSelBlock;
        s[u] = e < end ? (uint32_t)__builtin_nontemporal_load(src + e) : 0u;
        d[u] = e < end ? (uint32_t)__builtin_nontemporal_load(dst + e) : 0u;
    }
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) { a[u] = own[s[u] >> 5]; b[u] = own[d[u] >> 5]; }
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
        const int64_t e = e0 + u * kSelBlock;
        if (e >= end) continue;
        const uint32_t x = rb_number(a[u], s[u]), y = rb_number(b[u], d[u]);
        const int k = (x >> 31) == (y >> 31) ? (int)(x >> 31) : 2;
        __builtin_nontemporal_store((uint8_t)k, key + e);
        __builtin_nontemporal_store((int32_t)(x & 0x7FFFFFFFu), tmp_s + e);
        __builtin_nontemporal_store((int32_t)(y & 0x7FFFFFFFu), tmp_d + e);
        n0 += k == 0; n1 += k == 1;
    }
    n0 = es_wave_sum(n0); n1 = es_wave_sum(n1);
    if (lane == 0) { c0[wave] = n0; c1[wave] = n1; }
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t x = 0, y = 0;
        for (int q = 0; q < kSelBlock / 64; ++q) { x += c0[q]; y += c1[q]; }
        bc0[g.tile0 + blockIdx.x] = x; bc1[g.tile0 + blockIdx.x] = y;
    }
}

// exclusive prefix sums of in[0..len) in place, by one workgroup of kBlock threads; returns the total
__device__ uint32_t es_block_scan(uint32_t* p, int64_t len, uint32_t* wsum /* kWaves words of LDS */)
{
    uint32_t carry = 0;
    for (int64_t base = 0; base < len; base += kBlock) {
        const int64_t i = base + threadIdx.x;
        const uint32_t x = i < len ? p[i] : 0u;
        uint32_t all;
        const uint32_t excl = es_block_exclusive(x, wsum, &all);
        if (i < len) p[i] = carry + excl;
        carry += all;
        __syncthreads();
    }
    return carry;
}

// one workgroup per group; totals[2 * group + half]: edges kept
__global__ __launch_bounds__(kBlock) void k_rb_split_scan(const EsGroup* __restrict__ groups, uint32_t* bc0, uint32_t* bc1,
                                                          long long* totals)
{
    __shared__ uint32_t wsum[kWaves];
    const EsGroup g = groups[blockIdx.x];
    const int64_t tiles = (g.m + kSelTile - 1) / kSelTile;
    const uint32_t t0 = es_block_scan(bc0 + g.tile0, tiles, wsum);
    const uint32_t t1 = es_block_scan(bc1 + g.tile0, tiles, wsum);
    if (threadIdx.x == 0) { totals[2 * (int64_t)g.id] = (long long)t0; totals[2 * (int64_t)g.id + 1] = (long long)t1; }
}

// stable: the edges of child 0 (key 0, as k_rb_split_count stored it) keep their order and land where the
// group's edges began, those of child 1 right after them
__global__ __launch_bounds__(kSelBlock) void k_rb_split_scatter(const EsGroup* __restrict__ groups, const int32_t* __restrict__ src,
                                                                const int32_t* __restrict__ dst, const uint8_t* __restrict__ key,
                                                                const uint32_t* __restrict__ bo0, const uint32_t* __restrict__ bo1,
                                                                int32_t* out_src, int32_t* out_dst,
                                                                const long long* __restrict__ totals)
{
    __shared__ uint32_t c0[kSelBlock / 64], c1[kSelBlock / 64];
    const EsGroup g = groups[blockIdx.y];
    if ((int64_t)blockIdx.x * kSelTile >= g.m) return;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t end = g.e_lo + g.m;
    const int64_t e0 = g.e_lo + (int64_t)blockIdx.x * kSelTile + (int64_t)threadIdx.x * kSelPer;
    int32_t s[kSelPer], d[kSelPer];
    int k[kSelPer];
    uint32_t n0 = 0, n1 = 0;
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
        const int64_t e = e0 + u;
        k[u] = 2; s[u] = 0; d[u] = 0;
        if (e < end) {
            s[u] = src[e]; d[u] = dst[e];
            k[u] = key[e];
            n0 += k[u] == 0; n1 += k[u] == 1;
        }
    }
    const uint32_t x0 = es_wave_inclusive(n0) - n0, x1 = es_wave_inclusive(n1) - n1;
    if (lane == 63) { c0[wave] = x0 + n0; c1[wave] = x1 + n1; }
    __syncthreads();
    int64_t p0 = g.e_lo + bo0[g.tile0 + blockIdx.x] + x0;
    int64_t p1 = g.e_lo + totals[2 * (int64_t)g.id] + bo1[g.tile0 + blockIdx.x] + x1;
    for (int q = 0; q < wave; ++q) { p0 += c0[q]; p1 += c1[q]; }
#pragma unroll
    for (int u = 0; u < kSelPer; ++u) {
        if (k[u] == 0) { out_src[p0] = s[u]; out_dst[p0] = d[u]; ++p0; }
        else if (k[u] == 1) { out_src[p1] = s[u]; out_dst[p1] = d[u]; ++p1; }
    }
}

// ---- host side ---------------------------------------------------------------------------------

struct EsProfile {
    std::mutex mu;
    bool on = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> count_events;
    int64_t edges = 0;      // edges handed to the timed launches
} es_prof;

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

inline int grid_for(int64_t items, int block, int64_t cap)
{
    int64_t g = (items + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (int)g;
}

// How a run is laid out.
//   binned  from 4M nodes on (the counts in memory, 8 bytes per node, then far outgrow the L2), if a chunk's pairs take no more
//           room than the estimates (asks take twice the pairs' beside them) and the table of the chunks' bins stays small.  A block is 32,768 nodes where a chunk has 0.34 ends per node or
//           fewer, or half as many (4M nodes: 256 blocks); two of them fit a CU's LDS either way.  Up to 0.72 ends per node its nodes are listed, above that
//           each has its count (14M nodes in chunks of 5 and 10 %: 5.8 and 5.8 ms so, 6.1 and 6.1 listed).  A bin is a block's nodes up to 67M or
//           134M nodes, 4096 bins, several blocks' beyond.
//   tile    8192 edges where that makes 512 tiles, or 4096 (14M nodes in groups, steps of 0.2 to 2M edges: bisection 39.7 -> 38.4 ms) and
//           where the bins' words leave less room in half a CU's LDS.
//   asked   from 2^25 nodes on, or 2^24 and 2^24 ends in a step (100 chunks of 20M nodes: 14.4 ms asked, 13.3 looked up; 10 chunks 7.0 and 7.3; 50 of 27M
//           12.7 and 12.7; 50 of 40M 18.0 and 21.2).
//   classes 8 where a step has 256 tiles or more (14M nodes 9.1 ms, 9.6 with one; 111M 82 and 92), or one: the table is the smaller.
//   blocks  otherwise kBlock * wpw nodes each: one word per wave up to a million nodes (the chip wants some 1024
//           blocks), more words beyond it, so that a block can add up all blocks' counts itself.
//   awpw    the admission's workgroups each add up all blocks' counts: as many words per wave as leave 256 workgroups or
//           fewer, up to kMaxAdmitWords (131,072 nodes per workgroup: more than 256 of them from 33M nodes on) and while the
//           groups' padding stays within their nodes (so with several groups there may be more from fewer nodes on).
struct EsShape {
    int wpw = 1, awpw = 1;
    int cb = 0, classes = 1, tile = 0;     // binned: nodes of a bin (2^cb), classes of tiles, edges of a tile
    uint32_t nb = 0;                       // ... and bins, rounded up
    bool asked = false;                    // binned: labels are looked up in LDS
    int ask_cb = 0;                        // ... nodes of a range (2^ask_cb)
    uint32_t ask_nb = 0;                   // ... and ranges, rounded up
    bool binned = false;
    bool packed = false;                   // binned: the estimates in 8 bytes
    bool sparse = false;                   // binned: a chunk's nodes are so few that a block lists them
    int64_t room = 0;                      // ... and of how many it has room for the counts
    int64_t nodes = 0;                     // room for the state: the nodes and the groups' padding
    uint32_t crowd_limit = 0;              // binned: a bin of more pairs is crowded ...
    int64_t crowd_bins = 0;                // ... and most bins of a chunk that can be
    int64_t bn() const { return (int64_t)kBlock * wpw; }
    int64_t an() const { return (int64_t)kBlock * awpw; }
    int64_t padded(int64_t nv) const { return (nv + an() - 1) / an() * an(); }
};
// of 4096 edges: a step of fewer is binned in tiles of 2048 (bisection of 14M nodes 38.3 -> 36.3 ms, 100 chunks of 5M nodes 4.67 -> 4.33; 488 tiles, 14M nodes,
// 9.6 ms in tiles of 4096 and 10.3 of 2048)
constexpr int64_t kBinFewTiles = 400;
constexpr int kBinWaveWords = 16;
constexpr int64_t kWideSparse = 340, kSparse = 720;
constexpr int64_t kAskMinNodes = 1ll << 25, kAskMinEnds = 1ll << 24;
constexpr int kAskBits = 17;                                 // 32 KB of labels
constexpr int64_t kBinMinNodes = 1ll << 22;
constexpr int64_t kBinMaxChunks = 8192;
constexpr int64_t kCrowdMin = 65535, kCrowdMean = 6, kCrowdMeanLean = 8;     // a crowded bin: more pairs than these, and than so many bins hold on
                                                             // average (their counts then take 1.3 bytes per node at most, or one)
constexpr int64_t kCrowdNodes = 32768;                       // a workgroup of k_es_crowd counts so many at a time
constexpr int64_t kHalfLds = 80 * 1000;
constexpr int kSortLds = 160000;
constexpr unsigned kCrowdGrid = 512;                         // workgroups of k_es_crowd: one per CU at a time
// The forms of a run, each of less memory than the one before it:
//   full     binned, with estimates in 8 bytes beside the doubles and, where they pay, asks
//   lean     binned, the estimates all doubles (in the caller's array if there is one), labels looked up, 1024 bins, one class, few blocks: 17 bytes per
//            node (one with a caller's array) for 26, and a third of the bytes per end where labels are asked for
//   counted  the counts in memory (8 bytes per node, the lean form's pairs up to 16)
enum class EsForm { full, lean, counted };
// n: nodes of the run; groups: most groups side by side; ends: of a chunk's edge ends over all groups
EsShape es_shape(int64_t n, int64_t groups, int64_t ends, int64_t chunks, EsForm form)
{
    EsShape s;
    // padding for every group, but no more than the nodes themselves take (a level of tiny groups goes in batches)
    auto room = [&] {
        const int64_t own = s.padded(n), pad = (groups - 1) * s.an();
        return own + (pad < own ? pad : own);
    };
    auto waves = [&](int wpw) {
        s.wpw = s.awpw = wpw;
        while (s.awpw < kMaxAdmitWords && n > s.an() * 256 && 2 * s.an() * groups <= n) s.awpw *= 2;
    };
    const int64_t per_mille = ends * 1000 / n;                 // ends of a chunk per thousand nodes
    waves(form == EsForm::lean || (per_mille <= kWideSparse && n >= 2 * kBinMinNodes) ? 2 * kBinWaveWords : kBinWaveWords);
    if (form != EsForm::counted && n >= kBinMinNodes && room() < (1ll << 30) && ends <= 4 * n && chunks <= kBinMaxChunks) {
        const bool full = form == EsForm::full;
        s.binned = true;
        s.packed = full;
        s.cb = s.wpw == kBinWaveWords ? 14 : 15;
        while ((room() >> s.cb) >= (full ? kBins : kBlock)) ++s.cb;              // (at most 18; 20)
        auto number = [&](int cb) { return (uint32_t)((room() >> cb) / kBlock + 1) * kBlock; };
        s.nb = number(s.cb);
        s.sparse = per_mille <= kSparse;
        // (two workgroups share a CU; a bin with more nodes of the chunk than there is room for is counted node by node)
        s.room = (kHalfLds - s.bn() / 4) / 6 / 64 * 64;
        s.asked = full && (n >= kAskMinNodes || (2 * n >= kAskMinNodes && ends >= kAskMinEnds));
        if (s.asked) {
            s.ask_cb = s.cb > kAskBits ? s.cb : kAskBits;
            s.ask_nb = number(s.ask_cb);
            s.tile = kAskEdges;
        } else {
            s.tile = ends / 2 >= 512 * kBinTile ? kBinTile : kBinTile / 2;
            if (es_sort_lds(2 * s.tile, 4, s.nb) > kHalfLds) s.tile = kBinTile / 2;
        }
        s.classes = full && ends / 2 / s.tile >= 256 ? 8 : 1;
    } else {
        int wpw = 1;
        while (wpw < kMaxWaveWords && n > (int64_t)kBlock * wpw * 1024) wpw *= 2;
        waves(wpw);
    }
    s.nodes = room();
    if (s.binned) {
        const int64_t nbins = (s.nodes + (1ll << s.cb) - 1) >> s.cb, most = (s.packed ? kCrowdMean : kCrowdMeanLean) * (ends / nbins + 1);
        s.crowd_limit = (uint32_t)(most > kCrowdMin ? most : kCrowdMin);
        s.crowd_bins = ends / ((int64_t)s.crowd_limit + 1);
    }
    return s;
}

// State of a run of up to `nodes` nodes (padding included) in `groups` groups; one allocation.
struct EsMemory {
    EsRun st{};
    EsGroup* groups = nullptr;
    uint32_t* blk_group = nullptr;
    u64* hc = nullptr;
    EsBins bins{}, ranges{};
    uint32_t *pairs = nullptr, *totals = nullptr, *ask_tiles = nullptr;
    uint2* asks = nullptr;
    EsCrowd crowd{};
    size_t bytes = 0;

    void layout(uint8_t* ws, const EsShape& sh, int64_t ngroups, int64_t ends, int64_t chunks, double* est_out)
    {
        const int64_t nodes = sh.nodes;
        size_t off = 0;
        auto take = [&](auto*& p, size_t count) {
            using T = std::remove_reference_t<decltype(*p)>;
            p = ws ? reinterpret_cast<T*>(ws + off) : nullptr;
            off += align256(count * sizeof(T));
        };
        const size_t blocks = (size_t)(nodes / sh.bn()), words = (size_t)(nodes / 64);
        take(st.flags, 2);                       // (S follows: one read-back brings both)
        take(st.S, (size_t)ngroups * 4);
        take(groups, (size_t)ngroups);
        take(blk_group, blocks);
        take(st.Lw, (size_t)(nodes / 32));
        if (est_out && !sh.packed) st.est = (double2*)est_out;
        else take(st.est, (size_t)nodes);
        take(st.mark, words); take(st.mv0, words); take(st.mv1, words); take(st.nw, words);
        take(st.bs, blocks);
        if (sh.binned) {
            bins.nb = sh.nb;
            bins.cb = sh.cb;
            bins.classes = sh.classes;
            take(bins.ends, (size_t)chunks * sh.nb * bins.classes);
            take(pairs, (size_t)ends);
            if (sh.asked) {
                ranges.nb = sh.ask_nb;
                ranges.cb = sh.ask_cb;
                ranges.classes = sh.classes;
                take(ranges.ends, (size_t)chunks * sh.ask_nb * sh.classes);
                take(totals, (size_t)chunks);
                take(ask_tiles, (size_t)chunks * (sh.ask_nb + 1));
                take(asks, (size_t)ends);
            }
            if (sh.packed) take(st.packed, (size_t)nodes);
            if (sh.packed) take(st.wide, blocks);
            take(crowd.place, (size_t)chunks * sh.nb);
            take(crowd.bins, (size_t)chunks);
            take(crowd.hc, (size_t)sh.crowd_bins << sh.cb);
            take(crowd.seen, ((size_t)sh.crowd_bins << sh.cb) / 32);
            crowd.limit = sh.crowd_limit;
        } else {
            take(hc, (size_t)nodes);
        }
        st.groups = groups;
        st.blk_group = blk_group;
        st.wpw = sh.wpw;
        st.awpw = sh.awpw;
        bytes = off;
    }
};

void es_fill(hipStream_t stream, void* p, size_t bytes, u64 value)
{
    const size_t count = bytes / 8;
    if (count)
        hipLaunchKernelGGL(k_es_fill64, dim3(grid_for((int64_t)count, 256, 16384)), dim3(256), 0, stream, (u64*)p, count, value);
}

// One run: everything from the cleared state to the last chunk's spill is enqueued.  groups_host: its groups, in the
// order of their nodes (also at mem.groups on the device, with mem.blk_group filled).  check(): called once the first chunk's seeds are
// counted and flags[] is complete, before anything uses the labels; its answer other than GREM_OK ends the run.
// check_ends (one group): flags[] and the endpoints' range are this call's business too, and the seeds' sizes check()'s.  check() waits for the
// stream where the run is binned.  est_nodes: entries of est to clear.  *par_out: which copy of the sizes is the final one.
template <typename Check>
int es_run(hipStream_t stream, EsMemory& mem, const EsShape& sh, const std::vector<EsGroup>& groups, int64_t nodes, int64_t est_nodes,
           const int32_t* src, const int32_t* dst, const int32_t* seed, int32_t mode, bool check_ends, Check&& check, int* par_out)
{
    EsRun& st = mem.st;
    st.ngroups = (uint32_t)groups.size();
    const unsigned ng = (unsigned)groups.size(), blocks = (unsigned)(nodes / sh.bn()), ablocks = (unsigned)(nodes / sh.an());
    int64_t most = 1, chunks = 1;                              // most edges in a chunk of one group; most chunks
    for (const EsGroup& g : groups) {
        if (g.m == 0) continue;
        if (g.c_size < g.m ? g.c_size > most : g.m > most) most = g.c_size < g.m ? g.c_size : g.m;
        const int64_t c = (g.m + g.c_size - 1) / g.c_size;
        if (c > chunks) chunks = c;
    }
    // (a step of few tiles is a tile's latency: smaller ones, several to a CU)
    int64_t step = 0;
    for (const EsGroup& g : groups) step += g.c_size < g.m ? g.c_size : g.m;
    const int tile = sh.binned && !sh.asked && sh.tile == kBinTile / 2 && step < kBinFewTiles * sh.tile ? sh.tile / 2 : sh.tile;
    if (ng == 1) st.only = groups[0];
    EsClears clears;
    if (check_ends) clears.add(st.flags, 8);
    clears.add(st.S, align256((size_t)ng * 32));
    clears.add(st.Lw, (size_t)nodes / 4);
    clears.add(st.mark, (size_t)nodes / 8);
    if (sh.binned) {
        clears.add(mem.bins.ends, align256((size_t)chunks * sh.nb * mem.bins.classes * 4));
        if (sh.asked) clears.add(mem.ranges.ends, align256((size_t)chunks * sh.ask_nb * sh.classes * 4));
        if (sh.packed) {
            clears.add(st.packed, (size_t)nodes * 8);
            clears.add(st.wide, align256((size_t)blocks * 4));
        }
    } else {
        clears.add(mem.hc, (size_t)nodes * 8);
    }
    if (!sh.packed) clears.add(st.est, (size_t)est_nodes * 16);
    hipLaunchKernelGGL(k_es_clear, dim3(grid_for((sh.packed ? 8 : sh.binned ? 16 : 24) * nodes / 64, 256, 16384)), dim3(256), 0, stream, clears);
    auto round = [&](int64_t grid) { return (grid + sh.classes - 1) / sh.classes * sh.classes; };
    std::vector<uint32_t> crowded;                             // per chunk: its crowded bins
    if (sh.binned) {
        // (workgroups of several tiles each: a workgroup's counts are added to the table once)
        // (asked: 128 KB of counts each; with 256 workgroups a chunk 4.4 ms at 111M nodes and 100 chunks, with 48 3.7)
        const int64_t per = sh.asked ? tile : kBinTile, parts = round(grid_for((most + per - 1) / per, 4, sh.asked ? std::min<int64_t>(std::max<int64_t>(4096 / (chunks * ng), 32), 256) : 256));
        const size_t hist_lds = (size_t)sh.nb * 4 * (sh.asked ? sh.classes : 1);
        if (hipFuncSetAttribute((const void*)k_es_hist, hipFuncAttributeMaxDynamicSharedMemorySize, kBins * 4 * 8) != hipSuccess) return GREM_ERR_HIP;
        hipLaunchKernelGGL(k_es_hist, dim3((unsigned)parts, ng, (unsigned)chunks), dim3(kBlock), hist_lds, stream, src, dst, st, mem.bins, mem.ranges, tile);
        hipLaunchKernelGGL(k_es_hist_scan, dim3((unsigned)chunks), dim3(kBlock), 0, stream, mem.bins, mem.crowd, mem.totals);
        if (sh.asked) {
            hipLaunchKernelGGL(k_es_hist_scan, dim3((unsigned)chunks), dim3(kBlock), 0, stream, mem.ranges, EsCrowd{}, (uint32_t*)nullptr);
            hipLaunchKernelGGL(k_es_ask_tiles, dim3((unsigned)chunks), dim3(kBlock), 0, stream, mem.ranges, (const uint32_t*)mem.totals, mem.ask_tiles);
        }
        crowded.resize((size_t)chunks);
        if (hipMemcpyAsync(crowded.data(), mem.crowd.bins, (size_t)chunks * 4, hipMemcpyDeviceToHost, stream) != hipSuccess) return GREM_ERR_HIP;
    }
    // (a binned run has checked the endpoints where it counted the bins)
    if (check_ends && !sh.binned)
        hipLaunchKernelGGL(k_es_check_mark, dim3((unsigned)grid_for(groups[0].m, kCountBlock, 8192)), dim3(kCountBlock), 0, stream, src, dst, st);
    else
        hipLaunchKernelGGL(k_es_mark, dim3((unsigned)grid_for(most, kCountBlock, 8192), ng), dim3(kCountBlock), 0, stream, src, dst, st);
    hipLaunchKernelGGL(k_es_seed, dim3(blocks), dim3(kBlock), 0, stream, st, seed);
    if (!check_ends) hipLaunchKernelGGL(k_es_seed_sizes, dim3((ng + 255) / 256), dim3(256), 0, stream, st);
    const int rc = check();
    if (rc != GREM_OK) return rc;
    for (int64_t i = 0; i < (int64_t)crowded.size(); ++i)
        if (crowded[(size_t)i]) {
            es_fill(stream, mem.crowd.hc, ((size_t)sh.crowd_bins << sh.cb) * 8, 0ull);
            es_fill(stream, mem.crowd.seen, ((size_t)sh.crowd_bins << sh.cb) / 8, 0ull);
            break;
        }
    const int64_t crowd_bn = sh.bn() < kCrowdNodes ? sh.bn() : kCrowdNodes;
    const size_t crowd_lds = (size_t)crowd_bn * 4 + (size_t)crowd_bn / 8, bins_lds = es_bins_lds(sh.bn(), sh.room);
    const auto bin = tile == 8192 ? k_es_bin8 : tile == 4096 ? k_es_bin4 : k_es_bin;
    // (always what any run may need: the limit is the process's, and other threads' runs are of other sizes)
    if (sh.binned &&
        (hipFuncSetAttribute((const void*)k_es_ask, hipFuncAttributeMaxDynamicSharedMemorySize, kSortLds) != hipSuccess ||
         hipFuncSetAttribute((const void*)k_es_answer, hipFuncAttributeMaxDynamicSharedMemorySize, kSortLds) != hipSuccess ||
         hipFuncSetAttribute((const void*)bin, hipFuncAttributeMaxDynamicSharedMemorySize, kSortLds) != hipSuccess ||
         hipFuncSetAttribute((const void*)k_es_crowd, hipFuncAttributeMaxDynamicSharedMemorySize, (int)(kCrowdNodes * 4 + kCrowdNodes / 8)) != hipSuccess ||
         hipFuncSetAttribute((const void*)k_es_score_bins, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kHalfLds) != hipSuccess))
        return GREM_ERR_HIP;
    bool profile;
    { std::lock_guard<std::mutex> lock(es_prof.mu); profile = es_prof.on; }
    const int fixed = mode == GREM_EDGE_FIXED ? 1 : 0;
    int par = 0;
    for (int64_t i = 0; i < chunks; ++i) {
        hipEvent_t e0 = nullptr, e1 = nullptr;
        if (profile) {
            // timing only: no system-scope fence when the events complete
            if (hipEventCreateWithFlags(&e0, hipEventDisableSystemFence) != hipSuccess ||
                hipEventCreateWithFlags(&e1, hipEventDisableSystemFence) != hipSuccess)
                return GREM_ERR_HIP;
            (void)hipEventRecord(e0, stream);
        }
        auto timed = [&] {                         // cnt_nbrs is done: binned, with the scoring that it is part of
            if (!profile) return;
            (void)hipEventRecord(e1, stream);
            std::lock_guard<std::mutex> lock(es_prof.mu);
            es_prof.count_events.emplace_back(e0, e1);
            for (const EsGroup& g : groups)
                if (i * g.c_size < g.m) es_prof.edges += g.m - i * g.c_size < g.c_size ? g.m - i * g.c_size : g.c_size;
        };
        if (sh.asked) {
            // k_es_ask: two workgroups per CU; k_es_answer: one
            const int64_t asks = round(std::min((most + tile - 1) / tile, std::max<int64_t>(512 / ng, 1)));
            const int64_t answers = round(std::min<int64_t>((int64_t)ng * ((2 * most + kAskTile - 1) / kAskTile) + sh.ask_nb, 256));
            hipLaunchKernelGGL(k_es_ask, dim3((unsigned)asks, ng), dim3(kBlock), es_sort_lds((size_t)kAskEdges * 2, 8, sh.ask_nb), stream, src, dst, st, i,
                               mem.ranges, mem.asks);
            hipLaunchKernelGGL(k_es_answer, dim3((unsigned)answers), dim3(kBlock), es_sort_lds(kAskTile, 4, sh.nb) + ((size_t)1 << sh.ask_cb) / 4, stream,
                               st, i, mem.ranges, (const uint32_t*)mem.ask_tiles, (const uint2*)mem.asks, mem.bins, (uint32_t)nodes, mem.pairs);
        } else if (sh.binned)
            hipLaunchKernelGGL(bin, dim3((unsigned)round((most + tile - 1) / tile), ng), dim3(kBlock), es_sort_lds((size_t)tile * 2, 4, sh.nb), stream, src, dst, st, i, mem.bins, mem.pairs);
        else
            hipLaunchKernelGGL(k_es_count, dim3((unsigned)grid_for(most, kCountBlock, 1 << 20), ng), dim3(kCountBlock), 0, stream, src, dst, st,
                               i, mem.hc);
        if (!sh.binned) timed();
        const int first = i == 0 ? 1 : 0;
        if (sh.binned && crowded[(size_t)i])
            hipLaunchKernelGGL(k_es_crowd, dim3(kCrowdGrid), dim3(kBlock), crowd_lds, stream, i, mem.bins, (uint32_t)crowd_bn, (uint32_t)(nodes / crowd_bn),
                               (const uint32_t*)mem.pairs, mem.crowd);
        if (sh.binned)
            hipLaunchKernelGGL(k_es_score_bins, dim3((blocks + 7) / 8 * 8), dim3(kBlock), bins_lds, stream, st, par, first, fixed, i,
                               mem.bins, blocks, (uint32_t)sh.room, sh.sparse ? 1 : 0, (const uint32_t*)mem.pairs, mem.crowd);
        else
            hipLaunchKernelGGL(k_es_score, dim3(blocks), dim3(kBlock), 0, stream, st, par, first, fixed, mem.hc);
        if (sh.binned) timed();
        if (first) continue;
        if (sh.awpw <= 64) hipLaunchKernelGGL(k_es_admit<1>, dim3(ablocks), dim3(kBlock), 0, stream, st, par);
        else hipLaunchKernelGGL(k_es_admit<2>, dim3(ablocks), dim3(kBlock), 0, stream, st, par);
        par ^= 1;
    }
    *par_out = par;
    return hipGetLastError() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
}

// The entry points' bodies.  ws: the call's scratch memory while it holds any; the caller gives it back if a body throws.
int es_bipartition(const int32_t* src, const int32_t* dst, int64_t m, int64_t n, int64_t c_size, int64_t P, const int32_t* seed_parts,
                   int32_t mode, int32_t* parts_out, int64_t* sizes_out, double* nbr_counts_out, void* stream_, uint8_t*& ws)
{
    if (!src || !dst || !seed_parts || !parts_out || m < 1 || n < 1 || n > INT32_MAX || c_size < 1 ||
        P < 1 || 2 * P < n || (mode != GREM_EDGE_REFINE && mode != GREM_EDGE_FIXED))
        return GREM_ERR_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    if (c_size > m) c_size = m;
    const int64_t chunks = (m + c_size - 1) / c_size, ends = 2 * c_size;
    EsShape sh;
    EsMemory mem;
    for (const EsForm form : {EsForm::full, EsForm::lean, EsForm::counted}) {
        sh = es_shape(n, 1, ends, chunks, form);
        mem.layout(nullptr, sh, 1, ends, chunks, nbr_counts_out);
        if (hipMallocAsync((void**)&ws, mem.bytes, stream) == hipSuccess) break;
        (void)hipGetLastError();
        ws = nullptr;
        if (!sh.binned) return GREM_ERR_NOMEM;
    }
    const int64_t nodes = sh.nodes;
    mem.layout(ws, sh, 1, ends, chunks, nbr_counts_out);
    std::vector<EsGroup> groups(1);
    groups[0] = EsGroup{0, m, c_size, (long long)P, 0, 0u, (uint32_t)n, 0u, (uint32_t)(nodes / sh.bn()), 0u, 0u};
    int par = 0;
    // the range check must be known before any kernel indexes with the endpoints
    int rc = es_run(stream, mem, sh, groups, nodes, n, src, dst, seed_parts, mode, true, [&]() -> int {
        struct { uint32_t flags[64]; u64 S[2]; } back{};
        static_assert(sizeof(back) == 256 + 16, "as EsMemory lays them out");
        if (hipMemcpyAsync(&back, mem.st.flags, sizeof(back), hipMemcpyDeviceToHost, stream) != hipSuccess ||
            hipStreamSynchronize(stream) != hipSuccess)
            return GREM_ERR_HIP;
        const bool full = (long long)back.S[0] > P || (long long)back.S[1] > P;
        return back.flags[0] ? GREM_ERR_ARG : back.flags[1] || full ? GREM_ERR_SEED : GREM_OK;
    }, &par);
    if (rc == GREM_OK) {
        hipLaunchKernelGGL(k_es_expand, dim3(grid_for(n, 256, 16384)), dim3(256), 0, stream, n, (const u64*)mem.st.Lw, parts_out,
                           (const u64*)(mem.st.S + 2 * par), sizes_out);
        if (sh.packed && nbr_counts_out)
            hipLaunchKernelGGL(k_es_expand_packed, dim3(grid_for(n, 256, 16384)), dim3(256), 0, stream, n, mem.st, (double2*)nbr_counts_out);
        if (hipGetLastError() != hipSuccess) rc = GREM_ERR_HIP;
    } else {
        (void)hipGetLastError();
    }
    if (hipFreeAsync(ws, stream) != hipSuccess && rc == GREM_OK) rc = GREM_ERR_HIP;
    return rc;
}

int es_bisection(const int32_t* src, const int32_t* dst, int64_t m, int64_t n, int32_t levels, int64_t chunks, double balance_slack,
                 const int32_t* seed_bits, int32_t mode, int32_t* labels_out, void* stream_, uint8_t*& ws)
{
    if (!src || !dst || !seed_bits || !labels_out || m < 1 || n < 1 || n > INT32_MAX || levels < 1 || levels > 20 ||
        chunks < 1 || !(balance_slack >= 1.0) || (mode != GREM_EDGE_REFINE && mode != GREM_EDGE_FIXED))
        return GREM_ERR_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    // The groups of a level run side by side, as many as the state has room for (a level of very many, tiny,
    // groups takes several batches).
    const int64_t c_max = chunks < m ? chunks : m;             // chunks a group can have
    constexpr int64_t kMaxBatch = 1024;
    const int64_t most_groups = (int64_t)1 << (levels - 1);
    const int64_t ends = 2 * ((m + c_max - 1) / c_max + kMaxBatch);         // of one step: each group's chunk is rounded up
    EsShape sh;
    EsMemory mem;
    const int64_t sel_blocks = (m + kSelTile - 1) / kSelTile + kMaxBatch;
    size_t off = 0;
    auto carve = [&](size_t bytes) { const size_t at = off; off += align256(bytes); return at; };
    const size_t o_totals = carve((size_t)most_groups * 24);     // per group: edges kept per half, nodes in half 0
    size_t o_gof[2], o_seed[2];                        // two generations of the groups' node lists
    for (int i = 0; i < 2; ++i) { o_gof[i] = carve((size_t)n * 4); o_seed[i] = carve((size_t)n * 4); }
    const size_t o_bc0 = carve((size_t)sel_blocks * 4), o_bc1 = carve((size_t)sel_blocks * 4);
    const size_t o_tmps = carve((size_t)m * 4), o_tmpd = carve((size_t)m * 4), o_key = carve((size_t)m);
    size_t o_lev[4];                                   // two generations of the grouped edge list
    for (int i = 0; i < 4; ++i) o_lev[i] = carve((size_t)m * 4);
    size_t o_halves = off, o_run = off;                // sized by the run's nodes; its state is the last piece
    for (const EsForm form : {EsForm::full, EsForm::lean, EsForm::counted}) {
        sh = es_shape(n, most_groups < kMaxBatch ? most_groups : kMaxBatch, ends, c_max, form);
        o_run = o_halves + align256((size_t)sh.nodes / 4);
        mem.layout(nullptr, sh, kMaxBatch, ends, c_max, nullptr);
        if (hipMallocAsync((void**)&ws, o_run + mem.bytes, stream) == hipSuccess) break;
        (void)hipGetLastError();
        ws = nullptr;
        if (!sh.binned) return GREM_ERR_NOMEM;
    }
    mem.layout(ws + o_run, sh, kMaxBatch, ends, c_max, nullptr);
    auto fail = [&](int code) { (void)hipGetLastError(); (void)hipStreamSynchronize(stream); (void)hipFreeAsync(ws, stream); return code; };
    long long* totals = (long long*)(ws + o_totals);
    long long* nodes0 = totals + 2 * most_groups;
    u64* halves = (u64*)(ws + o_halves);
    uint32_t *bc0 = (uint32_t*)(ws + o_bc0), *bc1 = (uint32_t*)(ws + o_bc1);
    int32_t *tmp_s = (int32_t*)(ws + o_tmps), *tmp_d = (int32_t*)(ws + o_tmpd);
    uint8_t* key = ws + o_key;

    es_fill(stream, mem.st.flags, 8, 0ull);
    hipLaunchKernelGGL(k_es_check, dim3(grid_for(m, 256, 8192)), dim3(256), 0, stream, src, dst, m, (uint32_t)n, mem.st.flags);
    uint32_t flags[2] = {0, 0};
    auto read_flags = [&]() {
        return hipMemcpyAsync(flags, mem.st.flags, sizeof(flags), hipMemcpyDeviceToHost, stream) == hipSuccess &&
               hipStreamSynchronize(stream) == hipSuccess;
    };
    if (!read_flags()) return fail(GREM_ERR_HIP);
    if (flags[0]) return fail(GREM_ERR_ARG);

    // level 0: one group, everyone, numbered by id; its edges and seed bits are the inputs themselves
    struct Part { int64_t e_lo, m, v_lo, nv; };
    std::vector<Part> parts{{0, m, 0, n}}, next;
    const int32_t *cur_s = src, *cur_d = dst;
    const int32_t *cur_gof = nullptr, *cur_seed = seed_bits;
    std::vector<long long> host;
    for (int32_t level = 0; level < levels; ++level) {
        const bool last = level + 1 == levels;
        int32_t* out_s = (int32_t*)(ws + o_lev[(level & 1) * 2]);
        int32_t* out_d = (int32_t*)(ws + o_lev[(level & 1) * 2 + 1]);
        int32_t* gof_next = (int32_t*)(ws + o_gof[level & 1]);
        int32_t* seed_next = (int32_t*)(ws + o_seed[level & 1]);
        const size_t count = parts.size();
        const int32_t* next_bits = last ? seed_bits : seed_bits + (size_t)(level + 1) * (size_t)n;
        es_fill(stream, ws + o_totals, (size_t)most_groups * 24, 0ull);
        std::vector<std::vector<EsGroup>> batches;       // (copied to the device: kept until the level's read-back)
        for (size_t g0 = 0; g0 < count;) {
            // the next batch: groups that have nodes, as many as fit
            batches.emplace_back();
            std::vector<EsGroup>& groups = batches.back();
            int64_t nodes = 0, tiles = 0;
            size_t g1 = g0;
            for (; g1 < count && (int64_t)groups.size() < kMaxBatch; ++g1) {
                const Part& p = parts[g1];
                if (p.nv == 0) continue;
                const int64_t padded = sh.padded(p.nv);
                if (nodes + padded > sh.nodes) break;
                groups.push_back(EsGroup{p.e_lo, p.m, p.m > 0 ? (p.m + chunks - 1) / chunks : 1,
                                         (long long)grem_capacity(p.nv, 2, balance_slack), p.v_lo, (uint32_t)nodes, (uint32_t)p.nv,
                                         (uint32_t)(nodes / sh.bn()), (uint32_t)(padded / sh.bn()), (uint32_t)tiles, (uint32_t)g1});
                nodes += padded;
                tiles += (p.m + kSelTile - 1) / kSelTile;
            }
            g0 = g1;
            if (groups.empty()) continue;
            const unsigned ng = (unsigned)groups.size(), blocks = (unsigned)(nodes / sh.bn());
            if (hipMemcpyAsync(mem.groups, groups.data(), groups.size() * sizeof(EsGroup), hipMemcpyHostToDevice, stream) != hipSuccess)
                return fail(GREM_ERR_HIP);
            hipLaunchKernelGGL(k_es_blk_groups, dim3(ng), dim3(256), 0, stream, (const EsGroup*)mem.groups, mem.blk_group);
            int par = 0;
            // a bad seed is looked for at the end of the level: until then it only leaves a node without a label
            const int rc = es_run(stream, mem, sh, groups, nodes, nodes, cur_s, cur_d, cur_seed, mode, false, [&] {
                return sh.binned && hipStreamSynchronize(stream) != hipSuccess ? GREM_ERR_HIP : GREM_OK;
            }, &par);
            if (rc != GREM_OK) return fail(rc);
            hipLaunchKernelGGL(k_rb_count, dim3(blocks), dim3(kBlock), 0, stream, mem.st);
            hipLaunchKernelGGL(k_rb_children, dim3(blocks), dim3(kBlock), 0, stream, mem.st, par, cur_gof, next_bits, halves, gof_next,
                               seed_next, last ? labels_out : (int32_t*)nullptr, nodes0);
            // the groups' edges that stay inside a half, in the halves' numbers, for the next level
            int64_t most = 0;
            for (const EsGroup& g : groups) if (g.m > most) most = g.m;
            if (!last && most > 0) {
                const dim3 grid((unsigned)((most + kSelTile - 1) / kSelTile), ng);
                hipLaunchKernelGGL(k_rb_split_count, grid, dim3(kSelBlock), 0, stream, (const EsGroup*)mem.groups, cur_s, cur_d,
                                   (const u64*)halves, key, tmp_s, tmp_d, bc0, bc1);
                hipLaunchKernelGGL(k_rb_split_scan, dim3(ng), dim3(kBlock), 0, stream, (const EsGroup*)mem.groups, bc0, bc1, totals);
                hipLaunchKernelGGL(k_rb_split_scatter, grid, dim3(kSelBlock), 0, stream, (const EsGroup*)mem.groups, (const int32_t*)tmp_s,
                                   (const int32_t*)tmp_d, (const uint8_t*)key, (const uint32_t*)bc0, (const uint32_t*)bc1, out_s, out_d,
                                   (const long long*)totals);
            }
        }
        // one read-back per level: the children's sizes, and whether every seed was sound
        host.assign((size_t)most_groups * 3, 0);
        if (hipMemcpyAsync(host.data(), ws + o_totals, (size_t)most_groups * 24, hipMemcpyDeviceToHost, stream) != hipSuccess || !read_flags())
            return fail(GREM_ERR_HIP);
        if (flags[1]) return fail(GREM_ERR_SEED);
        next.clear();
        for (size_t g = 0; g < count && !last; ++g) {
            const Part& p = parts[g];
            const int64_t t0 = host[2 * g], t1 = host[2 * g + 1], c0 = host[(size_t)2 * most_groups + g];
            next.push_back({p.e_lo, t0, p.v_lo, c0});
            next.push_back({p.e_lo + t0, t1, p.v_lo + c0, p.nv - c0});
        }
        parts.swap(next);
        cur_s = out_s; cur_d = out_d;
        cur_gof = gof_next; cur_seed = seed_next;
    }
    int rc = hipGetLastError() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
    if (hipFreeAsync(ws, stream) != hipSuccess) rc = GREM_ERR_HIP;
    return rc;
}

// nothing throws at the C interface: host memory that cannot be had is an error like any other
template <typename F>
int es_guarded(void* stream_, F&& f)
{
    hipStream_t stream = (hipStream_t)stream_;
    uint8_t* ws = nullptr;
    try {
        return f(ws);
    } catch (const std::bad_alloc&) {
        (void)hipStreamSynchronize(stream);
        if (ws) (void)hipFreeAsync(ws, stream);
        return GREM_ERR_NOMEM;
    }
}

}  // namespace

extern "C" {

int grem_edge_stream_bipartition(const int32_t* src, const int32_t* dst, int64_t m, int64_t n,
                                 int64_t c_size, int64_t P, const int32_t* seed_parts, int32_t mode,
                                 int32_t* parts_out, int64_t* sizes_out, double* nbr_counts_out,
                                 void* stream_)
{
    return es_guarded(stream_, [&](uint8_t*& ws) {
        return es_bipartition(src, dst, m, n, c_size, P, seed_parts, mode, parts_out, sizes_out, nbr_counts_out, stream_, ws);
    });
}

int grem_recursive_bisection(const int32_t* src, const int32_t* dst, int64_t m, int64_t n, int32_t levels,
                             int64_t chunks, double balance_slack, const int32_t* seed_bits, int32_t mode,
                             int32_t* labels_out, void* stream_)
{
    return es_guarded(stream_, [&](uint8_t*& ws) {
        return es_bisection(src, dst, m, n, levels, chunks, balance_slack, seed_bits, mode, labels_out, stream_, ws);
    });
}

int grem_edge_list_cut(const int32_t* src, const int32_t* dst, int64_t m, const int32_t* parts,
                       int64_t* cut_out, void* stream_)
{
    if (!src || !dst || !parts || !cut_out || m < 0) return GREM_ERR_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    hipLaunchKernelGGL(k_es_fill64, dim3(1), dim3(256), 0, stream, (u64*)cut_out, (size_t)1, 0ull);
    if (m > 0)
        hipLaunchKernelGGL(k_es_cut, dim3(grid_for(m, 256, 8192)), dim3(256), 0, stream, src, dst, m, parts, (u64*)cut_out);
    return hipGetLastError() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
}

int grem_edge_stream_profile_enable(int32_t on)
{
    std::lock_guard<std::mutex> lock(es_prof.mu);
    es_prof.on = on != 0;
    return GREM_OK;
}

int grem_edge_stream_profile_read(double* count_ms, int64_t* launches, int64_t* edges)
{
    std::lock_guard<std::mutex> lock(es_prof.mu);
    double total = 0.0;
    int rc = GREM_OK;
    for (auto& ev : es_prof.count_events) {
        float ms = 0.f;
        if (hipEventSynchronize(ev.second) != hipSuccess || hipEventElapsedTime(&ms, ev.first, ev.second) != hipSuccess)
            rc = GREM_ERR_HIP;
        total += ms;
        (void)hipEventDestroy(ev.first);
        (void)hipEventDestroy(ev.second);
    }
    if (count_ms) *count_ms = total;
    if (launches) *launches = (int64_t)es_prof.count_events.size();
    if (edges) *edges = es_prof.edges;
    es_prof.count_events.clear();
    es_prof.edges = 0;
    return rc;
}

}  // extern "C"
