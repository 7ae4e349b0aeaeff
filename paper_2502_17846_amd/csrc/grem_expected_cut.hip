// Expected number of edge cuts of fixed greedy decisions made from a fraction x of the edges, for gfx950
// (Armada paper, Sec. 4.2, Eq. (1)): for a two-way labelling, node i has k_i labelled neighbours, k0_i of
// them in the partition that holds more; with d_i = floor(k_i x + 0.5) of its edges in hand the greedy
// decision is wrong with probability q_i = Pr(K < d_i / 2), K ~ Hypergeometric(k_i, k0_i, d_i), and
//   E[C] = sum_i (k_i - k0_i) (1 - q_i) + k0_i q_i.
// Refinement over two chunks is the same expression at 2x (Sec. 4.2, "The Benefit of Refinement").
//
// Nodes are taken in tiles of 256: a workgroup walks a tile's CSR entries edge-parallel and counts the labels per
// node, then every thread sums the tail of one node's distribution term by term: in the log domain (first term from
// lgamma, the following ones by the ratio of consecutive probabilities), or, for a node with few draws, as plain
// products of ratios.  A tile of very many entries (ids in order of degree put the longest rows side by side) is
// counted in pieces by all workgroups.  Every 64 nodes have a sum of their own and those are added in a fixed
// order, so the result is reproducible whichever workgroup counted what.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>
#include <type_traits>

#include "grem.h"

// The sums, the packed labels and the split tiles' counts of the entry point that allocates nothing
// (grem_expected_cut_noalloc).  One copy per GPU, held until the process ends; host code reaches it only through the address
// hipGetSymbolAddress returns for the current device, never through this name.
constexpr int64_t kXcStaticBytes = 1 << 22;
constexpr int64_t kXcStaticMaxN = 4194304;         // their labels, two bits each, take 1 MiB of it
static __device__ __align__(256) double scratch[kXcStaticBytes / sizeof(double)];

namespace {

constexpr int kXcBlock = 256;

// log of C(k0, j) C(r, d - j) / C(k, d), the nine lgamma's one after the other (inlined nine times they take 250
// registers)
__device__ __forceinline__ double xc_log_pmf(double k0, double r, double k, double d, double j)
{
    double sum = 0.0, part = 0.0;
#pragma unroll 1
    for (int i = 0; i < 9; ++i) {
        const int which = i / 3, term = i - 3 * which;             // choose(a, b) = lg(a+1) - lg(b+1) - lg(a-b+1)
        const double a = which == 0 ? k0 : which == 1 ? r : k;
        const double b = which == 0 ? j : which == 1 ? d - j : d;
        const double g = lgamma((term == 0 ? a : term == 1 ? b : a - b) + 1.0);
        part = term == 0 ? g : part - g;
        if (term == 2) sum = which == 0 ? part : which == 1 ? sum + part : sum - part;
    }
    return sum;
}

constexpr long long kXcFewDraws = 256;     // up to this many draws the tail is summed without logarithms

// One node's terms of Eq. (1) from its two neighbour counts: *ec = (k - k0)(1 - q) + k0 q, *base = k - k0
// (both left as they are for a node without labelled neighbours).
__device__ __forceinline__ void xc_node_terms(uint32_t c0, uint32_t c1, double x, double* ec_out, double* base_out)
{
    const long long k = (long long)c0 + c1, k0 = c0 > c1 ? c0 : c1, r = k - k0;
    if (k <= 0) return;
    long long d = (long long)floor((double)k * x + 0.5);
    if (d > k) d = k;
    if (d < 0) d = 0;
    // q = sum of pmf(j) over the support with 2j < d
    const long long jlo = d - r > 0 ? d - r : 0;
    long long jhi = (d + 1) / 2 - 1;
    if (jhi > k0) jhi = k0;
    double q = 0.0;
    if (jhi >= jlo && jlo == 0 && d <= kXcFewDraws) {
        // few draws, all of which the minority could fill (the usual node at small x): pmf(0) = C(r, d) / C(k, d)
        // as a product of d ratios, the following terms by the ratio of consecutive probabilities -- no
        // lgamma, log or exp.  pmf(0) is about (r/k)^d: whenever the tail is not negligible (at least
        // 1e-20, which takes (r/k)^(d/2) 2^d >= 1e-20) it stays above 1e-40 / 4^d, far from the smallest
        // double for d <= 256; where pmf(0) does underflow, the tail is zero to every digit that counts.
        // (the factors are small integers held in doubles and stepped by one: exact, and no 64-bit
        // integer-to-double conversions in the loops)
        double p = 1.0, rr = (double)r, kk = (double)k;
        for (int i = 0; i < (int)d; ++i) { p *= rr / kk; rr -= 1.0; kk -= 1.0; }
        q = p;
        double a = (double)k0, b = (double)d, c = 1.0, e = (double)(r - d + 1);
        for (int j = 0; j < (int)jhi; ++j) {
            p *= (a * b) / (c * e);
            q += p;
            a -= 1.0; b -= 1.0; c += 1.0; e += 1.0;
        }
        if (q > 1.0) q = 1.0;
    } else if (jhi >= jlo) {
        double logp = xc_log_pmf((double)k0, (double)r, (double)k, (double)d, (double)jlo);
        q = exp(logp);
        for (long long j = jlo; j < jhi; ++j) {
            // pmf(j+1) / pmf(j)
            logp += log((double)(k0 - j)) + log((double)(d - j)) - log((double)(j + 1)) - log((double)(r - d + j + 1));
            q += exp(logp);
        }
        if (q > 1.0) q = 1.0;
    }
    *ec_out = (double)r * (1.0 - q) + (double)k0 * q;
    *base_out = (double)r;
}

// sums of a wave's terms -> *sum_ec, *sum_base
__device__ __forceinline__ void xc_wave_sums(double ec, double base, double* sum_ec, double* sum_base)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { ec += __shfl_down(ec, o); base += __shfl_down(base, o); }
    if ((threadIdx.x & 63) == 0) { *sum_ec = ec; *sum_base = base; }
}

// Small graphs, whose labels the caches hold as they are: sixteen lanes per node count its row's labels and one of
// them sums the tail; one launch and the total.
constexpr int kXcGroup = 16;                       // lanes that share one node's row
constexpr int kXcRows = kXcBlock / kXcGroup;       // nodes per workgroup
template <typename RowT>
__global__ __launch_bounds__(kXcBlock) void k_xc_small(const RowT* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                       int64_t n, const int32_t* __restrict__ labels, double x,
                                                       double* sum_ec, double* sum_base)
{
    const int sub = threadIdx.x & (kXcGroup - 1);
    const int64_t v = (int64_t)blockIdx.x * kXcRows + threadIdx.x / kXcGroup;
    double ec = 0.0, base = 0.0;
    uint32_t c0 = 0, c1 = 0;
    if (v < n) {
        const int64_t end = (int64_t)rowptr[v + 1];
        constexpr int kTurn = 4;                   // entries in flight per lane
        for (int64_t e = (int64_t)rowptr[v] + sub; e < end; e += kTurn * kXcGroup) {
            int32_t c[kTurn], l[kTurn];
#pragma unroll
            for (int u = 0; u < kTurn; ++u) c[u] = e + u * kXcGroup < end ? colidx[e + u * kXcGroup] : -1;
#pragma unroll
            for (int u = 0; u < kTurn; ++u) l[u] = c[u] >= 0 ? labels[c[u]] : -1;
#pragma unroll
            for (int u = 0; u < kTurn; ++u) { c0 += l[u] == 0; c1 += l[u] == 1; }
        }
    }
#pragma unroll
    for (int o = kXcGroup / 2; o > 0; o >>= 1) { c0 += __shfl_xor(c0, o); c1 += __shfl_xor(c1, o); }
    if (v < n && sub == 0) xc_node_terms(c0, c1, x, &ec, &base);
    const int64_t unit = (int64_t)blockIdx.x * (kXcBlock / 64) + (threadIdx.x >> 6);
    xc_wave_sums(ec, base, sum_ec + unit, sum_base + unit);
}

constexpr int kXcTile = kXcBlock;                  // nodes per tile
constexpr int kXcTileUnits = kXcTile / 64;         // sums per tile: one per wave, so that no wave waits for another's tails
constexpr int64_t kXcGrid = 2048;                  // workgroups that walk them: all of them resident (eight per CU)

// Tiles of more than `limit` entries, half a workgroup's share of all, are left to k_xc_split: one of 12.8M entries (a
// graph in order of degree) kept one workgroup busy for 17 ms.  The list cannot overflow: fewer than `cap` tiles have more than nnz / cap entries.
constexpr int64_t kXcSplitMin = 1 << 17;
constexpr uint32_t kXcPiece = 16384;               // entries per workgroup and turn of k_xc_split
struct XcSplit {
    uint32_t count, cap;
    uint2 tile[1];                                 // the tile, its pieces
};
__device__ __forceinline__ int64_t xc_split_limit(int64_t nnz, const XcSplit* split)
{
    const int64_t half = nnz / (2 * kXcGrid), fair = nnz / split->cap + 1;
    const int64_t most = half > fair ? half : fair;
    return most > kXcSplitMin ? most : kXcSplitMin;
}

// What bounds the walk is the look-up of every entry's label: a table larger than an XCD's 4 MB of L2 serves
// 57 to 121 G/s, a smaller one 267 G/s.  Only three kinds of label count (0, 1, any other), so they are
// packed two bits each first, a sixteenth of the int32 table: 16.7M nodes fit the L2.
__global__ __launch_bounds__(kXcBlock) void k_xc_pack(const int32_t* __restrict__ labels, int64_t n, uint32_t* __restrict__ words,
                                                      XcSplit* split, uint32_t cap)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) { split->count = 0u; split->cap = cap; }
    const int64_t count = (n + 15) / 16;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; w < count; w += stride) {
        const int64_t v0 = w * 16;
        const int here = n - v0 < 16 ? (int)(n - v0) : 16;
        uint32_t out = 0;
        for (int i = 0; i < here; ++i) {
            const uint32_t l = (uint32_t)labels[v0 + i];
            out |= (l < 2u ? l : 2u) << (2 * i);
        }
        words[w] = out;
    }
}

// Adds to cnt[label][node of the tile] the entries [first, first + end) of the tile's, the whole workgroup together.
// Ends with a barrier.
template <typename RowT>
__device__ __forceinline__ void xc_count(const RowT* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                         const uint32_t* __restrict__ words, int64_t v0, int nv, int64_t e0, int64_t first,
                                         uint32_t end, uint32_t* rowrel, uint32_t (*cnt)[kXcTile])
{
    constexpr int U = 8;                           // entries in flight per thread
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i <= kXcTile; i += kXcBlock) {
        const int64_t off = (int64_t)rowptr[v0 + (i < nv ? i : nv)] - e0 - first;
        rowrel[i] = off < 0 ? 0u : off > (int64_t)end ? end : (uint32_t)off;
    }
    __syncthreads();
    const int32_t* cbase = colidx + e0 + first;
    const uint32_t wave0 = (uint32_t)(tid & ~63);
    // consecutive lanes hold consecutive entries; uniform trip count over a wave
    for (uint32_t base = wave0; base < end; base += kXcBlock * U) {
        int32_t col[U];
        uint32_t kind[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t i = base + u * kXcBlock + lane;
            col[u] = i < end ? __builtin_nontemporal_load(cbase + i) : -1;
        }
#pragma unroll
        for (int u = 0; u < U; ++u) kind[u] = col[u] >= 0 ? words[(uint32_t)col[u] >> 4] : 0u;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t at = base + u * kXcBlock;
            if (at >= end) break;
            const uint32_t k = col[u] >= 0 ? (kind[u] >> (((uint32_t)col[u] & 15u) * 2u)) & 3u : 2u;
            // the row that owns the entry (the last one that starts at or before it)
            int r = 0;
#pragma unroll
            for (int step = kXcTile >> 1; step >= 1; step >>= 1)
                if (rowrel[r + step] <= at + lane) r += step;
            // lanes of one row are neighbours: the first of them adds up the wave's ballots over the run,
            // one LDS atomic per row and wave however long the row
            const int before = __shfl_up(r, 1);
            const bool head = lane == 0 || before != r;
            const unsigned long long heads = __ballot(head);
            const unsigned long long b0 = __ballot(k == 0u), b1 = __ballot(k == 1u);
            if (head) {
                const unsigned long long later = heads & ~((2ull << lane) - 1ull);
                const unsigned long long run = (later ? (later & (~later + 1ull)) - 1ull : ~0ull) & ~((1ull << lane) - 1ull);
                const uint32_t c0 = (uint32_t)__popcll(b0 & run), c1 = (uint32_t)__popcll(b1 & run);
                if (c0) atomicAdd(&cnt[0][r], c0);
                if (c1) atomicAdd(&cnt[1][r], c1);
            }
        }
    }
    __syncthreads();
}

// FUSED: the terms are summed here as well, as the entry point without allocations needs it.  The tail's code takes
// 220 registers, and the two waves per SIMD that they leave cannot keep enough look-ups in flight; the other form
// writes the counts (8 bytes per node) for k_xc_terms_counts.  13,875,000 nodes, 400M entries: 6.16 ms from the int32
// table with sixteen lanes per row, 5.3 ms fused, 2.19 + 0.68 ms as two kernels.
// `counts`: FUSED: 256 per split tile, in the order of the list; else one per node.
template <typename RowT, bool FUSED>
__global__ __launch_bounds__(kXcBlock) void k_xc_terms(const RowT* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                       int64_t n, const uint32_t* __restrict__ words, double x,
                                                       uint2* __restrict__ counts, XcSplit* split, double* sum_ec, double* sum_base)
{
    __shared__ uint32_t rowrel[kXcTile + 1];
    __shared__ uint32_t cnt[2][kXcTile];
    __shared__ uint32_t s_slot;
    const int tid = threadIdx.x;
    const int64_t tiles = (n + kXcTile - 1) / kXcTile, limit = xc_split_limit((int64_t)rowptr[n], split);
    // four neighbouring tiles at a time (13.9M nodes, 395M entries: 2.18 ms; one at a time 2.24, a contiguous range per
    // workgroup 2.15, but 130 in order of degree); one where the tails are summed as well (1.03 ms for 1.13 at 4M nodes)
    constexpr int64_t kTurn = FUSED ? 1 : 4;
    for (int64_t i = 0;; ++i) {
        const int64_t tile = ((int64_t)blockIdx.x + i / kTurn * gridDim.x) * kTurn + i % kTurn;
        if (tile >= tiles) break;
        const int64_t v0 = tile * kXcTile;
        const int nv = n - v0 < kXcTile ? (int)(n - v0) : kXcTile;
        const int64_t e0 = (int64_t)rowptr[v0], ne = (int64_t)rowptr[v0 + nv] - e0;
        if (ne > limit) {
            if (tid == 0) {
                s_slot = atomicAdd(&split->count, 1u);
                split->tile[s_slot] = make_uint2((uint32_t)tile, (uint32_t)((ne + kXcPiece - 1) / kXcPiece));
            }
            __syncthreads();
            if (FUSED) counts[(size_t)s_slot * kXcTile + tid] = make_uint2(0u, 0u);
            else if (tid < nv) counts[v0 + tid] = make_uint2(0u, 0u);
            __syncthreads();
            continue;
        }
        // (a thread's own counts of the tile before are read: the barrier in xc_count covers the clearing)
        cnt[0][tid] = 0; cnt[1][tid] = 0;
        xc_count(rowptr, colidx, words, v0, nv, e0, (int64_t)0, (uint32_t)ne, rowrel, cnt);
        if constexpr (FUSED) {
            double ec = 0.0, base = 0.0;
            if (tid < nv) xc_node_terms(cnt[0][tid], cnt[1][tid], x, &ec, &base);
            const int64_t unit = tile * kXcTileUnits + (tid >> 6);
            if (unit * 64 < n) xc_wave_sums(ec, base, sum_ec + unit, sum_base + unit);
        } else {
            if (tid < nv) counts[v0 + tid] = make_uint2(cnt[0][tid], cnt[1][tid]);
        }
    }
}

// the split tiles' entries, a piece per workgroup and turn: whole numbers, so they may add up in any order
template <typename RowT, bool FUSED>
__global__ __launch_bounds__(kXcBlock) void k_xc_split(const RowT* __restrict__ rowptr, const int32_t* __restrict__ colidx, int64_t n,
                                                       const uint32_t* __restrict__ words, uint2* counts, const XcSplit* split)
{
    __shared__ uint32_t rowrel[kXcTile + 1];
    __shared__ uint32_t cnt[2][kXcTile];
    __shared__ uint2 list[kXcBlock];
    const int tid = threadIdx.x;
    const uint32_t total = split->count, grid = gridDim.x;
    uint32_t next = blockIdx.x;                    // this workgroup's next piece, counted from the tile at hand's first
    for (uint32_t base = 0; base < total; base += kXcBlock) {
        __syncthreads();
        if (base + tid < total) list[tid] = split->tile[base + tid];
        __syncthreads();
        const uint32_t here = total - base < kXcBlock ? total - base : kXcBlock;
        for (uint32_t j = 0; j < here; ++j) {
            const int64_t tile = list[j].x, v0 = tile * kXcTile;
            const uint32_t pieces = list[j].y;
            for (; next < pieces; next += grid) {
                const int nv = n - v0 < kXcTile ? (int)(n - v0) : kXcTile;
                const int64_t e0 = (int64_t)rowptr[v0], ne = (int64_t)rowptr[v0 + nv] - e0, first = (int64_t)next * kXcPiece;
                cnt[0][tid] = 0; cnt[1][tid] = 0;
                xc_count(rowptr, colidx, words, v0, nv, e0, first, (uint32_t)(ne - first < kXcPiece ? ne - first : kXcPiece), rowrel, cnt);
                uint32_t* to = reinterpret_cast<uint32_t*>(counts + (FUSED ? (size_t)(base + j) * kXcTile : (size_t)v0) + tid);
                if (cnt[0][tid]) atomicAdd(to, cnt[0][tid]);
                if (cnt[1][tid]) atomicAdd(to + 1, cnt[1][tid]);
                __syncthreads();
            }
            next -= pieces;
        }
    }
}

// The terms from neighbour counts that are at hand, one lane per node (x, y: its labelled neighbours in partition 0 and
// 1).  split == nullptr: counts of all nodes, else of the split tiles, 256 each.
__global__ __launch_bounds__(kXcBlock) void k_xc_terms_counts(const uint2* __restrict__ counts, int64_t n, double x,
                                                              const XcSplit* __restrict__ split, double* sum_ec, double* sum_base)
{
    const int64_t tiles = split ? (int64_t)split->count : (n + kXcTile - 1) / kXcTile;
    for (int64_t i = blockIdx.x; i < tiles; i += gridDim.x) {
        const int64_t v = (split ? (int64_t)split->tile[i].x : i) * kXcTile + threadIdx.x;
        double ec = 0.0, base = 0.0;
        if (v < n) {
            const uint2 c = counts[i * kXcTile + threadIdx.x];
            xc_node_terms(c.x, c.y, x, &ec, &base);
        }
        const int64_t unit = v >> 6;
        if (unit * 64 < n) xc_wave_sums(ec, base, sum_ec + unit, sum_base + unit);
    }
}

// Sum of `units` pairs: by one workgroup, or workgroup b of several takes the b-th of gridDim.x ranges.
__global__ __launch_bounds__(1024) void k_xc_total(const double* __restrict__ sum_ec, const double* __restrict__ sum_base,
                                                   int64_t units, double* out_ec, double* out_base)
{
    __shared__ double s_ec[16], s_base[16];
    const int64_t each = (units + gridDim.x - 1) / gridDim.x, lo = (int64_t)blockIdx.x * each, hi = lo + each < units ? lo + each : units;
    double a = 0.0, b = 0.0;
    for (int64_t i = lo + threadIdx.x; i < hi; i += 1024) { a += sum_ec[i]; b += sum_base[i]; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { a += __shfl_down(a, o); b += __shfl_down(b, o); }
    if ((threadIdx.x & 63) == 0) { s_ec[threadIdx.x >> 6] = a; s_base[threadIdx.x >> 6] = b; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double x = 0.0, y = 0.0;
        for (int q = 0; q < 16; ++q) { x += s_ec[q]; y += s_base[q]; }
        out_ec[blockIdx.x] = x; out_base[blockIdx.x] = y;
    }
}

constexpr int64_t kXcSmallN = 1 << 16;             // below it: k_xc_small
constexpr int64_t kXcOneTotal = 16384;             // most sums that one workgroup adds up
constexpr int64_t kXcParts = 256;
constexpr uint32_t kXcSplitCap = 16384, kXcSplitCapStatic = 896;       // most split tiles

// The scratch of a call, in doubles from `base` (null: only its size): the units' sums, the parts' sums, the packed
// labels, the list of split tiles and the counts (of every node, of the split tiles only, or none).
enum class XcCounts { kNone, kSplit, kAll };
struct XcScratch {
    int64_t units;
    double *ec, *base, *part_ec, *part_base;
    uint32_t* words;
    XcSplit* split;
    uint32_t cap;
    uint2* counts;
    size_t bytes;
};
constexpr int64_t xc_waves(int64_t n) { return (n + 63) / 64; }
constexpr int64_t xc_units(int64_t n) { return n < kXcSmallN ? (n + kXcRows - 1) / kXcRows * (kXcBlock / 64) : xc_waves(n); }
constexpr int64_t xc_words8(int64_t n) { return ((n + 15) / 16 * 4 + 7) / 8; }
inline XcScratch xc_scratch(double* base, int64_t n, int64_t units, XcCounts counts)
{
    XcScratch s{};
    int64_t off = 0;
    auto take = [&](auto*& p, int64_t doubles) {
        p = base ? reinterpret_cast<std::remove_reference_t<decltype(p)>>(base + off) : nullptr;
        off += doubles;
    };
    s.units = units;
    s.cap = counts == XcCounts::kSplit ? kXcSplitCapStatic : kXcSplitCap;
    take(s.ec, units);
    take(s.base, units);
    take(s.part_ec, kXcParts);
    take(s.part_base, kXcParts);
    if (n >= kXcSmallN && counts != XcCounts::kNone) {
        take(s.words, xc_words8(n));
        take(s.split, 1 + (int64_t)s.cap);
        take(s.counts, counts == XcCounts::kAll ? n : (int64_t)s.cap * kXcTile);
    }
    s.bytes = (size_t)off * sizeof(double);
    return s;
}
static_assert((2 * xc_waves(kXcStaticMaxN) + 2 * kXcParts + xc_words8(kXcStaticMaxN) + 1 + kXcSplitCapStatic * (1 + kXcTile)) * 8 <= kXcStaticBytes &&
              (2 * xc_units(kXcSmallN - 1) + 2 * kXcParts) * 8 <= kXcStaticBytes, "the fixed buffer holds the largest input");
static_assert(sizeof(XcSplit) == 16, "a head of 8 bytes and 8 per tile");

void xc_total(const XcScratch& s, double* out, hipStream_t stream)
{
    if (s.units <= kXcOneTotal) {
        hipLaunchKernelGGL(k_xc_total, dim3(1), dim3(1024), 0, stream, (const double*)s.ec, (const double*)s.base, s.units, out, out + 1);
        return;
    }
    hipLaunchKernelGGL(k_xc_total, dim3((unsigned)kXcParts), dim3(1024), 0, stream, (const double*)s.ec, (const double*)s.base, s.units,
                       s.part_ec, s.part_base);
    hipLaunchKernelGGL(k_xc_total, dim3(1), dim3(1024), 0, stream, (const double*)s.part_ec, (const double*)s.part_base, kXcParts, out, out + 1);
}

// workgroups that walk the tiles
inline int64_t xc_walk(int64_t n)
{
    const int64_t tiles = (n + kXcTile - 1) / kXcTile;
    return tiles < kXcGrid ? tiles : kXcGrid;
}

// FUSED: s has no counts but those of the split tiles
template <typename RowT, bool FUSED>
void xc_launch(const void* rowptr_, const int32_t* colidx, int64_t n, const int32_t* labels, double x, const XcScratch& s, double* out,
               hipStream_t stream)
{
    const RowT* rowptr = (const RowT*)rowptr_;
    if (n < kXcSmallN) {
        hipLaunchKernelGGL(k_xc_small<RowT>, dim3((unsigned)((n + kXcRows - 1) / kXcRows)), dim3(kXcBlock), 0, stream, rowptr, colidx, n, labels,
                           x, s.ec, s.base);
    } else {
        const int64_t pack = ((n + 15) / 16 + kXcBlock - 1) / kXcBlock, walk = xc_walk(n);
        hipLaunchKernelGGL(k_xc_pack, dim3((unsigned)(pack < 4096 ? pack : 4096)), dim3(kXcBlock), 0, stream, labels, n, s.words, s.split, s.cap);
        hipLaunchKernelGGL((k_xc_terms<RowT, FUSED>), dim3((unsigned)walk), dim3(kXcBlock), 0, stream, rowptr, colidx, n,
                           (const uint32_t*)s.words, x, s.counts, s.split, s.ec, s.base);
        hipLaunchKernelGGL((k_xc_split<RowT, FUSED>), dim3((unsigned)kXcGrid), dim3(kXcBlock), 0, stream, rowptr, colidx, n,
                           (const uint32_t*)s.words, s.counts, (const XcSplit*)s.split);
        hipLaunchKernelGGL(k_xc_terms_counts, dim3((unsigned)(FUSED && walk > s.cap ? s.cap : walk)), dim3(kXcBlock), 0, stream,
                           (const uint2*)s.counts, n, x, FUSED ? (const XcSplit*)s.split : (const XcSplit*)nullptr, s.ec, s.base);
    }
    xc_total(s, out, stream);
}

constexpr int kXcMaxDevices = 64;
std::mutex xc_mu;
double* xc_scratch_ptr[kXcMaxDevices] = {};        // device address of `scratch`, per GPU

}  // namespace

extern "C" int64_t grem_expected_cut_noalloc_max_n(void) { return kXcStaticMaxN; }

extern "C" int grem_expected_cut_noalloc(const void* rowptr, int32_t rowptr_bits, const int32_t* colidx, int64_t n,
                                         const int32_t* labels, double x, double* out, void* stream_)
{
    if (!rowptr || !colidx || !labels || !out || n < 1 || (rowptr_bits != 32 && rowptr_bits != 64) || !(x > 0.0) ||
        !(x <= 1.0))
        return GREM_ERR_ARG;
    if (n > kXcStaticMaxN) return GREM_ERR_LIMIT;
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess) return GREM_ERR_HIP;
    if (dev < 0 || dev >= kXcMaxDevices) return GREM_ERR_LIMIT;
    double* partial = nullptr;
    {
        std::lock_guard<std::mutex> lock(xc_mu);
        if (!xc_scratch_ptr[dev]) {          // first call on this GPU: look its copy of the array up
            void* p = nullptr;
            if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
                (void)hipGetLastError();
                return GREM_ERR_HIP;
            }
            xc_scratch_ptr[dev] = (double*)p;
        }
        partial = xc_scratch_ptr[dev];
    }
    // all sums, the packed labels, the list and the counts of what it holds are written before they are
    // read: nothing has to start at zero, whatever an earlier call left behind
    hipStream_t stream = (hipStream_t)stream_;
    const XcScratch s = xc_scratch(partial, n, xc_units(n), XcCounts::kSplit);
    if (rowptr_bits == 64) xc_launch<int64_t, true>(rowptr, colidx, n, labels, x, s, out, stream);
    else xc_launch<int32_t, true>(rowptr, colidx, n, labels, x, s, out, stream);
    return hipGetLastError() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
}

extern "C" int grem_expected_cut(const void* rowptr, int32_t rowptr_bits, const int32_t* colidx, int64_t n,
                                 const int32_t* labels, double x, double* out, void* stream_)
{
    if (!rowptr || !colidx || !labels || !out || n < 1 || n > INT32_MAX || (rowptr_bits != 32 && rowptr_bits != 64) ||
        !(x > 0.0) || !(x <= 1.0))
        return GREM_ERR_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    double* partial = nullptr;
    bool counts_fit = true;
    if (hipMallocAsync((void**)&partial, xc_scratch(nullptr, n, xc_units(n), XcCounts::kAll).bytes, stream) != hipSuccess) {
        (void)hipGetLastError();
        counts_fit = false;
        if (hipMallocAsync((void**)&partial, xc_scratch(nullptr, n, xc_units(n), XcCounts::kSplit).bytes, stream) != hipSuccess) {
            (void)hipGetLastError();
            return GREM_ERR_NOMEM;
        }
    }
    const XcScratch s = xc_scratch(partial, n, xc_units(n), counts_fit ? XcCounts::kAll : XcCounts::kSplit);
    auto go = [&](auto row, auto fused) {
        xc_launch<decltype(row), decltype(fused)::value>(rowptr, colidx, n, labels, x, s, out, stream);
    };
    if (rowptr_bits == 64) counts_fit ? go(int64_t{}, std::false_type{}) : go(int64_t{}, std::true_type{});
    else counts_fit ? go(int32_t{}, std::false_type{}) : go(int32_t{}, std::true_type{});
    int rc = hipGetLastError() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
    if (hipFreeAsync(partial, stream) != hipSuccess) rc = GREM_ERR_HIP;
    return rc;
}

// Eq. (1) on a plan: the neighbour counts come from the plan's re-laid-out copy of the entries (every label
// look-up served from LDS) instead of one look-up through the caches per CSR entry.
extern "C" int grem_plan_expected_cut(const grem_plan* plan, const int32_t* labels, double x, double* out, void* stream_)
{
    const int64_t n = grem_plan_n(plan);
    if (!plan || n < 1 || !labels || !out || !(x > 0.0) || !(x <= 1.0)) return GREM_ERR_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    uint32_t* counts = nullptr;
    double* partial = nullptr;
    if (hipMallocAsync((void**)&counts, (size_t)n * 2 * sizeof(uint32_t), stream) != hipSuccess) {
        (void)hipGetLastError();
        return GREM_ERR_NOMEM;
    }
    if (hipMallocAsync((void**)&partial, xc_scratch(nullptr, n, xc_waves(n), XcCounts::kNone).bytes, stream) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFreeAsync(counts, stream);
        return GREM_ERR_NOMEM;
    }
    int rc = grem_plan_neighbour_counts(plan, 2, labels, counts, stream);
    if (rc == GREM_OK) {
        const XcScratch s = xc_scratch(partial, n, xc_waves(n), XcCounts::kNone);
        hipLaunchKernelGGL(k_xc_terms_counts, dim3((unsigned)xc_walk(n)), dim3(kXcBlock), 0, stream, (const uint2*)counts, n, x,
                           (const XcSplit*)nullptr, s.ec, s.base);
        xc_total(s, out, stream);
        if (hipGetLastError() != hipSuccess) rc = GREM_ERR_HIP;
    }
    if (hipFreeAsync(partial, stream) != hipSuccess) rc = rc == GREM_OK ? GREM_ERR_HIP : rc;
    if (hipFreeAsync(counts, stream) != hipSuccess) rc = rc == GREM_OK ? GREM_ERR_HIP : rc;
    return rc;
}
