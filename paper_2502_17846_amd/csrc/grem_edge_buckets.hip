// Edge buckets for gfx950 (Armada paper, Sec. 3, storage layer): given the partition of every node, the
// edges are grouped so that bucket (i, j) holds the edges from nodes of partition i to nodes of
// partition j, each bucket stored as one sequential list; buckets follow each other in the order of
// i*k + j and an edge keeps its stream position relative to the other edges of its bucket (the paper
// fixes no order inside a bucket; this makes the result unique).
//
// A stable counting sort by key = label[src]*k + label[dst], one workgroup per tile of the stream:
//   k_eb_hist     keys of the tile's edges (two look-ups into a byte-per-node label table), stored as
//                 uint16 for the second pass, and the tile's histogram over the k*k buckets in LDS
//                 -> H[tile][bucket].  Where the table outgrows the L2 the look-ups are served from LDS instead
//                 (k_eb_bin, k_eb_lookup, k_eb_keys: below) and k_eb_hist_keys takes the keys as they are
//   k_eb_colsum / k_eb_bases / k_eb_colscan
//                 exclusive prefix sums of H in bucket-major order (bucket, then tile): H[tile][bucket]
//                 becomes the output position of the tile's first edge of that bucket
//   k_eb_scatter  the tile again, 256 edges at a time in stream order: lanes with equal keys are matched
//                 inside a wave (one ballot per key bit), the waves take their ranges from the LDS
//                 cursors one after the other, every edge is written to cursor + rank
//   k_eb_scatter_lds  (tiles of 4,096 or 8,192 edges, up to 1,024 buckets) the tile is sorted in LDS first and then
//                 written out run by run
#include <hip/hip_runtime.h>

#include <cstdint>
#include <type_traits>

#include "grem.h"

namespace {

typedef unsigned long long u64;
constexpr int kEbBlock = 256;
constexpr int kEbWaves = kEbBlock / 64;
constexpr int kEbMaxK = 128;                       // k*k*4 bytes of LDS: 64 KB at k = 128
constexpr int64_t kEbMaxCells = (int64_t)1 << 27;  // tiles * k*k
// Tiles of 8192 edges for long lists with many buckets, of 4096 for all others.  Few buckets make long runs in either, and the
// larger tile's kernel is the slower one by itself; it wins where runs of a 4,096-edge tile are short (64 edges: k = 8) and the
// table of the tiles' counts outgrows the L2 (m * k * k = 6.5e9: 6.3 MB of it).  All kernels of a call, 4096 | 8192, ms:
//   34M edges   k = 2 0.53 | 0.57, 8 0.62 | 0.65, 12 0.68 | 0.69, 16 0.72 | 0.71, 32 0.92 | 0.89, 33 1.42 | 1.40, 64 1.81 | 1.64
//   68M         k = 4 1.20 | 1.28, 8 1.28 | 1.31, 10 1.34 | 1.33, 12 1.39 | 1.36, 16 1.45 | 1.40
//   200M        k = 2 3.53 | 3.69, 4 3.54 | 3.63, 6 3.72 | 3.67, 8 3.80 | 3.72, 16 4.80 | 3.95
//   400M        k = 2 7.4 | 7.6, 8 7.5-8.2 | 7.6, 10 7.8-8.7 | 7.7, 16 9.2-9.9 | 8.1, 32 11.5 | 10.6, 33 16.2-17.7 | 15.6
//   1.6e9       k = 2 33.1 | 34.0, 3 31.8 | 33.9, 6 33.2 | 34.1, 8 33.7 | 34.3, 10 34.4 | 34.5, 16 39.4-42.5 | 35.4
// (k >= 33 does not fit k_eb_scatter_lds and gains by the smaller table alone.)
constexpr int64_t kEbWideMinM = 1 << 25, kEbWideMinCells = 6'500'000'000;
constexpr int32_t kEbWideMinBuckets = 64;
inline bool eb_wide(int64_t m, int32_t k2) { return m >= kEbWideMinM && k2 >= kEbWideMinBuckets && m * k2 >= kEbWideMinCells; }
constexpr uint32_t kBadLabel = 0xFFu;
constexpr int64_t kEbBinMinN = 1ll << 23, kEbBinMinM = 1 << 22, kEbBinMinNM = 200'000'000'000'000;

__global__ __launch_bounds__(256) void k_eb_zero(uint32_t* p, size_t count)
{
    const size_t stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += stride) p[i] = 0u;
}

// one byte per node; labels outside [0, k) become kBadLabel (*bad_labels = 1 if there are any)
__global__ __launch_bounds__(256) void k_eb_compact(int64_t n, const int32_t* __restrict__ labels, int32_t k, uint8_t* L8,
                                                    uint32_t* bad_labels)
{
    bool bad = false;
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const int32_t l = labels[v];
        const bool fits = l >= 0 && l < k;
        L8[v] = fits ? (uint8_t)l : (uint8_t)kBadLabel;
        bad |= !fits;
    }
    if (bad) *bad_labels = 1u;
}

// flags[0]: an endpoint outside [0, n); flags[1]: an endpoint whose label lies outside [0, k)
__global__ __launch_bounds__(kEbBlock) void k_eb_hist(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                      int64_t m, uint32_t n, int64_t tile, const uint8_t* __restrict__ L8,
                                                      int32_t k, uint16_t* __restrict__ key16, uint32_t* __restrict__ H,
                                                      uint32_t* flags)
{
    extern __shared__ uint32_t hist[];
    const int k2 = k * k;
    for (int b = threadIdx.x; b < k2; b += kEbBlock) hist[b] = 0u;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * tile, hi = lo + tile < m ? lo + tile : m;
    bool bad = false, outside = false;
    for (int64_t e = lo + threadIdx.x; e < hi; e += kEbBlock) {
        const uint32_t s = (uint32_t)src[e], d = (uint32_t)dst[e];
        uint32_t key = 0u;
        if (s < n && d < n) {
            const uint32_t ls = L8[s], ld = L8[d];
            if (ls < (uint32_t)k && ld < (uint32_t)k) key = ls * (uint32_t)k + ld;
            else bad = true;
        } else {
            outside = true;
        }
        key16[e] = (uint16_t)key;
        atomicAdd(&hist[key], 1u);
    }
    if (outside) flags[0] = 1u;
    if (bad) flags[1] = 1u;
    __syncthreads();
    uint32_t* row = H + (size_t)blockIdx.x * (size_t)k2;
    for (int b = threadIdx.x; b < k2; b += kEbBlock) row[b] = hist[b];
}

// partial[b*S + seg] = sum over the tiles of segment seg of H[tile][b]
__global__ __launch_bounds__(256) void k_eb_colsum(const uint32_t* __restrict__ H, int64_t tiles, int32_t k2, int32_t S,
                                                   int64_t seg_len, uint32_t* partial)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)k2 * S) return;
    const int b = (int)(id % k2), seg = (int)(id / k2);
    const int64_t t0 = seg * seg_len, t1 = t0 + seg_len < tiles ? t0 + seg_len : tiles;
    uint32_t sum = 0;
    for (int64_t t = t0; t < t1; ++t) sum += H[(size_t)t * k2 + b];
    partial[(size_t)b * S + seg] = sum;
}

// One workgroup: exclusive prefix sums of partial (bucket-major) in place, and the buckets' offsets.
__global__ __launch_bounds__(1024) void k_eb_bases(uint32_t* partial, int64_t len, int32_t k2, int32_t S,
                                                   int64_t m, int64_t* bucket_offsets)
{
    __shared__ uint32_t wsum[16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t carry = 0;
    for (int64_t base = 0; base < len; base += 1024) {
        const int64_t i = base + threadIdx.x;
        const uint32_t x = i < len ? partial[i] : 0u;
        uint32_t incl = x;
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o);
            if (lane >= o) incl += y;
        }
        if (lane == 63) wsum[wave] = incl;
        __syncthreads();
        uint32_t before = 0, all = 0;
        for (int q = 0; q < 16; ++q) {
            const uint32_t t = wsum[q];
            if (q < wave) before += t;
            all += t;
        }
        if (i < len) {
            const uint32_t excl = carry + before + incl - x;
            partial[i] = excl;
            if (i % S == 0) bucket_offsets[i / S] = (int64_t)excl;
        }
        carry += all;
        __syncthreads();
    }
    if (threadIdx.x == 0) bucket_offsets[k2] = m;
}

// H[tile][b] becomes the output position of the tile's first edge of bucket b
__global__ __launch_bounds__(256) void k_eb_colscan(uint32_t* __restrict__ H, int64_t tiles, int32_t k2, int32_t S,
                                                    int64_t seg_len, const uint32_t* __restrict__ segbase)
{
    const int64_t id = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (id >= (int64_t)k2 * S) return;
    const int b = (int)(id % k2), seg = (int)(id / k2);
    const int64_t t0 = seg * seg_len, t1 = t0 + seg_len < tiles ? t0 + seg_len : tiles;
    uint32_t run = segbase[(size_t)b * S + seg];
    for (int64_t t = t0; t < t1; ++t) {
        const uint32_t c = H[(size_t)t * k2 + b];
        H[(size_t)t * k2 + b] = run;
        run += c;
    }
}

// ---- the keys of large graphs: look-ups from LDS ------------------------------------------------------------
//
// A look-up in a table that outgrows the L2 is a 64-byte miss: 55 G/s at 111M nodes, 57 ms for the two ends of 1.6e9
// edges.  Instead, a batch of edges at a time:
//   k_eb_bin      a workgroup sorts the ends of its tile of edges by bins of 2^cb nodes, in LDS, and writes them run by
//                 run to the bins' lists (the node's place in its bin), beside where its runs went and, per edge,
//                 the places of its two ends in the sorted tile
//   k_eb_lookup   a bin's labels in LDS, its list streamed through them: a byte per entry
//   k_eb_keys     a tile's runs of labels collected in LDS; every edge picks its two up: its key
// All of it is long streams: 27 bytes per end where the miss moves 64.  (k_eb_bin_count and k_eb_bin_scan beforehand: the
// lists' sizes for every batch, and the range check of the endpoints; ends out of range count as the last
// node.)
// 1.6e9 edges of 111M nodes: 57.4 ms with look-ups in the table, 27.5 in these kernels.  Below 8M nodes the table's
// look-ups are the faster way (4M nodes, 50M edges: 1.35 ms against 1.5 to 1.7), and the lists' memory takes some 0.3 ms to get
// and give back, which the table's misses must outweigh (binned against table, k = 16: 8.4M nodes and 12M edges 0.68 and 0.52 ms,
// 24M edges 0.73 and 0.96; 20M nodes and 8.4M edges 0.63 and 0.52, 12M edges 0.57 and 0.64; 60M nodes and 6M edges 0.53 and 0.57).
constexpr int kEbBins = 1024;
constexpr int kEbBinThreads = 1024;
constexpr int kEbBinTile = 8192;                  // edges per workgroup (16,384 and one workgroup per CU: 47.5 ms a call for 46)
constexpr int kEbBinPer = kEbBinTile / kEbBinThreads;

// exclusive prefix of x over kEbBinThreads threads; wsum: 16 words of LDS
__device__ __forceinline__ uint32_t eb_block_exclusive(uint32_t x, uint32_t* wsum)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl = x;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t before = incl - x;
    for (int q = 0; q < wave; ++q) before += wsum[q];
    return before;
}

__device__ __forceinline__ uint32_t eb_end(int32_t id, uint32_t n) { return (uint32_t)id < n ? (uint32_t)id : n - 1u; }

// rank among the ends counted so far of the same bin.  Lanes that share the first active lane's bin (edges sorted by
// source, popular ids) take one atomic together if they are many: equal addresses are served one after the other.
__device__ __forceinline__ uint32_t eb_count(uint32_t* hist, uint32_t bin)
{
    const uint32_t first = (uint32_t)__builtin_amdgcn_readfirstlane((int)bin);
    const u64 same = __ballot(bin == first);
    if (__popcll(same) < 16) return atomicAdd(&hist[bin], 1u);
    const u64 below = (1ull << (threadIdx.x & 63)) - 1ull;
    uint32_t base = 0u;
    if (bin != first) return atomicAdd(&hist[bin], 1u);
    if ((same & below) == 0ull) base = atomicAdd(&hist[bin], (uint32_t)__popcll(same));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + (uint32_t)__popcll(same & below);
}

// table[batch][bin]: ends of the batch's edges; table[batch][kEbBins]: how many of them lie in bins that its workgroup
// met at least four times per 128-byte line of their labels
__global__ __launch_bounds__(kEbBinThreads) void k_eb_bin_count(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                                int64_t m, int64_t batch, uint32_t n, int cb,
                                                                uint32_t* __restrict__ table, uint32_t* flags)
{
    __shared__ uint32_t hist[kEbBins];
    const int64_t lo = (int64_t)blockIdx.y * batch, hi = lo + batch < m ? lo + batch : m;
    hist[threadIdx.x] = 0u;
    __syncthreads();
    bool bad = false;
    for (int64_t t = lo + (int64_t)blockIdx.x * kEbBinTile; t < hi; t += (int64_t)gridDim.x * kEbBinTile) {
        int32_t s[kEbBinPer], d[kEbBinPer];
#pragma unroll
        for (int u = 0; u < kEbBinPer; ++u) {
            const int64_t e = t + u * kEbBinThreads + threadIdx.x;
            s[u] = e < hi ? src[e] : 0;
            d[u] = e < hi ? dst[e] : 0;
        }
#pragma unroll
        for (int u = 0; u < kEbBinPer; ++u) {
            if (t + u * kEbBinThreads + threadIdx.x >= hi) continue;
            bad |= (uint32_t)s[u] >= n || (uint32_t)d[u] >= n;
            (void)eb_count(hist, eb_end(s[u], n) >> cb);
            (void)eb_count(hist, eb_end(d[u], n) >> cb);
        }
    }
    if (bad) flags[0] = 1u;
    __syncthreads();
    const uint32_t c = hist[threadIdx.x];
    uint32_t* row = table + (size_t)blockIdx.y * (kEbBins + 1);
    if (c) atomicAdd(&row[threadIdx.x], c);
    uint32_t local = c >= 1u << (cb - 5) ? c : 0u;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) local += __shfl_xor(local, o);
    if (local && (threadIdx.x & 63) == 0) atomicAdd(&row[kEbBins], local);
}

// sizes -> starts (a workgroup per batch); cursors: a second copy, which k_eb_bin moves on.  parts: how many workgroups
// of k_eb_lookup share a bin's list, as starts: in proportion to its length, `want` in all and at most one more per
// bin.  (Cut into the same number of parts each, lists of popular ids kept a few workgroups busy: ids in order of
// degree, a batch of 33M edges of 111M nodes: 1139 us for 136 on permuted ids.)
// A batch of which more than 52 % of the ends are local (see k_eb_bin_count) gets no parts: its look-ups go to the table,
// whose lines the caches then hold.  400M edges of 111M nodes in order of degree and sorted by source (66 % local):
// 9.5 ms that way, 11.2 binned; sorted by source alone (50 %) 12.8 and 11.2, in order of degree alone (39 %) 12.9 and 12.5.
__global__ __launch_bounds__(kEbBins) void k_eb_bin_scan(uint32_t* table, uint32_t* cursors, uint32_t* parts, uint32_t want)
{
    __shared__ uint32_t wsum[16], s_total;
    uint32_t* row = table + (size_t)blockIdx.x * (kEbBins + 1);
    const uint32_t c = row[threadIdx.x], local = row[kEbBins];
    const uint32_t excl = eb_block_exclusive(c, wsum);
    row[threadIdx.x] = excl;
    cursors[(size_t)blockIdx.x * kEbBins + threadIdx.x] = excl;
    if (threadIdx.x == kEbBins - 1) { row[kEbBins] = excl + c; s_total = excl + c; }
    __syncthreads();
    const uint32_t fair = (uint32_t)(((uint64_t)c * want + s_total / 2u) / s_total);      // (a batch has edges)
    const bool direct = (uint64_t)local * 25u > (uint64_t)s_total * 13u;
    const uint32_t mine = c == 0u || direct ? 0u : fair == 0u ? 1u : fair;
    const uint32_t first = eb_block_exclusive(mine, wsum);
    uint32_t* prow = parts + (size_t)blockIdx.x * (kEbBins + 1);
    prow[threadIdx.x] = first;
    if (threadIdx.x == kEbBins - 1) prow[kEbBins] = first + mine;
}

// runs[tile][bin]: (where the tile's run of the bin went, its start in the sorted tile); places[edge of the batch]: those of
// its two ends in the sorted tile, 16 bits each
template <typename Item>
__global__ __launch_bounds__(kEbBinThreads, 8) void k_eb_bin(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                          int64_t count, uint32_t n, int cb, int nbins,
                                                          const uint32_t* __restrict__ prow, uint32_t* __restrict__ cursors,
                                                          Item* __restrict__ lists, uint2* __restrict__ runs,
                                                          uint32_t* __restrict__ places)
{
    if (prow[kEbBins] == 0u) return;               // (look-ups in the table: k_eb_keys)
    extern __shared__ uint32_t items[];            // 2 * kEbBinTile: place in bin, bin above it
    __shared__ uint32_t hist[kEbBins], start[kEbBins], at[kEbBins], wsum[16];
    const int tid = threadIdx.x;
    const int64_t lo = (int64_t)blockIdx.x * kEbBinTile;
    hist[tid] = 0u;
    uint32_t a[kEbBinPer], b[kEbBinPer];
#pragma unroll
    for (int u = 0; u < kEbBinPer; ++u) {
        const int64_t e = lo + u * kEbBinThreads + tid;
        a[u] = e < count ? eb_end(__builtin_nontemporal_load(src + e), n) : 0u;
        b[u] = e < count ? eb_end(__builtin_nontemporal_load(dst + e), n) : 0u;
    }
    __syncthreads();
    uint32_t rank[kEbBinPer];                      // of the two ends among their bins, 16 bits each (below 16,384)
#pragma unroll
    for (int u = 0; u < kEbBinPer; ++u) {
        rank[u] = 0u;
        if (lo + u * kEbBinThreads + tid < count) {
            rank[u] = eb_count(hist, a[u] >> cb);
            rank[u] |= eb_count(hist, b[u] >> cb) << 16;
        }
    }
    __syncthreads();
    const uint32_t c = hist[tid];
    const uint32_t excl = eb_block_exclusive(c, wsum);
    start[tid] = excl;
    if (tid < nbins) {
        const uint32_t to = c ? atomicAdd(&cursors[tid], c) : 0u;
        at[tid] = to - excl;
        runs[(size_t)blockIdx.x * nbins + tid] = make_uint2(to, excl);
    }
    __syncthreads();
    const uint32_t mask = (1u << cb) - 1u;
#pragma unroll
    for (int u = 0; u < kEbBinPer; ++u) {
        const int64_t e = lo + u * kEbBinThreads + tid;
        if (e >= count) continue;
        const uint32_t pa = start[a[u] >> cb] + (rank[u] & 0xFFFFu), pb = start[b[u] >> cb] + (rank[u] >> 16);
        items[pa] = a[u];
        items[pb] = b[u];
        places[e] = pa | (pb << 16);
    }
    __syncthreads();
    const uint32_t total = start[kEbBins - 1] + hist[kEbBins - 1];
    for (uint32_t i = tid; i < total; i += kEbBinThreads) {
        const uint32_t x = items[i];
        lists[at[x >> cb] + i] = (Item)(x & mask);
    }
}

// a part of a bin's list: the labels, one byte per entry.  PACK: two labels per byte in LDS (k <= 16; a node without a
// valid label is then looked for in the table, if the graph has any: *bad_labels).
template <typename Item, bool PACK>
__global__ __launch_bounds__(kEbBinThreads) void k_eb_lookup(const uint8_t* __restrict__ L8, int64_t n, int cb,
                                                             const uint32_t* __restrict__ prow, const uint32_t* __restrict__ row, const Item* __restrict__ lists,
                                                             uint8_t* __restrict__ labels, const uint32_t* __restrict__ bad_labels,
                                                             uint32_t* flags)
{
    extern __shared__ uint32_t tab[];              // 2^cb labels, a byte or half a byte each
    const int tid = threadIdx.x;
    __shared__ uint32_t s_bin;
    if (blockIdx.x >= prow[kEbBins]) return;
    if (blockIdx.x >= prow[tid] && blockIdx.x < prow[tid + 1]) s_bin = (uint32_t)tid;
    __syncthreads();
    const uint32_t bin = s_bin, parts = prow[bin + 1] - prow[bin], part = blockIdx.x - prow[bin];
    const uint32_t i0 = row[bin], len = row[bin + 1] - i0;
    // (parts meet at multiples of four entries)
    const uint32_t first = (uint32_t)((uint64_t)len * part / parts), last = (uint32_t)((uint64_t)len * (part + 1) / parts);
    auto edge = [&](uint32_t x) { const uint32_t y = (i0 + x) & ~3u; return y < i0 ? i0 : y; };
    const uint32_t b = part == 0 ? i0 : edge(first), e = part + 1 == parts ? i0 + len : edge(last);
    if (b >= e) return;
    const int64_t v0 = (int64_t)bin << cb;
    const uint32_t nodes = n - v0 < (1ll << cb) ? (uint32_t)(n - v0) : 1u << cb;
    // (L8 is 256-byte aligned and padded to that: whole words)
    const uint32_t* l4 = reinterpret_cast<const uint32_t*>(L8 + v0);
    if (PACK) {
        for (uint32_t w = tid; w < (nodes + 7) / 8; w += kEbBinThreads) {
            const uint32_t x = l4[2 * w], y = l4[2 * w + 1];
            const uint32_t p = (x & 15u) | ((x >> 4) & 0xF0u) | ((x >> 8) & 0xF00u) | ((x >> 12) & 0xF000u);
            const uint32_t q = (y & 15u) | ((y >> 4) & 0xF0u) | ((y >> 8) & 0xF00u) | ((y >> 12) & 0xF000u);
            tab[w] = p | (q << 16);
        }
    } else {
        for (uint32_t w = tid; w < (nodes + 3) / 4; w += kEbBinThreads) tab[w] = l4[w];
    }
    const bool some_bad = *bad_labels != 0u;
    __syncthreads();
    const uint8_t* tb = reinterpret_cast<const uint8_t*>(tab);
    bool bad = false;
    auto look = [&](uint32_t x) -> uint32_t {
        if (some_bad) bad |= L8[v0 + x] == kBadLabel;
        return PACK ? ((uint32_t)tb[x >> 1] >> (4 * (x & 1u))) & 15u : (uint32_t)tb[x];
    };
    // four entries per thread and turn, from a multiple of four on; single ones before and after
    const uint32_t b4 = (b + 3u) & ~3u, e4 = e & ~3u;
    for (uint32_t i = b + tid; i < (b4 < e ? b4 : e); i += kEbBinThreads) labels[i] = (uint8_t)look(lists[i]);
    if (b4 < e) for (uint32_t i = (e4 > b4 ? e4 : b4) + tid; i < e; i += kEbBinThreads) labels[i] = (uint8_t)look(lists[i]);
    struct alignas(4 * sizeof(Item)) Four { Item x[4]; };
    constexpr int U = 4;
    for (uint32_t i = b4 + 4 * tid; i < e4; i += 4 * kEbBinThreads * U) {
        Four f[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + 4 * kEbBinThreads * u < e4) f[u] = *reinterpret_cast<const Four*>(lists + i + 4 * kEbBinThreads * u);
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (i + 4 * kEbBinThreads * u < e4)
                *reinterpret_cast<uint32_t*>(labels + i + 4 * kEbBinThreads * u) =
                    look(f[u].x[0]) | (look(f[u].x[1]) << 8) | (look(f[u].x[2]) << 16) | (look(f[u].x[3]) << 24);
    }
    if (bad) flags[1] = 1u;
}

// The tile's labels back in its sorted order (sixteen lanes per run, some 20 to 80 bytes each; what a run has beyond
// kEbLongRun is left to the whole workgroup: edges sorted by source put half a tile in one run, 425 us for 161), then
// the edges' keys.
constexpr uint32_t kEbLongRun = 256;
__global__ __launch_bounds__(kEbBinThreads, 8) void k_eb_keys(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                           int64_t count, uint32_t n, const uint8_t* __restrict__ L8, int nbins, int32_t k,
                                                           const uint32_t* __restrict__ prow, const uint2* __restrict__ runs,
                                                           const uint32_t* __restrict__ places, const uint8_t* __restrict__ labels,
                                                           uint16_t* __restrict__ key16, uint32_t* flags)
{
    __shared__ uint8_t lab[2 * kEbBinTile];
    __shared__ uint32_t s_long, longs[2 * kEbBinTile / kEbLongRun];
    const int tid = threadIdx.x, l = tid & 15;
    if (tid == 0) s_long = 0u;
    const int64_t lo = (int64_t)blockIdx.x * kEbBinTile;
    if (prow[kEbBins] == 0u) {                     // a batch without lists
        uint32_t ls[kEbBinPer], ld[kEbBinPer];
        bool bad = false;
#pragma unroll
        for (int u = 0; u < kEbBinPer; ++u) {
            const int64_t e = lo + u * kEbBinThreads + tid;
            ls[u] = e < count ? eb_end(__builtin_nontemporal_load(src + e), n) : 0u;
            ld[u] = e < count ? eb_end(__builtin_nontemporal_load(dst + e), n) : 0u;
        }
#pragma unroll
        for (int u = 0; u < kEbBinPer; ++u) { ls[u] = L8[ls[u]]; ld[u] = L8[ld[u]]; }
#pragma unroll
        for (int u = 0; u < kEbBinPer; ++u) {
            const int64_t e = lo + u * kEbBinThreads + tid;
            if (e >= count) continue;
            bad |= ls[u] == kBadLabel || ld[u] == kBadLabel;
            key16[e] = ls[u] < (uint32_t)k && ld[u] < (uint32_t)k ? (uint16_t)(ls[u] * (uint32_t)k + ld[u]) : (uint16_t)0;
        }
        if (bad) flags[1] = 1u;
        return;
    }
    const uint32_t total = 2u * (uint32_t)(count - lo < kEbBinTile ? count - lo : kEbBinTile);
    const uint2* own = runs + (size_t)blockIdx.x * nbins;
    __syncthreads();
    constexpr int U = 2, groups = kEbBinThreads / 16;
    for (int b0 = tid / 16; b0 < nbins; b0 += groups * U) {
        uint2 r[U];
        uint32_t end[U], x[U][2];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int b = b0 + u * groups;
            r[u] = b < nbins ? own[b] : make_uint2(0u, 0u);
            end[u] = b + 1 < nbins ? own[b + 1].y : b < nbins ? total : 0u;
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t i = r[u].y + l + 16 * h;
                x[u][h] = i < end[u] ? (uint32_t)labels[r[u].x + (i - r[u].y)] : 0u;
            }
#pragma unroll
        for (int u = 0; u < U; ++u) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t i = r[u].y + l + 16 * h;
                if (i < end[u]) lab[i] = (uint8_t)x[u][h];
            }
            const bool cut = end[u] > r[u].y + kEbLongRun;
            const uint32_t stop = cut ? r[u].y + kEbLongRun : end[u];
            for (uint32_t i = r[u].y + l + 32; i < stop; i += 16) lab[i] = labels[r[u].x + (i - r[u].y)];
            if (cut && l == 0) longs[atomicAdd(&s_long, 1u)] = (uint32_t)(b0 + u * groups);
        }
    }
    uint32_t at[kEbBinPer];
#pragma unroll
    for (int u = 0; u < kEbBinPer; ++u) {
        const int64_t e = lo + u * kEbBinThreads + tid;
        at[u] = e < count ? __builtin_nontemporal_load(places + e) : 0u;
    }
    __syncthreads();
    for (uint32_t j = 0; j < s_long; ++j) {
        const int b = (int)longs[j];
        const uint2 r = own[b];
        const uint32_t end = b + 1 < nbins ? own[b + 1].y : total;
        for (uint32_t i = r.y + kEbLongRun + tid; i < end; i += kEbBinThreads) lab[i] = labels[r.x + (i - r.y)];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEbBinPer; ++u) {
        const int64_t e = lo + u * kEbBinThreads + tid;
        if (e >= count) continue;
        const uint32_t ls = lab[at[u] & 0xFFFFu], ld = lab[at[u] >> 16];
        // (an end without a valid label has been flagged: its key is never used, but stays in range)
        key16[e] = ls < (uint32_t)k && ld < (uint32_t)k ? (uint16_t)(ls * (uint32_t)k + ld) : (uint16_t)0;
    }
}

// H[tile][bucket] from the keys
__global__ __launch_bounds__(kEbBlock) void k_eb_hist_keys(int64_t m, int64_t tile, int32_t k2, const uint16_t* __restrict__ key16,
                                                           uint32_t* __restrict__ H)
{
    extern __shared__ uint32_t hist[];
    for (int b = threadIdx.x; b < k2; b += kEbBlock) hist[b] = 0u;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * tile, hi = lo + tile < m ? lo + tile : m;
    constexpr int U = 8;
    for (int64_t e = lo + threadIdx.x; e < hi; e += kEbBlock * U) {
        uint32_t key[U];
#pragma unroll
        for (int u = 0; u < U; ++u) key[u] = e + u * kEbBlock < hi ? (uint32_t)key16[e + u * kEbBlock] : 0xFFFFFFFFu;
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (key[u] != 0xFFFFFFFFu) atomicAdd(&hist[key[u]], 1u);
    }
    __syncthreads();
    uint32_t* row = H + (size_t)blockIdx.x * (size_t)k2;
    for (int b = threadIdx.x; b < k2; b += kEbBlock) row[b] = hist[b];
}

__global__ __launch_bounds__(kEbBlock) void k_eb_scatter(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                         int64_t m, int64_t tile, const uint16_t* __restrict__ key16,
                                                         int32_t k2, int32_t key_bits, const uint32_t* __restrict__ H,
                                                         int32_t* __restrict__ out_src, int32_t* __restrict__ out_dst)
{
    extern __shared__ uint32_t cur[];
    const uint32_t* row = H + (size_t)blockIdx.x * (size_t)k2;
    for (int b = threadIdx.x; b < k2; b += kEbBlock) cur[b] = row[b];
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u64 below = (1ull << lane) - 1ull;
    const int64_t lo = (int64_t)blockIdx.x * tile, hi = lo + tile < m ? lo + tile : m;
    for (int64_t base = lo; base < hi; base += kEbBlock) {        // uniform trip count over the workgroup
        const int64_t e = base + threadIdx.x;
        const bool valid = e < hi;
        uint32_t key = 0u;
        int32_t s = 0, d = 0;
        if (valid) { key = key16[e]; s = src[e]; d = dst[e]; }
        // lanes of this wave that hold the same key
        u64 same = __ballot(valid);
        for (int bit = 0; bit < key_bits; ++bit) {
            const bool one = (key >> bit) & 1u;
            const u64 b = __ballot(one);
            same &= one ? b : ~b;
        }
        const uint32_t rank = __popcll(same & below);
        uint32_t first = 0u;
        for (int w = 0; w < kEbWaves; ++w) {
            if (wave == w && valid && rank == 0u) {
                first = cur[key];
                cur[key] = first + (uint32_t)__popcll(same);
            }
            __syncthreads();
        }
        const int leader = valid ? __builtin_ctzll(same) : lane;
        const uint32_t pos = __shfl(first, leader) + rank;
        if (valid) { out_src[pos] = s; out_dst[pos] = d; }
    }
}

// The same placement for tiles of 8 edges per thread and at most kEbLdsBuckets buckets, with the tile sorted
// in LDS first so that the output is written in whole runs: each wave owns 512 edges of the
// tile (consecutive stream positions), counts them, the counts become per-wave cursors into the tile's sorted
// order (bucket, then wave, then stream position = stable), every wave places its edges into LDS without
// waiting for the others, and the sorted tile is written out with consecutive lanes on consecutive
// addresses of a bucket's run; with 1024 threads the sources first, then, through the same LDS, the targets, so that up to k = 30
// two workgroups of sixteen waves stand on a CU (their 64 registers leave 44 bytes per lane in scratch).  Bound by the runs,
// pieces of the output of 128 bytes at 256 buckets: with tiles of 4,096 edges and runs of 64 bytes 1.6e9 edges took 9.3 to 12 ms
// in some processes and 14.3 to 18 in others (the same within one), with 8,192 10.6 to 11.0; a form of 36 registers, with the same
// loads and stores, that spills nothing took 13.8 (its cause was not found).  Shorter lists, which the caches hold, want both
// ends at once (a list whose whole call takes 416 us took 438 with turns for them).
constexpr int kEbLdsBuckets = 1024;
constexpr int kEbTurns = 8;                             // edges per thread
template <int THREADS> constexpr int kEbScatterTile = THREADS * kEbTurns;
template <int THREADS> constexpr bool kEbTurnsForEnds = THREADS == 1024;
template <int THREADS> constexpr size_t eb_scatter_lds_bytes(int32_t k2)
{
    return (size_t)kEbScatterTile<THREADS> * (kEbTurnsForEnds<THREADS> ? 6 : 10) + (size_t)k2 * (4 + 2 * (THREADS / 64)) + 16;
}

template <int THREADS>
__global__ __launch_bounds__(THREADS, kEbTurnsForEnds<THREADS> ? 8 : 1) void k_eb_scatter_lds(const int32_t* __restrict__ src, const int32_t* __restrict__ dst,
                                                               int64_t m, const uint16_t* __restrict__ key16, int32_t k2,
                                                               int32_t key_bits, const uint32_t* __restrict__ H,
                                                               int32_t* __restrict__ out_src, int32_t* __restrict__ out_dst)
{
    constexpr int kTile = kEbScatterTile<THREADS>, kWaves = THREADS / 64, kSeg = 64 * kEbTurns;
    constexpr bool kTurns = kEbTurnsForEnds<THREADS>;
    extern __shared__ uint32_t lds[];
    int32_t* ends = (int32_t*)lds;                          // kTile
    int32_t* others = kTurns ? ends : ends + kTile;         // kTile
    uint32_t* delta = (uint32_t*)(others + kTile);          // k2: output position of a bucket's edge less that in the sorted tile
    uint16_t* curw = (uint16_t*)(delta + k2);               // kWaves * k2: counts, then cursors, per wave
    uint16_t* skey = curw + kWaves * k2;                    // kTile
    __shared__ uint32_t wsum[kWaves];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t lo = (int64_t)blockIdx.x * kTile, hi = lo + kTile < m ? lo + kTile : m;
    const int count = (int)(hi - lo);
    const uint32_t* row = H + (size_t)blockIdx.x * (size_t)k2;
    // the wave's edges, kEbTurns per lane: the keys first; where the ends take turns, the sources while the counts are added up
    // and the targets while the sources are written (all of them at once spilled more)
    const int seg0 = wave * kSeg, seg1 = seg0 + kSeg < count ? seg0 + kSeg : count;
    uint32_t key[kEbTurns];
    int32_t s[kEbTurns], d[kEbTurns];
    auto load = [&](const int32_t* __restrict__ from, int32_t (&to)[kEbTurns]) {
#pragma unroll
        for (int u = 0; u < kEbTurns; ++u) {
            const int p = seg0 + u * 64 + lane;
            to[u] = p < seg1 ? __builtin_nontemporal_load(from + lo + p) : 0;
        }
    };
#pragma unroll
    for (int u = 0; u < kEbTurns; ++u) {
        const int p = seg0 + u * 64 + lane;
        key[u] = p < seg1 ? (uint32_t)key16[lo + p] : 0u;
    }
    if (!kTurns) { load(src, s); load(dst, d); }
    for (int b = tid; b < k2; b += THREADS) delta[b] = row[b];
    for (int b = tid; b < kWaves * k2; b += THREADS) curw[b] = 0;
    __syncthreads();
    // counts of the wave's edges: the first lane of those with equal keys adds them up (a wave's own row of curw: no
    // atomics; the ranks inside the 64 are kept for the placement)
    uint16_t* mine = curw + wave * k2;
    const u64 below = (1ull << lane) - 1ull;
    uint32_t rank[kEbTurns];                                // rank | number of equal keys << 8 | first such lane << 16
#pragma unroll
    for (int u = 0; u < kEbTurns; ++u) {
        const bool valid = seg0 + u * 64 + lane < seg1;
        u64 same = __ballot(valid);
        for (int bit = 0; bit < key_bits; ++bit) {
            const bool one = (key[u] >> bit) & 1u;
            const u64 b = __ballot(one);
            same &= one ? b : ~b;
        }
        const uint32_t r = (uint32_t)__popcll(same & below), n = (uint32_t)__popcll(same);
        rank[u] = r | (n << 8) | ((uint32_t)(valid ? __builtin_ctzll(same) : lane) << 16);
        if (valid && r == 0u) mine[key[u]] = (uint16_t)(mine[key[u]] + n);
    }
    if (kTurns) load(src, s);
    __syncthreads();
    // exclusive sums over (bucket, wave): a thread owns up to kEbLdsBuckets / THREADS consecutive buckets
    const int per = (k2 + THREADS - 1) / THREADS;
    const int b0 = tid * per, b1 = b0 + per < k2 ? b0 + per : k2;
    uint32_t own = 0;
    for (int b = b0; b < b1; ++b)
#pragma unroll
        for (int w = 0; w < kWaves; ++w) own += curw[w * k2 + b];
    uint32_t incl = own;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t y = __shfl_up(incl, o);
        if (lane >= o) incl += y;
    }
    if (lane == 63) wsum[wave] = incl;
    __syncthreads();
    uint32_t run = incl - own;
    for (int w = 0; w < wave; ++w) run += wsum[w];
    for (int b = b0; b < b1; ++b) {
        delta[b] -= run;
#pragma unroll
        for (int w = 0; w < kWaves; ++w) { const uint32_t c = curw[w * k2 + b]; curw[w * k2 + b] = (uint16_t)run; run += c; }
    }
    __syncthreads();
    // every wave places its edges, 64 at a time in stream order
#pragma unroll
    for (int u = 0; u < kEbTurns; ++u) {
        const bool valid = seg0 + u * 64 + lane < seg1;
        const uint32_t r = rank[u] & 0xFFu, n = (rank[u] >> 8) & 0xFFu;
        uint32_t first = 0u;
        if (valid && r == 0u) { first = mine[key[u]]; mine[key[u]] = (uint16_t)(first + n); }
        rank[u] = __shfl(first, (int)(rank[u] >> 16)) + r;  // from here on the place
        if (valid) { ends[rank[u]] = s[u]; skey[rank[u]] = (uint16_t)key[u]; }
        if (valid && !kTurns) others[rank[u]] = d[u];
    }
    if (kTurns) load(dst, d);
    __syncthreads();
    uint32_t at[kEbTurns];
#pragma unroll
    for (int u = 0; u < kEbTurns; ++u) {
        const int p = u * THREADS + tid;
        at[u] = p < count ? delta[skey[p]] + (uint32_t)p : 0u;
        if (p < count) out_src[at[u]] = ends[p];
        if (p < count && !kTurns) out_dst[at[u]] = others[p];
    }
    if (!kTurns) return;
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEbTurns; ++u)
        if (seg0 + u * 64 + lane < seg1) ends[rank[u]] = d[u];
    __syncthreads();
#pragma unroll
    for (int u = 0; u < kEbTurns; ++u) {
        const int p = u * THREADS + tid;
        if (p < count) out_dst[at[u]] = ends[p];
    }
}

inline size_t eb_align(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace

extern "C" int grem_edge_buckets(const int32_t* src, const int32_t* dst, int64_t m, int64_t n,
                                 const int32_t* labels, int32_t k, int32_t* out_src, int32_t* out_dst,
                                 int64_t* bucket_offsets, void* stream_)
{
    if (!src || !dst || !labels || !out_src || !out_dst || !bucket_offsets || m < 1 || m > (int64_t)0xFFFFFFFFll ||
        n < 1 || n > INT32_MAX || k < 1 || k > kEbMaxK)
        return GREM_ERR_ARG;
    hipStream_t stream = (hipStream_t)stream_;
    const int32_t k2 = k * k;
    int64_t tile = (m * k2 + kEbMaxCells - 1) / kEbMaxCells;
    const int64_t least = eb_wide(m, k2) ? kEbScatterTile<1024> : kEbScatterTile<512>;
    if (tile < least) tile = least;
    tile = (tile + kEbBlock - 1) / kEbBlock * kEbBlock;
    const int64_t tiles = (m + tile - 1) / tile;
    int32_t S = 65536 / k2;
    if (S < 1) S = 1;
    if (S > tiles) S = (int32_t)tiles;
    const int64_t seg_len = (tiles + S - 1) / S;
    int key_bits = 0;
    while ((1 << key_bits) < k2) ++key_bits;

    size_t off = 0;
    auto carve = [&](size_t bytes) { const size_t at = off; off += eb_align(bytes); return at; };
    const size_t o_flags = carve(256), o_l8 = carve((size_t)n), o_key = carve((size_t)m * 2);
    const size_t o_h = carve((size_t)tiles * k2 * 4), o_part = carve((size_t)k2 * S * 4);
    // the binned look-ups, where the label table outgrows the L2 and a bin's labels fit LDS; without the memory for their
    // lists the look-ups go to the table
    const int cb = n <= (int64_t)kEbBins << 16 ? 16 : 17;
    const bool pack = k <= 16, small_item = cb == 16;      // (16 bits hold the place in a bin of 2^16 nodes)
    bool binned = n >= kEbBinMinN && m >= kEbBinMinM && n <= (int64_t)kEbBins << 17 && n * m >= kEbBinMinNM;
    const int nbins = (int)((n + (1ll << cb) - 1) >> cb);
    // edges per batch: their lists, places and labels take 5 or 7 bytes per end (16M edges of 14M nodes: 5.8 ms for 200M
    // edges instead of 6.0 with 33M; 33M of 111M nodes: 50.2 ms for 1.6e9 instead of 52.4 with 16M)
    const int64_t most = small_item ? (int64_t)1 << 24 : (int64_t)1 << 25, batch = m < most ? m : most, batches = (m + batch - 1) / batch;
    const int64_t bin_tiles = (batch + kEbBinTile - 1) / kEbBinTile;
    const size_t plain_off = off;
    const size_t o_table = carve((size_t)batches * (kEbBins + 1) * 4), o_parts = carve((size_t)batches * (kEbBins + 1) * 4), o_cursors = carve((size_t)batches * kEbBins * 4);
    const size_t o_lists = carve((size_t)batch * 2 * (small_item ? 2 : 4)), o_labels = carve((size_t)batch * 2 + 4);
    const size_t o_runs = carve((size_t)bin_tiles * nbins * 8), o_places = carve((size_t)batch * 4);
    uint8_t* ws = nullptr;
    if (binned && hipMallocAsync((void**)&ws, off, stream) != hipSuccess) { (void)hipGetLastError(); binned = false; ws = nullptr; }
    if (!binned && hipMallocAsync((void**)&ws, plain_off, stream) != hipSuccess) { (void)hipGetLastError(); return GREM_ERR_NOMEM; }
    auto fail = [&](int code) { (void)hipGetLastError(); (void)hipStreamSynchronize(stream); (void)hipFreeAsync(ws, stream); return code; };
    uint32_t* flags = (uint32_t*)(ws + o_flags);
    uint8_t* L8 = ws + o_l8;
    uint16_t* key16 = (uint16_t*)(ws + o_key);
    uint32_t* H = (uint32_t*)(ws + o_h);
    uint32_t* partial = (uint32_t*)(ws + o_part);
    const size_t lds = (size_t)k2 * 4;
    // (the limits are the process's: always what any call may need)
    if (lds > 48 * 1024) {
        constexpr int most = kEbMaxK * kEbMaxK * 4;
        if (hipFuncSetAttribute((const void*)k_eb_hist, hipFuncAttributeMaxDynamicSharedMemorySize, most) != hipSuccess ||
            hipFuncSetAttribute((const void*)k_eb_hist_keys, hipFuncAttributeMaxDynamicSharedMemorySize, most) != hipSuccess ||
            hipFuncSetAttribute((const void*)k_eb_scatter, hipFuncAttributeMaxDynamicSharedMemorySize, most) != hipSuccess)
            return fail(GREM_ERR_HIP);
    }
    auto grid = [](int64_t items, int64_t cap) { int64_t g = (items + 255) / 256; if (g < 1) g = 1; if (g > cap) g = cap; return (int)g; };
    hipLaunchKernelGGL(k_eb_zero, dim3(1), dim3(256), 0, stream, flags, (size_t)64);
    uint32_t host_flags[2] = {0, 0};
    hipLaunchKernelGGL(k_eb_compact, dim3(grid(n, 16384)), dim3(256), 0, stream, n, labels, k, L8, flags + 2);
    if (binned) {
        uint32_t *table = (uint32_t*)(ws + o_table), *part_rows = (uint32_t*)(ws + o_parts), *cursors = (uint32_t*)(ws + o_cursors), *places = (uint32_t*)(ws + o_places);
        uint8_t* found = ws + o_labels;
        uint2* runs = (uint2*)(ws + o_runs);
        const size_t items_lds = (size_t)kEbBinTile * 8, tab_lds = pack ? (size_t)1 << (cb - 1) : (size_t)1 << cb;
        const int parts = nbins * (nbins >= 1024 ? 1 : (1024 + nbins - 1) / nbins);
        hipLaunchKernelGGL(k_eb_zero, dim3(256), dim3(256), 0, stream, table, (size_t)batches * (kEbBins + 1));
        hipLaunchKernelGGL(k_eb_bin_count, dim3((unsigned)((bin_tiles + 7) / 8), (unsigned)batches), dim3(kEbBinThreads), 0, stream, src, dst, m, batch,
                           (uint32_t)n, cb, table, flags);
        hipLaunchKernelGGL(k_eb_bin_scan, dim3((unsigned)batches), dim3(kEbBins), 0, stream, table, cursors, part_rows, (uint32_t)parts);
        auto run = [&](auto item, auto packed) {
            using Item = decltype(item);
            constexpr bool PACK = decltype(packed)::value;
            if (hipFuncSetAttribute((const void*)k_eb_bin<Item>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)items_lds) != hipSuccess ||
                hipFuncSetAttribute((const void*)k_eb_lookup<Item, PACK>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)tab_lds) != hipSuccess)
                return false;
            Item* lists = (Item*)(ws + o_lists);
            for (int64_t i = 0; i < batches; ++i) {
                const int64_t lo = i * batch, count = m - lo < batch ? m - lo : batch;
                const unsigned tiles_now = (unsigned)((count + kEbBinTile - 1) / kEbBinTile);
                const uint32_t* prow = part_rows + (size_t)i * (kEbBins + 1);
                hipLaunchKernelGGL((k_eb_bin<Item>), dim3(tiles_now), dim3(kEbBinThreads), items_lds, stream, src + lo, dst + lo, count,
                                   (uint32_t)n, cb, nbins, prow, cursors + (size_t)i * kEbBins, lists, runs, places);
                hipLaunchKernelGGL((k_eb_lookup<Item, PACK>), dim3((unsigned)(parts + nbins)), dim3(kEbBinThreads), tab_lds, stream,
                                   (const uint8_t*)L8, n, cb, prow, (const uint32_t*)(table + (size_t)i * (kEbBins + 1)), (const Item*)lists,
                                   found, (const uint32_t*)(flags + 2), flags);
                hipLaunchKernelGGL(k_eb_keys, dim3(tiles_now), dim3(kEbBinThreads), 0, stream, src + lo, dst + lo, count, (uint32_t)n,
                                   (const uint8_t*)L8, nbins, k, prow, (const uint2*)runs, (const uint32_t*)places, (const uint8_t*)found,
                                   key16 + lo, flags);
            }
            return true;
        };
        bool ok;
        if (small_item) ok = pack ? run(uint16_t{}, std::true_type{}) : run(uint16_t{}, std::false_type{});
        else ok = pack ? run(uint32_t{}, std::true_type{}) : run(uint32_t{}, std::false_type{});
        if (!ok) return fail(GREM_ERR_HIP);
        hipLaunchKernelGGL(k_eb_hist_keys, dim3((unsigned)tiles), dim3(kEbBlock), lds, stream, m, tile, k2, (const uint16_t*)key16, H);
    } else {
        hipLaunchKernelGGL(k_eb_hist, dim3((unsigned)tiles), dim3(kEbBlock), lds, stream, src, dst, m, (uint32_t)n, tile, L8, k, key16, H,
                           flags);
    }
    if (hipMemcpyAsync(host_flags, flags, sizeof(host_flags), hipMemcpyDeviceToHost, stream) != hipSuccess ||
        hipStreamSynchronize(stream) != hipSuccess)
        return fail(GREM_ERR_HIP);
    if (host_flags[0] || host_flags[1]) return fail(GREM_ERR_ARG);
    const int64_t cells = (int64_t)k2 * S;
    hipLaunchKernelGGL(k_eb_colsum, dim3(grid(cells, 1 << 20)), dim3(256), 0, stream, H, tiles, k2, S, seg_len, partial);
    hipLaunchKernelGGL(k_eb_bases, dim3(1), dim3(1024), 0, stream, partial, cells, k2, S, m, bucket_offsets);
    hipLaunchKernelGGL(k_eb_colscan, dim3(grid(cells, 1 << 20)), dim3(256), 0, stream, H, tiles, k2, S, seg_len, partial);
    if (tile == least && k2 <= kEbLdsBuckets) {
        auto scatter = [&](auto kernel, int threads, size_t lds2, size_t most_lds) {
            if (hipFuncSetAttribute((const void*)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most_lds) != hipSuccess) return false;
            hipLaunchKernelGGL(kernel, dim3((unsigned)tiles), dim3(threads), lds2, stream, src, dst, m, key16, k2, key_bits, H, out_src, out_dst);
            return true;
        };
        if (!(least == kEbScatterTile<1024> ? scatter(k_eb_scatter_lds<1024>, 1024, eb_scatter_lds_bytes<1024>(k2), eb_scatter_lds_bytes<1024>(kEbLdsBuckets))
                                            : scatter(k_eb_scatter_lds<512>, 512, eb_scatter_lds_bytes<512>(k2), eb_scatter_lds_bytes<512>(kEbLdsBuckets))))
            return fail(GREM_ERR_HIP);
    } else {
        hipLaunchKernelGGL(k_eb_scatter, dim3((unsigned)tiles), dim3(kEbBlock), lds, stream, src, dst, m, tile, key16, k2, key_bits, H,
                           out_src, out_dst);
    }
    int rc = hipGetLastError() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
    if (hipFreeAsync(ws, stream) != hipSuccess) rc = GREM_ERR_HIP;
    return rc;
}
