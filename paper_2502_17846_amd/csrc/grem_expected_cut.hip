// Expected number of edge cuts of fixed greedy decisions made from a fraction x of the edges, for gfx950
// (Armada paper, Sec. 4.2, Eq. (1)): for a two-way labelling, node i has k_i labelled neighbours, k0_i of
// them in the partition that holds more; with d_i = floor(k_i x + 0.5) of its edges in hand the greedy
// decision is wrong with probability q_i = Pr(K < d_i / 2), K ~ Hypergeometric(k_i, k0_i, d_i), and
//   E[C] = sum_i (k_i - k0_i) (1 - q_i) + k0_i q_i.
// Refinement over two chunks is the same expression at 2x (Sec. 4.2, "The Benefit of Refinement").
//
// A workgroup takes tiles of 256 nodes in turn: it walks their CSR entries edge-parallel, counts the labels
// per node, and then every thread sums the tail of one node's distribution term by term: in the log domain
// (first term from lgamma, the following ones by the ratio of consecutive probabilities), or, for a node with
// few draws, as plain products of ratios.  A workgroup's sum runs over its tiles in order, and one workgroup
// adds the workgroups' sums in a fixed order, so the result is reproducible.
#include <hip/hip_runtime.h>

#include <cstdint>
#include <mutex>

#include "grem.h"

// Per-workgroup partial sums and the packed labels of the entry point that allocates nothing
// (grem_expected_cut_noalloc).  One copy per GPU, held until the process ends; host code reaches it only through the address
// hipGetSymbolAddress returns for the current device, never through this name.
constexpr int64_t kXcStaticBlocks = 262144;        // 4 MiB
constexpr int64_t kXcStaticMaxN = 4194304;         // their labels, two bits each, take 1 MiB of it
static __device__ __align__(256) double scratch[2 * kXcStaticBlocks];

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

// What bounds the walk is the look-up of every entry's label: a table larger than an XCD's 4 MB of L2 serves
// 57 to 121 G/s, a smaller one 267 G/s.  Only three kinds of label count (0, 1, any other), so they are
// packed two bits each first, a sixteenth of the int32 table: 16.7M nodes fit the L2.
//
// FUSED: the terms are summed here as well, as the entry point without allocations needs it.  The tail's code takes
// 220 registers, and the two waves per SIMD that they leave cannot keep enough look-ups in flight; the other form
// writes the counts (8 bytes per node) for k_xc_terms_counts, which maps nodes to threads in the same way, so that
// every sum has the same order.  13,875,000 nodes, 400M entries: 6.16 ms from the int32 table with sixteen lanes per
// row, 5.3 ms fused, 2.19 + 0.68 ms as two kernels.
__global__ __launch_bounds__(kXcBlock) void k_xc_pack(const int32_t* __restrict__ labels, int64_t n, uint32_t* __restrict__ words)
{
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

constexpr int kXcTile = kXcBlock;                  // nodes per workgroup and turn
// workgroups: all of them resident (eight per CU), a contiguous range of tiles each; a constant, so that the
// order of the sums does not depend on the device
constexpr int64_t kXcGrid = 2048;

// the range of tiles that workgroup b of `blocks` owns
__device__ __forceinline__ int64_t xc_first_tile(int64_t tiles, int64_t blocks, int64_t b)
{
    const int64_t each = tiles / blocks, more = tiles % blocks;
    return b * each + (b < more ? b : more);
}

__device__ __forceinline__ void xc_block_sums(double ec, double base, double* partial_ec, double* partial_base)
{
    __shared__ double s_ec[kXcBlock / 64], s_base[kXcBlock / 64];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { ec += __shfl_down(ec, o); base += __shfl_down(base, o); }
    if ((threadIdx.x & 63) == 0) { s_ec[threadIdx.x >> 6] = ec; s_base[threadIdx.x >> 6] = base; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0.0, b = 0.0;
        for (int q = 0; q < kXcBlock / 64; ++q) { a += s_ec[q]; b += s_base[q]; }
        partial_ec[blockIdx.x] = a; partial_base[blockIdx.x] = b;
    }
}

template <typename RowT, bool FUSED>
__global__ __launch_bounds__(kXcBlock) void k_xc_terms(const RowT* __restrict__ rowptr, const int32_t* __restrict__ colidx,
                                                       int64_t n, const uint32_t* __restrict__ words, double x,
                                                       uint2* __restrict__ counts, double* partial_ec, double* partial_base)
{
    constexpr int U = 8;                           // entries in flight per thread
    __shared__ uint32_t rowrel[kXcTile + 1];
    __shared__ uint32_t cnt[2][kXcTile];
    const int tid = threadIdx.x, lane = tid & 63;
    const int64_t tiles = (n + kXcTile - 1) / kXcTile;
    const int64_t t1 = xc_first_tile(tiles, gridDim.x, (int64_t)blockIdx.x + 1);
    double ec_sum = 0.0, base_sum = 0.0;
    for (int64_t tile = xc_first_tile(tiles, gridDim.x, blockIdx.x); tile < t1; ++tile) {
        const int64_t v0 = tile * kXcTile;
        const int nv = n - v0 < kXcTile ? (int)(n - v0) : kXcTile;
        const int64_t e0 = (int64_t)rowptr[v0], ne = (int64_t)rowptr[v0 + nv] - e0;
        // (the threads' own counts of the tile before are read: no barrier needed before they are cleared)
        cnt[0][tid] = 0; cnt[1][tid] = 0;
        // pieces of fewer than 2^31 entries, so that 32 bits hold the offsets whatever the rows' lengths
        for (int64_t p0 = 0; p0 < ne; p0 += (int64_t)1 << 30) {
            const uint32_t end = (uint32_t)(ne - p0 < ((int64_t)1 << 30) ? ne - p0 : ((int64_t)1 << 30));
            __syncthreads();
            for (int i = tid; i <= kXcTile; i += kXcBlock) {
                const int64_t off = (int64_t)rowptr[v0 + (i < nv ? i : nv)] - e0 - p0;
                rowrel[i] = off < 0 ? 0u : off > (int64_t)end ? end : (uint32_t)off;
            }
            __syncthreads();
            const int32_t* cbase = colidx + e0 + p0;
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
        }
        __syncthreads();
        if constexpr (FUSED) {
            double ec = 0.0, base = 0.0;
            if (tid < nv) xc_node_terms(cnt[0][tid], cnt[1][tid], x, &ec, &base);
            ec_sum += ec; base_sum += base;
        } else {
            if (tid < nv) counts[v0 + tid] = make_uint2(cnt[0][tid], cnt[1][tid]);
        }
    }
    if constexpr (FUSED) xc_block_sums(ec_sum, base_sum, partial_ec, partial_base);
}

// The same terms from neighbour counts that are at hand (counts[2 v], counts[2 v + 1]: the labelled
// neighbours of node v in partition 0 and 1), one lane per node.
__global__ __launch_bounds__(kXcBlock) void k_xc_terms_counts(const uint32_t* __restrict__ counts, int64_t n, double x,
                                                              double* partial_ec, double* partial_base)
{
    const int64_t tiles = (n + kXcTile - 1) / kXcTile;
    const int64_t t1 = xc_first_tile(tiles, gridDim.x, (int64_t)blockIdx.x + 1);
    double ec_sum = 0.0, base_sum = 0.0;
    for (int64_t tile = xc_first_tile(tiles, gridDim.x, blockIdx.x); tile < t1; ++tile) {
        const int64_t v = tile * kXcTile + threadIdx.x;
        double ec = 0.0, base = 0.0;
        if (v < n) {
            const uint2 c = *reinterpret_cast<const uint2*>(counts + 2 * v);
            xc_node_terms(c.x, c.y, x, &ec, &base);
        }
        ec_sum += ec; base_sum += base;
    }
    xc_block_sums(ec_sum, base_sum, partial_ec, partial_base);
}

__global__ __launch_bounds__(1024) void k_xc_total(const double* __restrict__ partial_ec, const double* __restrict__ partial_base,
                                                   int64_t blocks, double* out)
{
    __shared__ double s_ec[16], s_base[16];
    double a = 0.0, b = 0.0;
    for (int64_t i = threadIdx.x; i < blocks; i += 1024) { a += partial_ec[i]; b += partial_base[i]; }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) { a += __shfl_down(a, o); b += __shfl_down(b, o); }
    if ((threadIdx.x & 63) == 0) { s_ec[threadIdx.x >> 6] = a; s_base[threadIdx.x >> 6] = b; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double x = 0.0, y = 0.0;
        for (int q = 0; q < 16; ++q) { x += s_ec[q]; y += s_base[q]; }
        out[0] = x; out[1] = y;
    }
}

inline int64_t xc_blocks(int64_t n)
{
    const int64_t tiles = (n + kXcTile - 1) / kXcTile;
    return tiles < kXcGrid ? tiles : kXcGrid;
}

// scratch: the workgroups' sums, then the packed labels; the counts, 8-byte aligned, if there is room for them
inline size_t xc_scratch_bytes(int64_t n)
{
    return (size_t)kXcGrid * 2 * sizeof(double) + ((size_t)((n + 15) / 16) * sizeof(uint32_t) + 7) / 8 * 8;
}
static_assert(kXcGrid * 2 * 8 + kXcStaticMaxN / 16 * 4 <= kXcStaticBlocks * 16, "the fixed buffer holds the largest input");

template <typename RowT>
void xc_launch(const void* rowptr, const int32_t* colidx, int64_t n, const int32_t* labels, double x, double* scratch_mem,
               bool counts_fit, double* out, hipStream_t stream)
{
    const int64_t blocks = xc_blocks(n);
    double* partial = scratch_mem;
    uint32_t* words = (uint32_t*)(scratch_mem + 2 * kXcGrid);
    const int64_t pack = ((n + 15) / 16 + kXcBlock - 1) / kXcBlock;
    hipLaunchKernelGGL(k_xc_pack, dim3((unsigned)(pack < 4096 ? pack : 4096)), dim3(kXcBlock), 0, stream, labels, n, words);
    if (counts_fit) {
        uint2* counts = (uint2*)((char*)scratch_mem + xc_scratch_bytes(n));
        hipLaunchKernelGGL((k_xc_terms<RowT, false>), dim3((unsigned)blocks), dim3(kXcBlock), 0, stream, (const RowT*)rowptr,
                           colidx, n, (const uint32_t*)words, x, counts, partial, partial + blocks);
        hipLaunchKernelGGL(k_xc_terms_counts, dim3((unsigned)blocks), dim3(kXcBlock), 0, stream, (const uint32_t*)counts, n, x,
                           partial, partial + blocks);
    } else {
        hipLaunchKernelGGL((k_xc_terms<RowT, true>), dim3((unsigned)blocks), dim3(kXcBlock), 0, stream, (const RowT*)rowptr,
                           colidx, n, (const uint32_t*)words, x, (uint2*)nullptr, partial, partial + blocks);
    }
    hipLaunchKernelGGL(k_xc_total, dim3(1), dim3(1024), 0, stream, partial, partial + blocks, blocks, out);
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
    // every workgroup writes its own two slots, the packed labels are written in full, and the kernels read
    // exactly those: nothing has to start at zero, whatever an earlier call left behind
    hipStream_t stream = (hipStream_t)stream_;
    if (rowptr_bits == 64) xc_launch<int64_t>(rowptr, colidx, n, labels, x, partial, false, out, stream);
    else xc_launch<int32_t>(rowptr, colidx, n, labels, x, partial, false, out, stream);
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
    if (hipMallocAsync((void**)&partial, xc_scratch_bytes(n) + (size_t)n * sizeof(uint2), stream) != hipSuccess) {
        (void)hipGetLastError();
        counts_fit = false;
        if (hipMallocAsync((void**)&partial, xc_scratch_bytes(n), stream) != hipSuccess) {
            (void)hipGetLastError();
            return GREM_ERR_NOMEM;
        }
    }
    if (rowptr_bits == 64) xc_launch<int64_t>(rowptr, colidx, n, labels, x, partial, counts_fit, out, stream);
    else xc_launch<int32_t>(rowptr, colidx, n, labels, x, partial, counts_fit, out, stream);
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
    const int64_t blocks = xc_blocks(n);
    uint32_t* counts = nullptr;
    double* partial = nullptr;
    if (hipMallocAsync((void**)&counts, (size_t)n * 2 * sizeof(uint32_t), stream) != hipSuccess) {
        (void)hipGetLastError();
        return GREM_ERR_NOMEM;
    }
    if (hipMallocAsync((void**)&partial, (size_t)blocks * 2 * sizeof(double), stream) != hipSuccess) {
        (void)hipGetLastError();
        (void)hipFreeAsync(counts, stream);
        return GREM_ERR_NOMEM;
    }
    int rc = grem_plan_neighbour_counts(plan, 2, labels, counts, stream);
    if (rc == GREM_OK) {
        hipLaunchKernelGGL(k_xc_terms_counts, dim3((unsigned)blocks), dim3(kXcBlock), 0, stream, (const uint32_t*)counts, n, x,
                           partial, partial + blocks);
        hipLaunchKernelGGL(k_xc_total, dim3(1), dim3(1024), 0, stream, partial, partial + blocks, blocks, out);
        if (hipGetLastError() != hipSuccess) rc = GREM_ERR_HIP;
    }
    if (hipFreeAsync(partial, stream) != hipSuccess) rc = rc == GREM_OK ? GREM_ERR_HIP : rc;
    if (hipFreeAsync(counts, stream) != hipSuccess) rc = rc == GREM_OK ? GREM_ERR_HIP : rc;
    return rc;
}
