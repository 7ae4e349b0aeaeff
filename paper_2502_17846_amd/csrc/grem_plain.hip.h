// The plain route in two launches per chunk (three in the first pass), for k <= 1024 and chunks of at most
// kPlainTiles admission tiles:
//   k_score_tile   counts, blends and proposes (Alg. 2 cnt_nbrs, Alg. 1 blend, Alg. 2 assign) for tiles of rows
//                  and, in the same launch, for the parts of the chunk's long rows; adds the movers up per
//                  admission tile and per kPlainCoarse of them
//   k_admit_tiles  admits by rank, relabels, adds to the sizes (Alg. 2 fix_sizes): every workgroup adds up the counts
//                  of the earlier tiles itself
//   k_spill_tiles  (first pass) places the rejected new vertices (Alg. 2 arg_min fallback)
// The sizes live in two copies: the score kernel copies the current one, the admission reads it and adds to the other;
// the mover counts live in two tables that take turns from chunk to chunk, each cleared while the other is in use.
//
// On graphs that the caches hold, launches and the latency inside each of them are what the time goes to: with
// count, scan and apply in launches of their own, rows of 16,384 entries on one workgroup and tiles of 256 rows
// (one workgroup of four waves per CU in a chunk of 65,536 rows), a run on 1,048,576 vertices and 31M entries
// (k = 8, 48 chunk steps) took 5.0 ms, one on 10,000 vertices (30 steps) 0.77 ms, one on 16.8M vertices with 64 rows
// of 2M entries (k = 256, 256 steps) 107 ms; now 1.9, 0.40 and 68 ms.
#pragma once
#include "grem_kernels.hip.h"

namespace grem {

constexpr int kPlainTiles = 1024;        // most admission tiles of a chunk
constexpr int kPlainMaxK = 1024;
constexpr int kPlainCoarse = 8;          // admission tiles per row of the coarse table
constexpr int kLongClasses = 16;         // rows of at least degree * 2^i entries, i = 0 .. 15, counted by the prepass

// The long rows of a chunk: rows of at least `degree` entries are left out of their tile; their entries are dealt
// out in parts of `part`, each a workgroup of its own.  Row i of the list has the parts pref[i] .. pref[i + 1) of the
// chunk (the last row's end at `parts`); the workgroup that finishes a row's last part picks its proposal, or, with more
// than kLongTicketParts of them, k_long_pick in a launch of its own: finding out who is last takes a write-back of the L2
// per part (3000 parts: 0.5 ms a chunk step, where a launch takes some 5 us).
constexpr uint32_t kLongTicketParts = 64;
struct LongParts {
    const uint32_t *row;
    const uint32_t *pref;
    uint32_t *ticket;                    // parts done, 0 between chunks; null: k_long_pick follows
    uint32_t rows, parts, degree, part;
};

// how many long rows and parts every chunk has
template <typename RowT>
__global__ __launch_bounds__(256) void k_long_count(const RowT *__restrict__ rowptr, int64_t n, int64_t chunk,
                                                    uint32_t degree, uint32_t part, uint32_t *__restrict__ nrows,
                                                    uint32_t *__restrict__ nparts) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const unsigned long long d = (unsigned long long)(rowptr[v + 1] - rowptr[v]);
        if (d >= degree) {
            atomicAdd(&nrows[v / chunk], 1u);
            atomicAdd(&nparts[v / chunk], (uint32_t)((d + part - 1) / part));
        }
    }
}

// their list, chunk by chunk (off: first place of a chunk; cur: zero before), in any order inside a chunk
template <typename RowT>
__global__ __launch_bounds__(256) void k_long_list(const RowT *__restrict__ rowptr, int64_t n, int64_t chunk,
                                                   uint32_t degree, const uint32_t *__restrict__ off,
                                                   uint32_t *__restrict__ cur, uint32_t *__restrict__ row,
                                                   uint32_t *__restrict__ ticket) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t v = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; v < n; v += stride) {
        const unsigned long long d = (unsigned long long)(rowptr[v + 1] - rowptr[v]);
        if (d >= degree) {
            const int64_t c = v / chunk;
            const uint32_t at = off[c] + atomicAdd(&cur[c], 1u);
            row[at] = (uint32_t)v;
            ticket[at] = 0u;
        }
    }
}

// one workgroup: exclusive prefix of nrows over the chunks
__global__ __launch_bounds__(kScanThreads) void k_long_offsets(const uint32_t *__restrict__ nrows, int64_t nchunks,
                                                               uint32_t *__restrict__ off) {
    __shared__ long long wave_total[kScanThreads / 64];
    __shared__ uint32_t s_carry;
    uint32_t carry = 0;
    for (int64_t base = 0; base < nchunks; base += kScanThreads) {
        const int64_t i = base + threadIdx.x;
        const uint32_t x = i < nchunks ? nrows[i] : 0u;
        const uint32_t excl = (uint32_t)block_exclusive_sum(x, wave_total);
        if (i < nchunks) off[i] = carry + excl;
        if (threadIdx.x == kScanThreads - 1) s_carry = carry + excl + x;
        __syncthreads();
        carry = s_carry;
    }
}

// one workgroup per chunk (in turn): the rows' first parts
template <typename RowT>
__global__ __launch_bounds__(256) void k_long_parts(const RowT *__restrict__ rowptr, int64_t nchunks, uint32_t part,
                                                    const uint32_t *__restrict__ nrows, const uint32_t *__restrict__ off,
                                                    const uint32_t *__restrict__ row, uint32_t *__restrict__ pref) {
    __shared__ long long wave_total[4];
    __shared__ uint32_t s_carry;
    for (int64_t c = blockIdx.x; c < nchunks; c += gridDim.x) {
        const uint32_t count = nrows[c], first = off[c];
        uint32_t carry = 0;
        for (uint32_t base = 0; base < count; base += 256) {
            const uint32_t i = base + threadIdx.x;
            uint32_t x = 0;
            if (i < count) {
                const int64_t v = (int64_t)row[first + i];
                x = (uint32_t)(((unsigned long long)(rowptr[v + 1] - rowptr[v]) + part - 1) / part);
            }
            const uint32_t excl = (uint32_t)block_exclusive_sum(x, wave_total);
            if (i < count) pref[first + i] = carry + excl;
            if (threadIdx.x == 255) s_carry = carry + excl + x;
            __syncthreads();
            carry = s_carry;
        }
    }
}

// the long rows' estimates start at zero: the parts' counts are added to them
__global__ __launch_bounds__(256) void k_long_clear(const uint32_t *__restrict__ row, uint32_t rows, uint32_t *__restrict__ E,
                                                    int k) {
    const size_t cells = (size_t)rows * (size_t)k, stride = (size_t)gridDim.x * blockDim.x;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < cells; i += stride)
        E[(size_t)row[i / k] * (size_t)k + i % k] = 0u;
}

// best partition with room by (E desc, room desc, id asc) among j = sub, sub + g, ... , then over the g lanes of the
// vertex (g a power of two, at most 64): its id in every lane
template <typename Est>
__device__ __forceinline__ uint32_t best_partition(Est &&est, const uint32_t *room, int k, uint32_t own, int sub, int g) {
    unsigned long long bestkey = 0;
    int bestj = 0x7fffffff;
    for (int j = sub; j < k; j += g) {
        const uint32_t rm = room[j] + ((uint32_t)j == own ? 1u : 0u);
        const unsigned long long key = rm ? (((unsigned long long)est(j) << 32) | rm) : 0ull;
        if (key > bestkey) { bestkey = key; bestj = j; }       // j ascends: first maximum kept
    }
    for (int off = g >> 1; off >= 1; off >>= 1) {
        const unsigned long long okey = __shfl_xor(bestkey, off);
        const int oj = __shfl_xor(bestj, off);
        if (okey > bestkey || (okey == bestkey && oj < bestj)) { bestkey = okey; bestj = oj; }
    }
    return (uint32_t)bestj;
}

// How the chunk's vertices stand before their admission.
constexpr int kAllLabelled = 0;          // refinement
constexpr int kNoneLabelled = 1;         // first pass without a seed (the label array says nothing about them)
constexpr int kSomeLabelled = 2;         // first pass with a seed

// The movers of an admission tile by partition: cnt[tile][t], and, when the chunk has so many cells that the admission's
// workgroups should not all read them, their sums over kPlainCoarse tiles, coarse[tile / kPlainCoarse][t] (else null).
// What these atomics cost is the number of them that meet at one address (some 15 ns each): with 16 tiles to a
// coarse row, and always one, 4096 workgroups of 16 rows took 65 us per chunk step at k = 8 where 2048 of 32 rows took 45;
// four 16-bit counts in one 64-bit atomic were slower, not faster.
constexpr int kPlainCells = 16384;       // tiles * k up to which there is no coarse table
__device__ __forceinline__ void add_movers(uint32_t *cnt, uint32_t *coarse, int k, uint32_t tile, uint32_t t, uint32_t count) {
    atomicAdd(&cnt[(size_t)tile * k + t], count);
    if (coarse) atomicAdd(&coarse[(size_t)(tile / kPlainCoarse) * k + t], count);
}

// A wave picks the proposal of the long row v from its complete estimates est(j); room: P - S.
template <typename LabelT, typename Est>
__device__ __forceinline__ void propose_long(int64_t v, Est &&est, const uint32_t *room, const LabelT *__restrict__ Lc,
                                             LabelT *__restrict__ prop, uint32_t *cnt, uint32_t *coarse, int64_t chunk_lo, int k,
                                             int pass, int standing) {
    const uint32_t none = LabelTraits<LabelT>::kUnassigned;
    const uint32_t old = standing == kNoneLabelled ? 0xFFFFFFFFu : (uint32_t)Lc[v];
    const bool had = standing == kAllLabelled || (standing == kSomeLabelled && old != none);
    uint32_t best = old;
    if (!(pass == 0 && had)) best = best_partition(est, room, k, had ? old : 0xFFFFFFFFu, lane_id(), 64);
    if (lane_id() == 0) {
        prop[v - chunk_lo] = (LabelT)best;
        if (!had || best != old) add_movers(cnt, coarse, k, (uint32_t)((v - chunk_lo) / kAdmitTile), best, 1u);
    }
}

// a wave per long row of the chunk
template <typename LabelT>
__global__ __launch_bounds__(kScoreThreads) void k_long_pick(const uint32_t *__restrict__ row, uint32_t rows,
                                                             const uint32_t *__restrict__ E, const LabelT *__restrict__ Lc,
                                                             const long long *__restrict__ S, LabelT *__restrict__ prop, uint32_t *cnt,
                                                             uint32_t *coarse, int64_t chunk_lo, int k, int pass, long long P,
                                                             int standing) {
    extern __shared__ uint32_t smem[];                      // k
    for (int j = threadIdx.x; j < k; j += kScoreThreads) smem[j] = (uint32_t)(P - S[j]);
    __syncthreads();
    const uint32_t i = blockIdx.x * (kScoreThreads / 64) + (threadIdx.x >> 6);
    if (i >= rows) return;
    const int64_t v = (int64_t)row[i];
    const uint32_t *erow = E + (size_t)v * (size_t)k;
    propose_long(v, [&](int j) { return erow[j]; }, smem, Lc, prop, cnt, coarse, chunk_lo, k, pass, standing);
}

// lane i's word in every lane, 0 for i >= 64 (i uniform over the wave)
__device__ __forceinline__ unsigned long long wave_word(unsigned long long x, int i) {
    const uint32_t lo = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)x, i & 63);
    const uint32_t hi = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(x >> 32), i & 63);
    return i < 64 ? (unsigned long long)hi << 32 | lo : 0ull;
}

// What bounds it: the look-up of every entry's label (a miss of 64 bytes once the labels outgrow the L2) and the
// tile's estimates, read before the counting starts and written once; on small graphs latency, hence tiles small
// enough for 2048 workgroups per chunk and g = 256 / tv lanes per vertex for the proposals.  The last pass keeps the
// estimates to itself unless the caller asked for them (store_e).
constexpr int kEstAhead = 8;             // estimates per thread requested ahead of the counting

// Packed estimates (PACKED; kept by the library, never the caller's): of a tile without long rows only the estimates that
// are not zero are stored, and a bit per cell that says which.  A wave owns up to 16 words of 64 cells; its values stand one
// after the other at the start of its cells' place in E.  A row has no more of them than entries: chunks of 262,144 rows of 47
// entries at k = 256 moved 268 MB of estimates in and out each, and a step of a refinement pass took 270 us; now 196 us, of
// which some 100 are instructions issued (a choice among the non-zero cells alone instead of all 256 gained nothing).

template <typename RowT, typename LabelT, bool PACKED>
__global__ __launch_bounds__(kScoreThreads) void k_score_tile(
    const RowT *__restrict__ rowptr, const int32_t *__restrict__ colidx, const LabelT *__restrict__ Lc,
    const long long *__restrict__ S, long long *__restrict__ Snext, uint32_t *__restrict__ E, LabelT *__restrict__ prop,
    uint32_t *__restrict__ cnt, uint32_t *__restrict__ coarse, int64_t chunk_lo, int64_t chunk_hi, int k, int tv, int pass,
    long long P, int64_t gather_limit, int standing, int store_e, LongParts lr, unsigned long long *__restrict__ bits) {
    extern __shared__ uint32_t smem[];
    __shared__ int s_last;
    constexpr int U = 8;
    const uint32_t none = LabelTraits<LabelT>::kUnassigned;
    const bool check = standing == kSomeLabelled;          // only then may a label that is looked up be missing
    const int tid = threadIdx.x;
    const int sh = pass == 0 ? 0 : pass - 1;

    if (blockIdx.x < lr.parts) {                            // a part of a long row
        uint32_t *hist = smem, *room = smem + k;
        const uint32_t x = blockIdx.x;
        uint32_t a = 0, b = lr.rows;                        // largest row i with pref[i] <= x
        while (b - a > 1) { const uint32_t mid = (a + b) >> 1; if (lr.pref[mid] <= x) a = mid; else b = mid; }
        const int64_t v = (int64_t)lr.row[a];
        const int64_t e0 = (int64_t)rowptr[v];
        const uint32_t deg = (uint32_t)((int64_t)rowptr[v + 1] - e0);
        const uint32_t from = (x - lr.pref[a]) * lr.part, to = deg - from < lr.part ? deg : from + lr.part;
        for (int j = tid; j < k; j += kScoreThreads) { hist[j] = 0; room[j] = (uint32_t)(P - S[j]); }
        __syncthreads();
        const int32_t *cbase = colidx + e0;
        for (uint32_t base = from + tid; base < to; base += kScoreThreads * U) {
            int32_t col[U];
            uint32_t lab[U];
#pragma unroll
            for (int u = 0; u < U; ++u) col[u] = to - base > (uint32_t)(u * kScoreThreads) ? __builtin_nontemporal_load(cbase + base + u * kScoreThreads) : -1;
#pragma unroll
            for (int u = 0; u < U; ++u) lab[u] = col[u] >= 0 && (int64_t)col[u] < gather_limit ? (uint32_t)Lc[col[u]] : 0xFFFFFFFFu;
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (lab[u] != 0xFFFFFFFFu && !(check && lab[u] == none)) atomicAdd(&hist[lab[u]], 1u);
            if (to - base <= (uint32_t)(kScoreThreads * U)) break;
        }
        __syncthreads();
        uint32_t *erow = E + (size_t)v * (size_t)k;
        for (int j = tid; j < k; j += kScoreThreads)
            if (hist[j]) atomicAdd(&erow[j], hist[j] << sh);
        if (!lr.ticket) return;
        // the row's last part to end, whichever it is, sees the others' counts: they are out before their tickets
        __threadfence();
        __syncthreads();
        if (tid == 0) {
            const uint32_t all = (a + 1 < lr.rows ? lr.pref[a + 1] : lr.parts) - lr.pref[a];
            const bool last = atomicAdd(&lr.ticket[a], 1u) + 1u == all;
            if (last) lr.ticket[a] = 0u;
            s_last = last ? 1 : 0;
        }
        __syncthreads();
        if (!s_last || tid >= 64) return;
        __threadfence();
        propose_long(v, [&](int j) { return __hip_atomic_load(erow + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }, room, Lc, prop, cnt,
                     coarse, chunk_lo, k, pass, standing);
        return;
    }

    uint32_t *hist = smem;                      // tv * k
    uint32_t *rowrel = hist + (size_t)tv * k;   // tv + 1
    uint32_t *room = rowrel + tv + 1;           // k
    uint32_t *moved = room + k;                 // k
    const uint32_t tile = blockIdx.x - lr.parts;
    const int64_t v0 = chunk_lo + (int64_t)tile * tv;
    const int64_t left = chunk_hi - v0;
    const int nv = left < tv ? (int)left : tv;
    const int64_t e0 = (int64_t)rowptr[v0];
    const int total = nv * k;
    uint32_t *Etile = E + (size_t)v0 * (size_t)k;
    // PACKED: the wave's words of the tile, from word0 on (lane i keeps word i), and its cells
    const int nwords = PACKED ? (tv * k + 63) >> 6 : 0, wwords = (nwords + kScoreThreads / 64 - 1) / (kScoreThreads / 64);
    const int lane = lane_id(), word0 = __builtin_amdgcn_readfirstlane(tid >> 6) * wwords;
    const bool keeper = lane < wwords && word0 + lane < nwords;
    uint32_t *Ewave = Etile + (size_t)word0 * 64;
    unsigned long long word = 0ull;
    if (PACKED) {
        bits += (size_t)tile * nwords + word0;
        if (pass > 0 && keeper) word = bits[lane];
    }
    const bool ahead = !PACKED && pass > 0 && total <= kEstAhead * kScoreThreads;
    uint32_t est[kEstAhead];
    if (ahead) {
#pragma unroll
        for (int u = 0; u < kEstAhead; ++u) {
            const int i = tid + u * kScoreThreads;
            est[u] = i < total ? __builtin_nontemporal_load(Etile + i) : 0u;
        }
    }
    for (int i = tid; i <= tv; i += kScoreThreads) rowrel[i] = (uint32_t)((int64_t)rowptr[v0 + (i < nv ? i : nv)] - e0);
    if (!PACKED || pass == 0)
        for (int i = tid; i < tv * k; i += kScoreThreads) hist[i] = 0;
    for (int j = tid; j < k; j += kScoreThreads) {
        const long long s = S[j];
        room[j] = (uint32_t)(P - s);
        moved[j] = 0;
        if (tile == 0) Snext[j] = s;
    }
    __syncthreads();
    bool any_long = false;
    if (lr.rows != 0) {
        bool mine = false;
        for (int i = tid; i < nv; i += kScoreThreads) mine |= rowrel[i + 1] - rowrel[i] >= lr.degree;
        any_long = __syncthreads_or(mine ? 1 : 0) != 0;
    }
    auto is_long = [&](int r) { return any_long && rowrel[r + 1] - rowrel[r] >= lr.degree; };
    // PACKED: the counts are added to the stored estimates, in LDS, as they are found
    const uint32_t one = PACKED ? 1u << sh : 1u;
    if (PACKED && pass > 0) {
        if (any_long) {
            for (int i = tid; i < total; i += kScoreThreads) hist[i] = __builtin_nontemporal_load(Etile + i);
        } else {
            constexpr int kAtOnce = 8;
            uint32_t at = 0;
            for (int w0 = 0; w0 < wwords; w0 += kAtOnce) {
                uint32_t before[kAtOnce];
#pragma unroll
                for (int u = 0; u < kAtOnce; ++u) {
                    const unsigned long long set = wave_word(word, w0 + u);
                    before[u] = (set >> lane) & 1ull ? __builtin_nontemporal_load(Ewave + at + __popcll(set & lanes_below(lane))) : 0u;
                    at += (uint32_t)__popcll(set);
                }
#pragma unroll
                for (int u = 0; u < kAtOnce; ++u) {
                    const int i = (word0 + w0 + u) * 64 + lane;
                    if (w0 + u < wwords && i < tv * k) hist[i] = before[u];
                }
            }
        }
        __syncthreads();
    }

    const int32_t *cbase = colidx + e0;
    // (the next turn's column ids are on their way while this turn's labels are looked up: a skewed tile takes many)
    auto count_entries = [&](uint32_t from, uint32_t to) {
        int32_t col[U];
        auto request = [&](uint32_t base) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const uint32_t i = base + u * kScoreThreads;
                col[u] = i < to ? __builtin_nontemporal_load(cbase + i) : -1;
            }
        };
        if (from + tid < to) request(from + tid);
        for (uint32_t base = from + tid; base < to; base += kScoreThreads * U) {
            uint32_t lab[U];
#pragma unroll
            for (int u = 0; u < U; ++u) lab[u] = col[u] >= 0 && (int64_t)col[u] < gather_limit ? (uint32_t)Lc[col[u]] : 0xFFFFFFFFu;
            if (base + kScoreThreads * U < to) request(base + kScoreThreads * U);
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (lab[u] != 0xFFFFFFFFu && !(check && lab[u] == none)) {
                    const int r = owning_row(rowrel, base + u * kScoreThreads, tv);
                    atomicAdd(&hist[r * k + (int)lab[u]], one);
                }
            }
        }
    };
    if (!any_long) {
        count_entries(0, rowrel[tv]);
    } else {                                    // the stretches between the long rows
        uint32_t from = 0;
        for (int r = 0; r < nv; ++r)
            if (is_long(r)) { count_entries(from, rowrel[r]); from = rowrel[r + 1]; }
        count_entries(from, rowrel[tv]);
    }
    __syncthreads();

    // blend: E = h (first pass) or E += h * 2^(pass-1); the blended row stays in LDS (a long row's estimates are its
    // parts' business)
    auto blend = [&](int i, uint32_t before) {
        const uint32_t e = before + (hist[i] << sh);
        hist[i] = e;
        if (store_e && !(any_long && is_long(i / k))) __builtin_nontemporal_store(e, Etile + i);
    };
    if (PACKED) {
        if (store_e && any_long) {
            for (int i = tid; i < total; i += kScoreThreads)
                if (!is_long(i / k)) __builtin_nontemporal_store(hist[i], Etile + i);
        } else if (store_e) {
            uint32_t at = 0;
            for (int w = 0; w < wwords; ++w) {
                const int i = (word0 + w) * 64 + lane;
                const uint32_t e = i < total ? hist[i] : 0u;
                const unsigned long long set = __ballot(e != 0u);
                if (lane == w) word = set;
                if (e) __builtin_nontemporal_store(e, Ewave + at + __popcll(set & lanes_below(lane)));
                at += (uint32_t)__popcll(set);
            }
            if (keeper) bits[lane] = word;
        }
    } else if (ahead) {
#pragma unroll
        for (int u = 0; u < kEstAhead; ++u) {
            const int i = tid + u * kScoreThreads;
            if (i < total) blend(i, est[u]);
        }
    } else {
        for (int i = tid; i < total; i += kScoreThreads) blend(i, pass == 0 ? 0u : __builtin_nontemporal_load(Etile + i));
    }
    if (!PACKED) __syncthreads();

    // proposals, g lanes per vertex
    const int g = tv >= kScoreThreads ? 1 : tv * 64 <= kScoreThreads ? 64 : kScoreThreads / tv;
    const int sub = tid & (g - 1);
    for (int t0 = 0; t0 < nv; t0 += kScoreThreads / g) {       // (every lane of a group takes part in its exchange)
        const int t = t0 + tid / g;
        const bool in = t < nv && !is_long(t < nv ? t : 0);
        uint32_t old = 0xFFFFFFFFu;
        if (in && standing != kNoneLabelled) old = (uint32_t)Lc[v0 + t];
        const bool had = in && (standing == kAllLabelled || (check && old != none));
        uint32_t best = old;
        const uint32_t *hrow = hist + (in ? t : 0) * k;
        const uint32_t b = best_partition([&](int j) { return hrow[j]; }, room, k, had ? old : 0xFFFFFFFFu, sub, g);
        if (!(pass == 0 && had)) best = b;
        if (in && sub == 0) {
            prop[v0 + t - chunk_lo] = (LabelT)best;
            if (!had || best != old) atomicAdd(&moved[best], 1u);
        }
    }
    __syncthreads();
    // (tv divides the admission tile: a workgroup's vertices lie in one of them)
    const uint32_t atile = (uint32_t)((v0 - chunk_lo) / kAdmitTile);
    for (int j = tid; j < k; j += kScoreThreads)
        if (moved[j]) add_movers(cnt, coarse, k, atile, (uint32_t)j, moved[j]);
}

// Admission of a tile of kAdmitTile vertices, a thread each: a mover is admitted while fewer than room[t] = P - S[t]
// earlier vertices of the chunk asked for its t.  Ranks are only worked out for partitions with room for some of the
// chunk's movers.  rej / ocnt: the rejected new vertices of the tile, a bit per vertex and their number (first
// pass).  Clears the other pair of tables.
// LDS: base[k], tot[k], dS[k], room[k] (64 bits), wcnt[16][k] (16 bits)
constexpr size_t admit_tiles_lds(int k) { return (size_t)k * (3 * 4 + 8 + (kAdmitTile / 64) * 2) + 16; }

template <typename LabelT>
__global__ __launch_bounds__(kAdmitTile) void k_admit_tiles(
    LabelT *__restrict__ Lc, const LabelT *__restrict__ prop, int64_t chunk_lo, int64_t chunk_hi, int k, long long P,
    const uint32_t *__restrict__ cnt, const uint32_t *__restrict__ coarse, uint32_t *__restrict__ cnt_other,
    uint32_t *__restrict__ coarse_other, int tiles_full, const long long *__restrict__ S,
    unsigned long long *__restrict__ Snext, unsigned long long *__restrict__ rej, uint32_t *__restrict__ ocnt, int standing) {
    extern __shared__ long long smem_ll[];
    constexpr int nwaves = kAdmitTile / 64;
    long long *room = smem_ll;                           // k
    uint32_t *base = (uint32_t *)(room + k);            // k  movers in earlier tiles
    uint32_t *tot = base + k;                           // k  movers of the chunk
    int32_t *dS = (int32_t *)(tot + k);                 // k
    uint16_t *wcnt = (uint16_t *)(dS + k);              // nwaves * k  movers per wave, ranked partitions only
    __shared__ int s_any;
    __shared__ uint32_t s_new;
    const uint32_t none = LabelTraits<LabelT>::kUnassigned;
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int tile = (int)blockIdx.x, tiles = (int)gridDim.x;
    const int64_t v = chunk_lo + (int64_t)tile * kAdmitTile + tid;
    const bool inside = v < chunk_hi;
    uint32_t t = 0, old = 0;
    if (inside) {
        t = (uint32_t)prop[v - chunk_lo];
        if (standing != kNoneLabelled) old = (uint32_t)Lc[v];
    }
    const bool had = inside && (standing == kAllLabelled || (standing == kSomeLabelled && old != none));
    const bool mover = inside && (!had || t != old);
    for (int j = tid; j < k; j += kAdmitTile) { base[j] = 0; tot[j] = 0; dS[j] = 0; room[j] = P - S[j]; }
    if (tid == 0) { s_any = 0; s_new = 0; }
    __syncthreads();
    {
        const int nseg = kAdmitTile / k, col = tid % k, seg = tid / k;
        if (seg < nseg) {
            uint32_t all = 0, before = 0;
            int first = 0, last = tiles;                // the tiles read one by one: all of them, or the coarse row's own
            if (coarse) {
                const int group = tile / kPlainCoarse, groups = (tiles + kPlainCoarse - 1) / kPlainCoarse;
                for (int r = seg; r < groups; r += nseg) {
                    const uint32_t c = coarse[(size_t)r * k + col];
                    all += c;
                    if (r < group) before += c;
                }
                first = group * kPlainCoarse;
                last = tile;
            }
            for (int r = first + seg; r < last; r += nseg) {
                const uint32_t c = cnt[(size_t)r * k + col];
                if (!coarse) all += c;
                if (r < tile) before += c;
            }
            if (all) atomicAdd(&tot[col], all);
            if (before) atomicAdd(&base[col], before);
        }
    }
    const size_t cells = (size_t)tiles_full * k, coarse_cells = coarse ? (size_t)((tiles_full + kPlainCoarse - 1) / kPlainCoarse) * k : 0;
    for (size_t i = (size_t)tile * kAdmitTile + tid; i < cells; i += (size_t)tiles * kAdmitTile) {
        cnt_other[i] = 0u;
        if (i < coarse_cells) coarse_other[i] = 0u;
    }
    __syncthreads();
    if (tid < k && room[tid] > 0 && (long long)tot[tid] > room[tid]) s_any = 1;
    __syncthreads();
    const long long rm = mover ? room[t] : 0;
    bool admitted = mover && rm > 0;
    if (s_any) {
        for (int j = tid; j < nwaves * k; j += kAdmitTile) wcnt[j] = 0;
        __syncthreads();
        const bool ranked = admitted && (long long)tot[t] > rm;
        int same_total; bool leader;
        const int wrank = rank_among_equal(ranked, t, lane, &same_total, &leader);
        if (leader) wcnt[wave * k + t] = (uint16_t)same_total;
        __syncthreads();
        if (ranked) {
            long long rank = (long long)base[t] + wrank;
            for (int w = 0; w < wave; ++w) rank += wcnt[w * k + t];
            admitted = rank < rm;
        }
    }
    if (admitted) {
        Lc[v] = (LabelT)t;
        atomicAdd(&dS[t], 1);
        if (had) atomicAdd(&dS[old], -1);
    }
    if (standing != kAllLabelled) {
        const unsigned long long m = __ballot(inside && !had && !admitted);
        if (lane == 0) {
            rej[(size_t)tile * nwaves + wave] = m;
            if (m) atomicAdd(&s_new, (uint32_t)__popcll(m));
        }
    }
    __syncthreads();
    for (int j = tid; j < k; j += kAdmitTile) {
        const int32_t d = dS[j];
        if (d != 0) atomicAdd(&Snext[j], (unsigned long long)(long long)d);
    }
    if (standing != kAllLabelled && tid == 0) ocnt[tile] = s_new;
}

// The spill of a chunk in one launch (see k_spill_scan for the level sequence: order the partitions by (size, id),
// C[a] placements are made before a + 1 of them are level).  Every workgroup builds the level tables for itself, takes
// the levels its tile's placements fall into one after the other, and looks the idx-th smallest id of the a
// smallest partitions up in a list of them (searching the ids one by one took 104 us per chunk at k = 256).  Sizes are
// read from Sin and written by workgroup 0 to Sout: the a smallest partitions that are level at the end share what is
// left over, the others keep theirs.
// LDS: Sl[k], sorted[k], C[k + 1] (64 bits), rnk[k], list[k]
constexpr size_t spill_tiles_lds(int k) { return (size_t)k * (3 * 8 + 2 * 4) + 16; }

template <typename LabelT>
__global__ __launch_bounds__(kAdmitTile) void k_spill_tiles(LabelT *__restrict__ Lc, int64_t chunk_lo, int k,
                                                            const unsigned long long *__restrict__ rej,
                                                            const uint32_t *__restrict__ ocnt,
                                                            const long long *__restrict__ Sin, long long *__restrict__ Sout) {
    extern __shared__ long long smem_ll[];
    constexpr int nwaves = kAdmitTile / 64;
    long long *Sl = smem_ll, *sorted = Sl + k, *C = sorted + k;
    int *rnk = (int *)(C + k + 1), *list = rnk + k;
    __shared__ long long wave_total[nwaves];
    __shared__ long long s_base, s_total;
    __shared__ int s_level;
    __shared__ uint32_t wfirst[nwaves];
    const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
    const int tile = (int)blockIdx.x, tiles = (int)gridDim.x;
    const uint32_t mine = tid < tiles ? ocnt[tid] : 0u;               // (at most kPlainTiles = kAdmitTile tiles)
    const long long ex = block_exclusive_sum((long long)mine, wave_total);
    if (tid == tile) s_base = ex;
    if (tid == kAdmitTile - 1) s_total = ex + mine;
    __syncthreads();
    const long long total = s_total, i_lo = s_base, i_hi = i_lo + ocnt[tile];
    if (total == 0) {
        if (tile == 0)
            for (int j = tid; j < k; j += kAdmitTile) Sout[j] = Sin[j];
        return;
    }
    if (i_lo == i_hi && tile != 0) return;
    for (int j = tid; j < k; j += kAdmitTile) Sl[j] = Sin[j];
    if (tid == 0) s_level = 0;
    __syncthreads();
    if (tid < k) {
        const long long sj = Sl[tid];
        int r = 0;
        for (int i = 0; i < k; ++i) r += (Sl[i] < sj || (Sl[i] == sj && i < tid)) ? 1 : 0;
        rnk[tid] = r;
        sorted[r] = sj;
    }
    __syncthreads();
    {
        const long long s = tid < k ? sorted[tid] : 0;
        const long long ps = block_exclusive_sum(s, wave_total);
        if (tid < k) {
            const long long c = (long long)tid * s - ps;              // sum over q < tid of (s - sorted[q])
            C[tid] = c;
            if (c < total) atomicAdd(&s_level, 1);
        }
        if (tid == 0) C[k] = 0x7fffffffffffffffLL;
    }
    __syncthreads();
    if (tile == 0 && tid < k) {
        const int a = s_level;                                        // partitions level at the end
        const long long rest = total - C[a - 1];
        long long size = Sl[tid];
        if (rnk[tid] < a) {
            int pos = 0;
            for (int q = 0; q < tid; ++q) pos += rnk[q] < a ? 1 : 0;
            size = sorted[a - 1] + rest / a + (pos < (int)(rest % a) ? 1 : 0);
        }
        Sout[tid] = size;
    }
    if (i_lo == i_hi) return;
    // the placement number of this thread's vertex
    const unsigned long long m = rej[(size_t)tile * nwaves + wave];
    const bool un = (m >> lane) & 1ull;
    if (lane == 0) wfirst[wave] = (uint32_t)__popcll(m);
    __syncthreads();
    long long i = i_lo + __popcll(m & lanes_below(lane));
    for (int w = 0; w < wave; ++w) i += wfirst[w];
    int a = 1;                                                        // smallest a with i_lo < C[a]
    {
        int hi_a = k;
        while (a < hi_a) { const int mid = (a + hi_a) >> 1; if (i_lo < C[mid]) hi_a = mid; else a = mid + 1; }
    }
    for (; a <= k && C[a - 1] < i_hi; ++a) {
        if (C[a] == C[a - 1]) continue;                               // (the same for every thread)
        if (a < k) {                                                  // the ids of the a smallest partitions, ascending
            const bool on = tid < k && rnk[tid] < a;
            const long long at = block_exclusive_sum(on ? 1 : 0, wave_total);
            if (on) list[at] = tid;
            __syncthreads();
        }
        if (un && i >= C[a - 1] && i < C[a]) {
            const int idx = (int)((unsigned long long)(i - C[a - 1]) % (unsigned)a);
            Lc[chunk_lo + (int64_t)tile * kAdmitTile + tid] = (LabelT)(a < k ? list[idx] : idx);
        }
        __syncthreads();
    }
}

static_assert(admit_tiles_lds(kPlainMaxK) <= 64 * 1024 && spill_tiles_lds(kPlainMaxK) <= 64 * 1024, "LDS that needs no asking for");

}  // namespace grem
