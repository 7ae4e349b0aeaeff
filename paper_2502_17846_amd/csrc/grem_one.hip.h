// A whole run of the plain route on one workgroup, for graphs so small that a chunk step is mostly launches and the
// latency inside them: labels, the chunk's histograms and the sizes stay in a CU's LDS from the first pass to the last,
// and a step is three barriers instead of two or three launches.
//   k_one_entries   (the whole chip) every entry with its row in the chunk beside it, in one word: nothing has to be searched for
//   k_one_run       Alg. 1's loop
// 10,000 vertices, k = 4, 30 steps of 1,024 rows and 10,000 entries: the call 387 -> 223 us, 5.6 us a step where three launches took 10 to 12.
// A CU adds an entry to its counter in some 0.35 ns (LDS reads and atomics), so that a chip's launches win from some 25,000 entries a step on.
#pragma once
#include "grem_plain.hip.h"

namespace grem {

constexpr int kOneThreads = 1024;
constexpr int kOneWaves = kOneThreads / 64;
constexpr int kOneSlots = 4;                         // rows per thread and chunk, kOneThreads apart
constexpr int kOneMaxK = 8;                          // (more counters than that are not worth one workgroup's while)
constexpr int64_t kOneMaxN = 65534;                  // an entry's column takes 16 bits, one of them says "none"
constexpr int64_t kOneMaxChunk = (int64_t)kOneSlots * kOneThreads;
constexpr int64_t kOneMaxChunks = 1024;
constexpr size_t kOneLds = 148 * 1024;
// counters of 16 bits, whole words per row; then the labels
inline size_t one_lds_bytes(int64_t n, int64_t cl, int k) { return (size_t)cl * ((k + 1) / 2) * 4 + (size_t)(n + 1 + 15) / 16 * 16; }

// rec[e] = column | row in its chunk << 16; a column that is no vertex becomes n.  A wave per row for a row's first kOnePart entries
// (blockIdx.y = 0), and for part y of the rows that are so long a wave per 64 rows, which finds them: one wave's 940 turns were
// a row of 60,000 entries.
constexpr int kOnePart = 2048;
template <typename RowT>
__global__ __launch_bounds__(256) void k_one_entries(const RowT *__restrict__ rowptr, const int32_t *__restrict__ colidx, int64_t n, int64_t cl,
                                                     uint32_t *__restrict__ rec) {
    const int64_t waves = (int64_t)gridDim.x * 4, first = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6), skip = (int64_t)blockIdx.y * kOnePart;
    auto part = [&](int64_t v, int64_t begin, int64_t end) {
        const uint32_t row = (uint32_t)(v % cl) << 16;
        begin += skip;
        if (end - begin > kOnePart) end = begin + kOnePart;
        for (int64_t e = begin + lane_id(); e < end; e += 64) {
            const uint32_t col = (uint32_t)colidx[e];
            rec[e] = (col < (uint32_t)n ? col : (uint32_t)n) | row;
        }
    };
    if (blockIdx.y == 0) {
        for (int64_t v = first; v < n; v += waves) part(v, (int64_t)rowptr[v], (int64_t)rowptr[v + 1]);
        return;
    }
    for (int64_t v0 = first * 64; v0 < n; v0 += waves * 64) {
        const int64_t v = v0 + lane_id();
        unsigned long long some = __ballot(v < n && (int64_t)rowptr[v + 1] - (int64_t)rowptr[v] > skip);
        for (; some; some &= some - 1ull) {
            const int64_t u = v0 + __builtin_ctzll(some);
            part(u, (int64_t)rowptr[u], (int64_t)rowptr[u + 1]);
        }
    }
}

// KM: room for k partitions (2, 4 or 8).  A thread takes eight neighbouring entries at a time: the lanes of a wave are then
// in different rows more often than not, and their counters seldom the same word (an entry per lane: 269 us for 229).  With a word
// per row, lanes in one long row would all queue at it (10,000 vertices, k = 2, 250,000 entries, most of
// them in rows of 200 to 60,000: 500 to 660 us, so 235 to 270; in launches 390 to 550).
template <typename RowT, int KM>
__global__ __launch_bounds__(kOneThreads) void k_one_run(const RowT *__restrict__ rowptr, const uint32_t *__restrict__ rec, int n, int k, int cl,
                                                         int R, int P, const uint8_t *__restrict__ Lc, const long long *__restrict__ S,
                                                         uint32_t *__restrict__ E, int keep_e, int32_t *__restrict__ labels_out,
                                                         int64_t *__restrict__ sizes_out) {
    extern __shared__ uint32_t hist[];               // cl rows of kk words
    constexpr uint32_t none = LabelTraits<uint8_t>::kUnassigned;
    constexpr int U = 8;
    __shared__ uint32_t first[kOneMaxChunks + 1];    // a chunk's first entry
    __shared__ int size[kOneMaxK], sorted[kOneMaxK], levels[kOneMaxK], rnk[kOneMaxK];
    __shared__ uint32_t room[kOneMaxK], gone[kOneMaxK];
    __shared__ uint16_t asked[kOneSlots * kOneWaves][kOneMaxK];          // movers by slot, wave and partition
    __shared__ uint16_t left[kOneSlots * kOneWaves];                      // rejected new vertices
    const int tid = threadIdx.x, lane = lane_id(), wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kk = (k + 1) / 2, nchunks = (n + cl - 1) / cl, slots = (cl + kOneThreads - 1) / kOneThreads;
    uint8_t *lab = (uint8_t *)(hist + (size_t)cl * kk);
    for (int i = tid; i < cl * kk; i += kOneThreads) hist[i] = 0u;
    for (int v = tid; v < n; v += kOneThreads) lab[v] = Lc[v];
    for (int c = tid; c <= nchunks; c += kOneThreads) first[c] = (uint32_t)rowptr[c < nchunks ? (int64_t)c * cl : (int64_t)n];
    if (tid == 0) lab[n] = (uint8_t)none;
    if (tid < k) {
        size[tid] = (int)S[tid];
        room[tid] = (uint32_t)(P - size[tid]);
        gone[tid] = 0u;
    }
    __syncthreads();
    uint32_t ahead[U];                               // the chunk's first entries, requested a step before
    const uint4 *eights = (const uint4 *)rec;        // (two to eight entries; padded)
    auto request = [&](uint32_t (&r)[U], uint32_t q, int c) {
        if (q * U >= first[c + 1]) return;
        const uint4 x = eights[2 * (size_t)q], y = eights[2 * (size_t)q + 1];
        r[0] = x.x; r[1] = x.y; r[2] = x.z; r[3] = x.w;
        r[4] = y.x; r[5] = y.y; r[6] = y.z; r[7] = y.w;
    };
    // cnt_nbrs (Alg. 2)
    auto count = [&](const uint32_t (&r)[U], uint32_t q, int c) {
        const uint32_t f0 = first[c], f1 = first[c + 1];
        if (q * U >= f1) return;
        uint32_t l[U];
#pragma unroll
        for (int u = 0; u < U; ++u) l[u] = q * U + u - f0 < f1 - f0 ? lab[r[u] & 0xFFFFu] : none;
        if constexpr (KM == 2) {                     // (a word per row: what neighbouring entries of a row add is added up first)
            uint32_t sum = 0;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                sum += l[u] == none ? 0u : l[u] ? 65536u : 1u;
                if (u + 1 < U && r[u] >> 16 == r[u + 1 < U ? u + 1 : u] >> 16) continue;
                if (sum) atomicAdd(&hist[r[u] >> 16], sum);
                sum = 0;
            }
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (l[u] != none) atomicAdd(&hist[(r[u] >> 16) * kk + (l[u] >> 1)], l[u] & 1u ? 65536u : 1u);
        }
    };
    request(ahead, first[0] / U + tid, 0);
    for (int pass = 0; pass <= R; ++pass) {
        const int sh = pass == 0 ? 0 : pass - 1;
        const bool store_e = pass < R || keep_e;
        for (int c = 0; c < nchunks; ++c) {
            const int lo = c * cl, len = n - lo < cl ? n - lo : cl;
            uint32_t before[KM];
            auto estimates = [&](int row) {
#pragma unroll
                for (int j = 0; j < KM; ++j) before[j] = pass > 0 && j < k && row < len ? E[(size_t)(lo + row) * k + j] : 0u;
            };
            estimates(tid);                          // of the thread's first row, requested before the counting
            uint32_t q = first[c] / U + tid;
            count(ahead, q, c);
            for (q += kOneThreads; q * U < first[c + 1]; q += kOneThreads) {
                uint32_t r[U];
                request(r, q, c);
                count(r, q, c);
            }
            if (c + 1 < nchunks || pass < R) {
                const int next = c + 1 < nchunks ? c + 1 : 0;
                request(ahead, first[next] / U + tid, next);
            }
            __syncthreads();
            // blend and assign, a row per thread and slot
            uint32_t want[kOneSlots], old[kOneSlots];
            int rank[kOneSlots];
#pragma unroll
            for (int s = 0; s < kOneSlots; ++s) {
                want[s] = old[s] = none;
                rank[s] = -1;                        // no mover
                if (s >= slots) continue;
                const int row = s * kOneThreads + tid;
                const bool in = row < len;
                if (s > 0) estimates(row);
                if (in) {
                    uint32_t *h = hist + row * kk, *e_row = E + (size_t)(lo + row) * k;
                    old[s] = lab[lo + row];
                    uint32_t pair[KM / 2];
#pragma unroll
                    for (int j = 0; j < KM / 2; ++j) {
                        pair[j] = j < kk ? h[j] : 0u;
                        if (j < kk) h[j] = 0u;
                    }
                    unsigned long long best = 0;
#pragma unroll
                    for (int j = 0; j < KM; ++j) {
                        if (j >= k) continue;
                        const uint32_t e = before[j] + ((j & 1 ? pair[j / 2] >> 16 : pair[j / 2] & 0xFFFFu) << sh);
                        if (store_e) e_row[j] = e;
                        const uint32_t rm = room[j] + ((uint32_t)j == old[s] ? 1u : 0u);
                        const unsigned long long key = rm ? ((unsigned long long)e << 32) | rm : 0ull;
                        if (key > best) { best = key; want[s] = (uint32_t)j; }       // the first of the best
                    }
                    if (pass == 0 && old[s] != none) want[s] = old[s];
                }
                const bool mover = in && want[s] != old[s];
                int total; bool leader;
                const int r = rank_among_equal(mover, want[s], lane, &total, &leader);
                if (mover) rank[s] = r;
                if (lane < kOneMaxK) asked[s * kOneWaves + wave][lane] = 0;
                if (leader) asked[s * kOneWaves + wave][want[s]] = (uint16_t)total;
            }
            __syncthreads();
            // every wave adds the movers up: lane t those to partition t
            const int cells = slots * kOneWaves;
            uint32_t total = 0;
            if (lane < k)
                for (int i = 0; i < cells; ++i) total += asked[i][lane];
            const uint32_t rm = lane < k ? room[lane] : 0u;
            const bool limited = __ballot(total > rm) != 0ull;
#pragma unroll
            for (int s = 0; s < kOneSlots; ++s) {
                if (s >= slots) continue;
                const int row = s * kOneThreads + tid;
                bool admitted = rank[s] >= 0;
                if (limited) {                       // by rank among the chunk's movers to the same partition
                    uint32_t earlier = 0;
                    if (lane < k)
                        for (int i = 0; i < s * kOneWaves + wave; ++i) earlier += asked[i][lane];
                    const uint32_t at = (uint32_t)__shfl((int)earlier, (int)(want[s] & 63u)) + (uint32_t)rank[s];
                    const uint32_t most = (uint32_t)__shfl((int)rm, (int)(want[s] & 63u));
                    admitted = admitted && at < most;
                }
                if (admitted) lab[lo + row] = (uint8_t)want[s];
                int many; bool leader;
                (void)rank_among_equal(admitted && old[s] != none, old[s], lane, &many, &leader);
                if (leader) atomicAdd(&gone[old[s]], (uint32_t)many);
                const unsigned long long rest = __ballot(row < len && old[s] == none && !admitted);
                if (pass == 0 && lane == 0) left[s * kOneWaves + wave] = (uint16_t)__popcll(rest);
                if (!((rest >> lane) & 1ull)) rank[s] = -1;
                else rank[s] = __popcll(rest & lanes_below(lane));                   // from here on: the rejected new vertex's among the wave's
            }
            __syncthreads();
            uint32_t rejected = 0;
            if (pass == 0) {
                for (int i = 0; i < cells; ++i) rejected += left[i];
            }
            if (wave == 0 && lane < k) {             // fix_sizes (Alg. 2)
                size[lane] += (int)(total < rm ? total : rm) - (int)gone[lane];
                gone[lane] = 0u;
                room[lane] = (uint32_t)(P - size[lane]);
            }
            if (rejected == 0) continue;
            // The rejected new vertices go to the smallest partition one after the other (lowest id on ties): ordered by (size, id),
            // levels[a] placements are made before a + 1 partitions are level.
            __syncthreads();
            if (wave == 0) {
                const int mine = lane < k ? size[lane] : 0;
                int r = 0;
                for (int i = 0; i < k; ++i) r += size[i] < mine || (size[i] == mine && i < lane) ? 1 : 0;
                if (lane < k) { rnk[lane] = r; sorted[r] = mine; }
            }
            __syncthreads();
            if (wave == 0) {
                int sum = 0;
                const int own = lane < k ? sorted[lane] : 0;
                for (int i = 0; i < k; ++i) sum += i < lane ? sorted[i] : 0;
                const int level = lane * own - sum;
                if (lane < k) levels[lane] = level;
                const int a = __popcll(__ballot(lane < k && level < (int)rejected));            // level at the end
                const int top = __shfl(own, a - 1), spare = (int)rejected - __shfl(level, a - 1);
                const unsigned long long in = __ballot(lane < k && rnk[lane < k ? lane : 0] < a);
                if ((in >> lane) & 1ull) {
                    size[lane] = top + spare / a + (__popcll(in & lanes_below(lane)) < spare % a ? 1 : 0);
                    room[lane] = (uint32_t)(P - size[lane]);
                }
            }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < kOneSlots; ++s) {
                if (s >= slots || rank[s] < 0) continue;
                int i = rank[s];
                for (int q = 0; q < s * kOneWaves + wave; ++q) i += left[q];
                int a = 1;
                while (a < k && levels[a] <= i) ++a;
                int idx = (i - levels[a - 1]) % a, id = 0;         // the idx-th smallest id of the a smallest partitions
                for (int j = 0; j < k; ++j)
                    if (rnk[j] < a && idx-- == 0) id = j;
                lab[lo + s * kOneThreads + tid] = (uint8_t)id;
            }
            __syncthreads();
        }
    }
    __syncthreads();
    for (int v = tid; v < n; v += kOneThreads) labels_out[v] = (int32_t)lab[v];
    if (sizes_out && tid < k) sizes_out[tid] = (int64_t)size[tid];
}

}  // namespace grem
