// Host side of the GREM library: argument checks, memory carve-up, and the stream-ordered sequence
// of launches for each chunk of each pass (Alg. 1's chunk loop).  See include/grem.h for the
// contract of every entry point.
//
// Structure:
//   Arena / carve      device memory for a call: pieces of the caller's workspace, or stream-ordered
//                      allocations
//   PlanData           the re-laid-out copy of a graph's entries for the two-phase route (k <= 32):
//                      built once per call, or once per graph behind a grem_plan
//   run_two_phase      Alg. 1's loop on a plan
//   run_plain          Alg. 1's loop straight on the CSR (any k)
#include "grem.h"

#include <hip/hip_runtime.h>

#include <algorithm>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <type_traits>
#include <vector>

#include "grem_kernels.hip.h"
#include "grem_one.hip.h"
#include "grem_plain.hip.h"
#include "grem_twophase.hip.h"

namespace {

using namespace grem;

constexpr int kLdsHistBytes = 32 * 1024;   // LDS spent on one tile's histograms
constexpr int kTileHistBytes = 16 * 1024;  // merged launches: the same (32 KB: 117 ms where 16 KB take 106 and 8 KB 107)
constexpr int kTileGrid = 2048;            // ... and workgroups per chunk (1024: 2.18 ms on a million vertices, 2048: 1.91,
                                           // 4096: 2.02, 8192: 2.52)
// Merged launches: estimates are packed where they outgrow the Infinity Cache, from 32 partitions on (fewer are mostly not
// zero; below 128 of them half of a row may be, and the estimates must outgrow it twice).  Whole and packed: k = 40, 480 MB 4.51 and
// 4.53 ms; 48, 768 MB 3.84 and 3.42; 64, 256 MB 1.70 and 1.71, 1 GB 4.2 and 3.6; 100, 120 MB 1.50 and 1.53; 256, 17 GB 63.8
// and 50.9; 400, 480 MB 2.31 and 2.01, 6.4 GB 15.6 and 12.3.  Rows of many entries gain less and lose nothing: 250 entries, k = 256
// 4.49 and 3.9 ms; 500 to 2,000 entries, k = 64 to 1024 within 2 %.
// Nor are they packed in tiles of fewer than kEstAhead * kScoreThreads = 2,048 cells, which chunks of few rows make: whole, a
// thread asks for all of its estimates before the counting starts, packed it has to see the bits first.  Three passes: k = 40, tiles of
// 640 cells 8.91 and 9.18, 1,280 5.14 and 5.15, 2,560 4.63 and 4.26; 64, 512 9.24 and 9.52, 2,048 4.75 and 4.80, 4,096 3.12 and 2.74;
// 100, 800 6.82 and 7.00, 1,600 4.23 and 4.23, 3,200 3.37 and 2.98; 128, 1,024 2.79 and 2.83, 2,048 1.87 and 1.85, 4,096 1.58 and 1.37.
constexpr int kPackMinK = 32, kPackManyK = 128;
constexpr size_t kPackMinBytes = 256u << 20;
// One workgroup does the whole run (grem_one.hip.h) where a step's entries and one and a half times its counters are no more than this: it
// takes some 1.3 us, 0.35 ns for an entry and 0.2 to 0.6 for a counter, the launches 12 to 15 us.  Calls in launches | so: 10,100 entries and 4,096
// counters 387 | 223 us; 15,000 and 4,000 980 | 710; 15,750 and 8,400 607 | 525; 16,000 and 4,000 223 | 187; 16,000 and 25,600 1060 | 1700; 40,000 and 8,000 568 | 787
constexpr unsigned long long kOneWork = 28672;
constexpr int kLdsMaxK = 1024;             // above this the histograms live in E's rows
constexpr int kLongRowDegree = 16384;      // plain score kernels: rows this long get a grid of their own ...
constexpr uint32_t kLongRowPart = 16384;   // ... that many entries per workgroup and turn
constexpr unsigned kLongRowGrid = 512;
constexpr int kLongDegree = 8192;          // merged launches: rows this long (4096 and 16384 were slower) are dealt out in parts ...
constexpr uint32_t kLongPart = 16384;      // ... of that many entries, of up to kLongPartMax when rows are longer than
constexpr int64_t kLongChunks = 1 << 16;   // most chunks whose long rows the prepass counts, for its read-back to bring along
constexpr uint32_t kLongPartMax = 65536;   // 64 parts: every part adds its k counts to the same row of estimates (rows of
                                           // 2M entries, k = 256: 92 ms in parts of 4096, 71.5 of 16384, 67.4 of 32768)
constexpr int kSweepMaxK = 32;             // two-phase route: 16-bit counters for 2048 rows: 64 KB of LDS up to k = 16
                                           // (4-bit labels), 128 KB up to k = 32 (8-bit labels)
constexpr int kHubsPerShare16 = 1024;      // hubs one hub share may touch: their 32-bit counters share the
constexpr int kHubsPerShare32 = 96;        // workgroup's LDS with the slice's counters
constexpr int64_t kSweepMinN = 1 << 22;    // AUTO: label table must exceed L2 for the route to pay
constexpr int64_t kSweepMinChunk = 1 << 14;   // AUTO: per-chunk launches must have work to do
constexpr int kDefaultColBits = 17;        // 2^17 labels, two per byte: 64 KB of LDS, two workgroups per CU
constexpr int kDefaultColBits32 = 16;      // k > 16: 2^16 labels, a byte each
constexpr int kDefaultHubDegree = 8192;
constexpr int64_t kMinSlices = 256;        // slices per chunk wanted: one per CU (and with 512 rows, of which two
                                           // share a tile's row of mover counts, never more than 256 tiles)
constexpr int64_t kMaxSegments = 1ll << 22;   // chunks * column blocks
constexpr int64_t kCutPackMinN = 1 << 20;  // edge cut: int32 labels of more vertices outgrow an XCD's 4 MB of L2
constexpr size_t kScoreLds16 = 150 * 1024, kScoreLds32 = 158 * 1024;   // k_tp_score's LDS: with the static counters for k <= 16
constexpr uint32_t kLookupFew = 256, kLookupMany = 512;   // workgroups of a chunk's look-up launch: short shares, long ones (grem_lookup_shares.hip.h; 128
                                           // and 384 for 256 were slower, at 25M and 111M vertices in chunks of 2^20 any was the same)
constexpr uint64_t kLookupSweep = 8192;    // workgroups of a look-up launch over all chunks: each copies a block's labels first (13.9M vertices, 106 blocks,
                                           // with one per 8192 entries 49,000 of them: 0.74 ms, so 0.38; 4096: k = 24 1.05 ms for 0.97, 16,384: k = 16 0.93 for 0.90)
constexpr int64_t kPlaceGrid = 1024;       // workgroups of k_tp_place wanted: four per CU
constexpr int kMaxParts = kPlanParts;      // parts of a slice (hub share) in the re-layout

// ---- process-wide state: the optional workspace and the measurement aids --------------------------
struct Global {
    std::mutex mu;
    void *ws = nullptr;
    size_t ws_bytes = 0;
    int prof_level = 0;
    struct Ev { int cls; hipEvent_t a, b; };
    std::vector<Ev> events;            // level 2: a pair per launch
    std::vector<hipEvent_t> marks;     // level 1: call start, first pass, end of every pass, end of call
    std::vector<hipEvent_t> pool;
};
Global g;

inline size_t align_up(size_t x, size_t a = 256) { return (x + a - 1) / a * a; }

// ---- options ---------------------------------------------------------------------------------------
struct Opts {
    int hist_mode = GREM_HIST_AUTO;
    int col_bits = 0;                       // 0 = automatic
    int hub_degree = kDefaultHubDegree;
    int long_row_degree = 0;                // 0 = automatic: see kLongRowDegree, kLongDegree
    int plan_max_k = 16;
};

bool resolve_options(const grem_options *o, Opts *out) {
    Opts r;
    if (o) {
        if (o->histogram_mode != GREM_HIST_AUTO && o->histogram_mode != GREM_HIST_LDS &&
            o->histogram_mode != GREM_HIST_GLOBAL && o->histogram_mode != GREM_HIST_SWEEP)
            return false;
        if (o->col_bits != 0 && (o->col_bits < 4 || o->col_bits > kMaxColBits)) return false;
        if (o->hub_degree < 0 || o->hub_degree > 65535) return false;
        if (o->long_row_degree < 0) return false;
        if (o->plan_max_k < 0 || o->plan_max_k > kSweepMaxK) return false;
        for (int i = 0; i < 3; ++i)
            if (o->reserved[i] != 0) return false;
        r.hist_mode = o->histogram_mode;
        r.col_bits = o->col_bits;
        if (o->hub_degree) r.hub_degree = o->hub_degree;
        if (o->long_row_degree) r.long_row_degree = o->long_row_degree;
        if (o->plan_max_k) r.plan_max_k = o->plan_max_k;
    }
    *out = r;
    return true;
}

// ---- device memory of a call -----------------------------------------------------------------------
// Bump mode: pieces of one caller-owned block, released by moving the top back.  Otherwise every
// request is an allocation of its own: stream-ordered (released stream-ordered) or, for memory that
// outlives the call, hipMalloc.
struct Arena {
    char *base = nullptr;
    size_t cap = 0, off = 0;
    hipStream_t stream = nullptr;
    bool persistent = false;
    std::vector<void *> owned;
    size_t total = 0;                       // bytes handed out (allocation modes)

    char *alloc(size_t bytes) {
        bytes = align_up(bytes ? bytes : 1);
        if (base) {
            if (off + bytes > cap) return nullptr;
            char *p = base + off;
            off += bytes;
            return p;
        }
        void *p = nullptr;
        const hipError_t e = persistent ? hipMalloc(&p, bytes) : hipMallocAsync(&p, bytes, stream);
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return nullptr;
        }
        owned.push_back(p);
        total += bytes;
        return (char *)p;
    }
    struct Mark { size_t off, count; };
    Mark mark() const { return {off, owned.size()}; }
    // gives back everything handed out since `m` (work already enqueued on the stream may still use it:
    // stream-ordered release, and in bump mode whatever takes the space next runs later on the same stream)
    void release_to(Mark m) {
        off = m.off;
        while (owned.size() > m.count) {
            if (persistent) (void)hipFree(owned.back());
            else (void)hipFreeAsync(owned.back(), stream);
            owned.pop_back();
        }
    }
    void release_all() { release_to({0, 0}); }
};

// Several arrays out of one request: the same function lays them out twice, first against a null
// base to find the size, then against the block.
struct Carver {
    char *base;
    size_t off = 0;
    // (an array of no elements is a null pointer, not the address of whatever comes next: code that asks
    // "is there such an array" must not be told yes)
    template <typename T> void take(T *&p, size_t count) {
        p = (base && count) ? reinterpret_cast<T *>(base + off) : nullptr;
        off += align_up(count * sizeof(T));
    }
};
template <typename F> bool carve(Arena &A, F &&f) {
    Carver dry{nullptr};
    f(dry);
    char *p = A.alloc(dry.off);
    if (!p) return false;
    Carver wet{p};
    f(wet);
    return true;
}
template <typename F> size_t carve_size(F &&f) {
    Carver dry{nullptr};
    f(dry);
    return align_up(dry.off ? dry.off : 1);
}

// ---- geometry of the two-phase route: chunks, row slices and column blocks (grem_twophase.hip.h) ---
struct TpGeom {
    int cb = 0, nbc = 0, nblk = 0, nch = 0, nsl = 0, srows = kSliceRows, shift = -1, gb = 0, ngroups = 1;
    uint32_t chunk = 0;
    bool ok = false;
};

// kmax: the largest k the layout is to serve (above 16 the look-up keeps a byte per label in LDS)
TpGeom tp_geometry(int64_t n, int64_t chunk, int col_bits_setting, int kmax) {
    TpGeom t;
    const int64_t cl = chunk < n ? chunk : n;
    const int64_t nch = (n + cl - 1) / cl;
    int cb = col_bits_setting;
    if (cb == 0) {
        const int want = kmax > 16 ? kDefaultColBits32 : kDefaultColBits;
        cb = 4;
        while (cb < want && (1ll << cb) < cl) ++cb;
    }
    const int64_t nbc = (cl + (1ll << cb) - 1) >> cb;
    const int64_t nblk = nch * nbc;
    // Rows per slice: a workgroup of the score kernel each, so a chunk of fewer slices than the chip has CUs is cut
    // finer -- as long as a sub-segment still has rows enough to be worth its padding and its table entries (some
    // two per column block: at the usual degrees tens of entries, padded to a multiple of eight).  The number of entries
    // is not known here, and sparse graphs pay for it in the plan, not in its runs: 13.9M vertices in chunks of 131,072
    // (k = 16) with 1 / 2 / 4 / 29 entries each, slices of 2048 and as cut here: plan 1.7 and 2.4, 1.9 and 2.4, 2.2 and
    // 2.4, 6.5 and 6.4 ms, its bytes 103 and 200, 173 and 270, 314 and 411, 2054 and 2169 MB, a two-pass run on
    // it 6.3 and 5.1, 6.5 and 5.2, 6.7 and 5.4, 9.3 and 6.8 ms: a plan and one run together are never slower.
    while (t.srows > 512 && (cl + t.srows - 1) / t.srows < kMinSlices && t.srows / 2 >= 2 * nblk) t.srows /= 2;
    const int64_t nsl = (cl + t.srows - 1) / t.srows;
    t.cb = cb;
    t.chunk = (uint32_t)cl;
    for (int b = 0; b < 31; ++b)
        if ((1ll << b) == cl) t.shift = b;
    t.ok = nblk <= kMaxBlocks && nch * nblk <= kMaxSegments && nch * nsl < (1ll << 28) &&
           nch * (nsl + 1) * nblk < (1ll << 40);
    if (t.ok) {
        t.nbc = (int)nbc; t.nblk = (int)nblk; t.nch = (int)nch; t.nsl = (int)nsl;
        // the intermediate copy keeps row (11 bits), block in group (gb) and column in block (cb) in 32 bits
        while (t.gb < 21 - cb && (1ll << t.gb) < nblk) ++t.gb;
        t.ngroups = (int)((nblk + (1ll << t.gb) - 1) >> t.gb);
    }
    return t;
}

bool args_ok(const void *rowptr, const int32_t *colidx, int64_t n, int32_t k, double slack,
             int64_t chunk, int32_t R) {
    if (!rowptr || !colidx) return false;
    if (n < 1 || n > (int64_t)INT32_MAX) return false;
    if (k < 1 || k > GREM_MAX_K) return false;
    if (chunk < 1 || R < 0) return false;
    if (!(slack >= 1.0) || std::isinf(slack)) return false;
    return true;
}

// ---- launch bracket: optional event pair per launch, error check after it --------------------------
struct Launcher {
    hipStream_t stream;
    int level = 0;                           // snapshot of the profiling level for this call
    int err = GREM_OK;
    hipEvent_t get_event() {
        {
            std::lock_guard<std::mutex> lock(g.mu);
            if (!g.pool.empty()) { hipEvent_t e = g.pool.back(); g.pool.pop_back(); return e; }
        }
        hipEvent_t e;
        // timing only: no system-scope fence (and the cache write-back it implies) when the event completes
        if (hipEventCreateWithFlags(&e, hipEventDisableSystemFence) != hipSuccess) { err = GREM_ERR_HIP; return nullptr; }
        return e;
    }
    template <typename F> void run(int cls, F &&f) {
        if (err) return;
        hipEvent_t a = nullptr, b = nullptr;
        if (level >= 2) {
            a = get_event(); b = get_event();
            if (err) return;
            if (hipEventRecord(a, stream) != hipSuccess) { err = GREM_ERR_HIP; return; }
        }
        f();
        if (hipGetLastError() != hipSuccess) { err = GREM_ERR_HIP; return; }
        if (level >= 2) {
            if (hipEventRecord(b, stream) != hipSuccess) { err = GREM_ERR_HIP; return; }
            std::lock_guard<std::mutex> lock(g.mu);
            g.events.push_back({cls, a, b});
        }
    }
    void mark() {
        if (err || level < 1) return;
        hipEvent_t e = get_event();
        if (err) return;
        if (hipEventRecord(e, stream) != hipSuccess) { err = GREM_ERR_HIP; return; }
        std::lock_guard<std::mutex> lock(g.mu);
        g.marks.push_back(e);
    }
    bool memset(void *p, int v, size_t bytes) {
        if (err) return false;
        if (bytes && hipMemsetAsync(p, v, bytes, stream) != hipSuccess) { err = GREM_ERR_HIP; return false; }
        return true;
    }
    bool read_back(void *host, const void *dev, size_t bytes) {
        if (err) return false;
        if (hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, stream) != hipSuccess ||
            hipStreamSynchronize(stream) != hipSuccess) { err = GREM_ERR_HIP; return false; }
        return true;
    }
};

size_t apply_lds_bytes(int k) { return (size_t)(1 + kAdmitThreads / 64 + 2) * (size_t)k * 4; }

// `most`: what any call of the kernel may need.  The limit is one of the process, so it is always the same: set to a call's own
// need, it could fall between another thread's setting and its launch.
bool set_lds(const void *f, size_t bytes, size_t most) {
    return bytes <= 64 * 1024 ||
           hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most) == hipSuccess;
}

// ======================================================================================================
// The re-laid-out copy of a graph's entries (two-phase route)
// ======================================================================================================
struct PlanData {
    const void *rowptr = nullptr;
    int rowptr_bits = 0;
    int64_t n = 0, nnz = 0;
    int hub_degree = 0;
    TpGeom geo;
    SweepPlan pl{};
    TpTables tb{};
    uint32_t *T = nullptr;
    uint16_t *R = nullptr;
    u64 *pmisc = nullptr;
    size_t slots = 0;
    unsigned long long maxdeg = 0, hub_entries = 0, total_hubs = 0, max_chunk_hubs = 0;
    bool have_degrees = false;              // maxdeg and nnz have been read back
    std::vector<uint32_t> nvs;              // hub shares per chunk (host copy of pl.ch_nvs)
    std::vector<uint32_t> chunk_hubs;       // hubs per chunk (host copy of pl.ch_nh)
    std::vector<u64> chunk_hub0;            // hubs of the chunks before it (host copy of pl.ch_hub0)
    std::vector<u64> chunk_entries;         // entries of the chunk's rows (0 in a graph without hubs)
    int share_hubs = 0;
    int max_k = 0;                          // largest k whose score workgroups fit the LDS
};

// Sizes of the plan's pieces as functions of what is known at each stage; the same functions serve the
// real carve and the workspace bound.
struct PlanDims {
    int64_t n, nnz;
    TpGeom geo;
    size_t G;                       // slices of all chunks
    size_t hubs;                    // hubs of all chunks (or a bound)
    int npr, nps;
    int nr;                         // rows per chunk: slices, then the most hub shares any chunk has
    size_t slots;
};

size_t plan_slots(int64_t nnz, const TpGeom &geo, int nr) {
    // every sub-segment is padded to a multiple of kSubPad tuples
    const size_t subs = (size_t)geo.nch * (size_t)nr * (size_t)geo.nblk;
    return (size_t)(nnz > 0 ? nnz : 0) + (kSubPad - 1) * subs;
}

void plan_stage1(Carver &c, const PlanDims &d, SweepPlan &pl, u64 *&pmisc) {
    const size_t nch = (size_t)d.geo.nch;
    c.take(pl.sl_reg_cnt, d.G);
    c.take(pl.sl_reg_start, d.G);
    c.take(pl.sl_nh, d.G);
    c.take(pl.sl_hub_start, d.G);
    c.take(pl.sl_hent, d.G);
    c.take(pl.sl_hent_start, d.G);
    c.take(pl.sl_part_reg0, d.G * (size_t)kPlanParts);
    c.take(pl.share_h0, d.G);
    c.take(pl.share_nhs, d.G);
    c.take(pl.ch_regtot, nch);
    c.take(pl.ch_nh, nch);
    c.take(pl.ch_H, nch);
    c.take(pl.ch_nvs, nch);
    c.take(pl.ch_hbase, nch + 1);
    c.take(pl.ch_reg0, nch + 1);
    c.take(pl.ch_hub0, nch + 1);                 // (behind the two before it: one copy to the host brings the three)
    c.take(pmisc, 16);
}

void plan_stage2(Carver &c, const PlanDims &d, SweepPlan &pl) {
    c.take(pl.hub_row, d.hubs + 1);
    c.take(pl.hub_off, d.hubs + (size_t)d.geo.nch + 1);
}

void plan_stage3(Carver &c, const PlanDims &d, TpTables &tb, uint32_t *&T, uint16_t *&R) {
    const size_t segs = (size_t)d.geo.nch * (size_t)d.geo.nblk;
    const size_t rows = (size_t)d.geo.nch * (size_t)d.nr;
    c.take(tb.ta, segs * ((size_t)d.nr + 1));
    c.take(tb.dd, segs * (size_t)d.nr);
    c.take(tb.tstart, segs + 1);
    c.take(tb.sstart, rows + 1);
    c.take(tb.lo, d.G * (size_t)d.npr * ((size_t)d.geo.ngroups + 1));
    c.take(tb.loh, d.G * (size_t)d.nps * ((size_t)d.geo.ngroups + 1));
    c.take(tb.ustart, d.G * (size_t)d.npr);
    c.take(tb.ustart_h, d.G * (size_t)d.nps);
    uint8_t *t8 = nullptr;
    c.take(t8, d.slots * 3 + 16);            // 24 bytes per group of eight tuples: their place in Lx, their columns
    T = reinterpret_cast<uint32_t *>(t8);
    c.take(R, d.slots + 8);                  // row field, 2 bytes per tuple
}

// Builds the plan for (rowptr, colidx, n, chunk) under `o`.  `keep` receives what the plan consists
// of, `temp` the intermediate copy (given back before the function returns).  strict: a graph the
// route cannot take is GREM_ERR_ARG; otherwise the function returns GREM_OK with P.T == nullptr and the
// caller takes the plain route (P.maxdeg and P.nnz are valid once P.have_degrees is set).
// k: the number of partitions of the run the plan is built for, or 0 for any k up to 16 (then
// P.max_k says how far the plan reaches).
template <typename RowT>
int build_plan(PlanData &P, const RowT *rowptr, const int32_t *colidx, int64_t n, int64_t chunk, int32_t k,
               const Opts &o, Arena &keep, Arena &temp, Launcher &L, bool strict) {
    hipStream_t stream = L.stream;
    const int kmax = k ? k : o.plan_max_k;
    const TpGeom geo = tp_geometry(n, chunk, o.col_bits, kmax);
    if (!geo.ok) return GREM_ERR_ARG;            // (callers check the geometry first)
    const int hub_degree = o.hub_degree;
    P.rowptr = rowptr;
    P.rowptr_bits = (int)sizeof(RowT) * 8;
    P.n = n;
    P.hub_degree = hub_degree;
    P.geo = geo;
    PlanDims d{};
    d.n = n;
    d.geo = geo;
    d.G = (size_t)geo.nch * (size_t)geo.nsl;
    const int64_t cl = (int64_t)geo.chunk;
    const int nsl = geo.nsl;
    const unsigned G = (unsigned)d.G;
    SweepPlan &pl = P.pl;
    TpTables &tb = P.tb;

    // ---- stage 1: per slice and per chunk, regular entries, hubs, hub entries, shares
    if (!carve(keep, [&](Carver &c) { plan_stage1(c, d, pl, P.pmisc); })) return GREM_ERR_NOMEM;
    L.memset(P.pmisc, 0, 16 * 8);
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL((k_plan_slices<RowT>), dim3(G), dim3(256), 0, stream, rowptr, n, cl, nsl,
                           geo.srows, (uint32_t)hub_degree, pl, P.pmisc);
    });
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL(k_plan_chunks, dim3((unsigned)geo.nch), dim3(256), 0, stream, n, cl, nsl, geo.srows, geo.nblk,
                           (uint32_t)(kmax > 16 ? kHubsPerShare32 : kHubsPerShare16), pl, P.pmisc);
    });
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL(k_tp_scan, dim3(3), dim3(1024), 0, stream, pl.ch_hbase, (int64_t)geo.nch, pl.ch_reg0,
                           (int64_t)geo.nch, pl.ch_hub0, (int64_t)geo.nch);
    });
    unsigned long long h[16] = {0};
    if (!L.read_back(h, P.pmisc, sizeof(h))) return L.err;
    P.maxdeg = h[0];
    P.nnz = (int64_t)h[3];
    P.have_degrees = true;
    P.max_chunk_hubs = h[6];
    P.hub_entries = h[8];
    P.total_hubs = h[12];
    d.nnz = P.nnz;
    d.hubs = (size_t)P.total_hubs;

    // ---- stage 2: the chunks' hub lists, the hubs every share touches
    if (!carve(keep, [&](Carver &c) { plan_stage2(c, d, pl); })) return GREM_ERR_NOMEM;
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL((k_plan_hubs<RowT>), dim3(G), dim3(256), 0, stream, rowptr, n, cl, nsl,
                           geo.srows, (uint32_t)hub_degree, pl);
    });
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL(k_plan_shares, dim3((G + 255) / 256), dim3(256), 0, stream, n, cl, nsl, (int)G, pl,
                           P.pmisc);
    });
    P.nvs.assign((size_t)geo.nch, 0u);
    P.chunk_hubs.assign((size_t)geo.nch, 0u);
    P.chunk_hub0.assign((size_t)geo.nch + 1, 0ull);
    P.chunk_entries.assign((size_t)geo.nch, 0ull);
    if (P.total_hubs != 0) {
        std::vector<u64> starts((size_t)(pl.ch_hub0 - pl.ch_hbase) + (size_t)geo.nch + 1);
        if (hipMemcpyAsync(P.nvs.data(), pl.ch_nvs, (size_t)geo.nch * 4, hipMemcpyDeviceToHost, stream) != hipSuccess ||
            hipMemcpyAsync(P.chunk_hubs.data(), pl.ch_nh, (size_t)geo.nch * 4, hipMemcpyDeviceToHost, stream) != hipSuccess ||
            hipMemcpyAsync(starts.data(), pl.ch_hbase, starts.size() * 8, hipMemcpyDeviceToHost, stream) != hipSuccess) {
            (void)hipStreamSynchronize(stream);
            return GREM_ERR_HIP;
        }
        if (!L.read_back(h, P.pmisc, sizeof(h))) return L.err;
        const u64 *hub = starts.data(), *regular = hub + (pl.ch_reg0 - pl.ch_hbase), *hubs = hub + (pl.ch_hub0 - pl.ch_hbase);
        for (int c = 0; c < geo.nch; ++c) P.chunk_entries[c] = hub[c + 1] - hub[c] + regular[c + 1] - regular[c];
        P.chunk_hub0.assign(hubs, hubs + geo.nch + 1);
    } else if (L.err) {
        return L.err;
    }
    const int share_hubs = (int)h[5];
    P.share_hubs = share_hubs;

    // ---- does the route fit?  A score workgroup's LDS (two per CU fit when a share touches few hubs);
    // a share may touch kMaxShareHubs hubs; sub-segment offsets are 32-bit
    {
        auto score_fits = [&](int kk) {
            const size_t dyn = ((size_t)geo.srows / 2 + (size_t)share_hubs * kk + 3 * (size_t)kk) * 4;
            if (kk <= 16) return dyn + (size_t)geo.srows * 32 <= kScoreLds16;
            return geo.cb <= 16 && dyn + (size_t)geo.srows * 64 <= kScoreLds32;    // (a byte per label in the look-up's LDS)
        };
        int max_k = kmax;
        while (max_k > 1 && !score_fits(max_k) && k == 0) --max_k;
        P.max_k = max_k;
        // (the index of a word of Lx -- eight labels -- travels in 32 bits of T)
        const bool fits = score_fits(max_k) && share_hubs <= kMaxShareHubs &&
                          plan_slots(P.nnz, geo, 2 * geo.nsl) < (1ull << 35) &&
                          h[7] + 8ull * (2ull * (unsigned long long)geo.nsl + 2) * geo.nblk < (1ull << 32);
        if (!fits) return strict ? GREM_ERR_ARG : GREM_OK;
    }

    // ---- stage 3: shapes of the re-layout kernels, then the tables and streams
    // step 1 collects a unit's tuples in LDS: cut the slices (shares) in as many parts as it takes for
    // the largest to fit, two workgroups per CU
    constexpr size_t kGroupLds = 79 * 1024;
    auto group_fixed = [&](bool share, int np) {
        return tp_group_words(share, np, share_hubs, geo.nblk, geo.ngroups) * 4;
    };
    auto group_cap = [&](bool share, int np) {
        const size_t fixed = group_fixed(share, np);
        return (uint32_t)(kGroupLds > fixed ? (kGroupLds - fixed) / 4 : 0);
    };
    int npr = 1, nps = 1;
    const int most_parts = geo.srows / kPlanThreads;        // of a slice
    // ... and, if that takes no more than kMaxParts, so small that a thread holds its share of the unit's
    // entries in registers (one round of kTpThreads * kTpBatch entries)
    const unsigned long long one_round = (unsigned long long)kTpThreads * kTpBatch;
    auto fits_unit = [&](bool share, int np, unsigned long long most, bool in_regs) {
        const unsigned long long unit = most / np + most / (8ull * np) + 64;
        return group_cap(share, np) >= unit && (!in_regs || unit <= one_round);
    };
    while (npr < most_parts && !fits_unit(false, npr, h[9], false)) npr *= 2;
    while (nps < kMaxParts && !fits_unit(true, nps, h[10], false)) nps += 1;
    {
        // slices differ in size: it is the average one whose parts should take one round (the larger ones
        // take two, and their tuples still fit LDS)
        const unsigned long long avg_slice =
            ((unsigned long long)P.nnz - P.hub_entries) / (unsigned long long)(d.G ? d.G : 1) + 1;
        int a = npr, b = nps;
        while (a < most_parts && !fits_unit(false, a, avg_slice, true)) a *= 2;
        while (b < kMaxParts && !fits_unit(true, b, h[10], true)) b += 1;
        if (fits_unit(false, a, avg_slice, true) && fits_unit(false, a, h[9], false)) npr = a;
        if (fits_unit(true, b, h[10], true)) nps = b;
    }
    d.npr = npr;
    d.nps = nps;
    const unsigned max_shares = (unsigned)h[11];            // no chunk has more hub shares than this
    d.nr = geo.nsl + (int)max_shares;
    d.slots = plan_slots(P.nnz, geo, d.nr);
    P.slots = d.slots;
    if (!carve(keep, [&](Carver &c) { plan_stage3(c, d, tb, P.T, P.R); })) { P.T = nullptr; return GREM_ERR_NOMEM; }
    tb.chunk = geo.chunk;
    tb.chunk_shift = geo.shift;
    {   // round-up magic number: exact for dividends below 2^31 (vertex ids are)
        uint32_t sh = 0;
        while ((1ull << sh) < geo.chunk) ++sh;
        tb.chunk_magic_shift = sh > 0 ? sh - 1 : 0;
        tb.chunk_magic = geo.chunk > 1
            ? (uint32_t)((((unsigned long long)1 << (32 + tb.chunk_magic_shift)) + geo.chunk - 1) / geo.chunk)
            : 0u;
        if (geo.chunk == 1) tb.chunk_shift = 0;
    }
    tb.nch = geo.nch;
    tb.nsl = geo.nsl;
    tb.srows = geo.srows;
    tb.nr = d.nr;
    tb.nbc = geo.nbc;
    tb.nblk = geo.nblk;
    tb.cb = geo.cb;
    tb.flat = (tb.chunk_shift >= geo.cb && geo.chunk > 1) ? 1 : 0;
    tb.gb = geo.gb;
    tb.ngroups = geo.ngroups;
    tb.npr = npr;
    tb.prows = geo.srows / npr;
    tb.pstep = geo.srows / kPlanThreads / npr;
    tb.nps = nps;

    const Arena::Mark tmark = temp.mark();
    const size_t subs = (size_t)geo.nch * (size_t)d.nr * (size_t)geo.nblk;
    uint32_t *U = (uint32_t *)temp.alloc((size_t)(P.nnz > 0 ? P.nnz : 0) * 4 + 16);
    tb.cnt = U ? (uint32_t *)temp.alloc(subs * 4) : nullptr;
    if (!U || !tb.cnt) { temp.release_to(tmark); P.T = nullptr; return GREM_ERR_NOMEM; }
    const u64 hub_base = (u64)P.nnz - P.hub_entries;        // U: the regular entries, then the hub streams

    const uint32_t capR = group_cap(false, npr), capS = group_cap(true, nps);
    const size_t groupR_lds = group_fixed(false, npr) + (size_t)capR * 4;
    const size_t groupS_lds = group_fixed(true, nps) + (size_t)capS * 4;
    // step 2: up to 8 slices at a time, but no more than fit the stage at the average row's size (a batch that does
    // not fit is halved by the kernel, at the price of setting its tables up again); four workgroups per CU, or
    // three if two rows at a time would not fit then (111M vertices: 10.1 ms with four of 39 KB, 10.6 with three)
    const int nbg = geo.nblk < (1 << geo.gb) ? geo.nblk : (1 << geo.gb);
    const int npm = npr > nps ? npr : nps;
    const double per_row = (double)d.slots / ((double)geo.nch * (double)d.nr) / (double)geo.ngroups;
    auto place_cap = [&](size_t lds, int rows) -> size_t {
        const size_t fixed = tp_place_fixed_bytes(nbg, rows, rows * npm);
        return lds > fixed ? (lds - fixed) / 4 : 0;
    };
    size_t place_room = 39 * 1024;
    if (per_row * 2.5 > (double)place_cap(place_room, 2)) place_room = 52 * 1024;
    int batch = 8192 / nbg;
    if (batch > 8) batch = 8;
    if (batch < 1) batch = 1;
    while (batch > 1 && per_row * 1.25 * batch > (double)place_cap(place_room, batch)) --batch;
    const int maxruns = batch * npm;
    const size_t place_fixed = tp_place_fixed_bytes(nbg, batch, maxruns);
    const uint32_t capP = (uint32_t)place_cap(place_room, batch);
    const size_t place_lds = place_fixed + (size_t)capP * 4;
    const int64_t place_wgs = (int64_t)geo.ngroups * geo.nch;
    int64_t split = (kPlaceGrid + place_wgs - 1) / place_wgs;      // (no more than a batch of rows each)
    if (split > (d.nr + batch - 1) / batch) split = (d.nr + batch - 1) / batch;
    L.memset(tb.cnt, 0, subs * 4);
    if (L.err || !set_lds((const void *)k_tp_group<RowT, false>, groupR_lds, kGroupLds) ||
        !set_lds((const void *)k_tp_group<RowT, true>, groupS_lds, kGroupLds)) {
        temp.release_to(tmark);
        P.T = nullptr;
        return GREM_ERR_HIP;
    }
    const unsigned segs = (unsigned)((int64_t)geo.nch * geo.nblk);
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL((k_tp_group<RowT, false>), dim3(G * (unsigned)npr), dim3(kTpThreads), groupR_lds, stream,
                           rowptr, colidx, n, (uint32_t)hub_degree, pl, tb, share_hubs, capR, (int)nsl, U, hub_base);
    });
    // shares: no chunk has more than max_shares of them (none at all: nothing to launch)
    if (max_shares != 0)
        L.run(GREM_KERNEL_RELAYOUT, [&] {
            hipLaunchKernelGGL((k_tp_group<RowT, true>), dim3((unsigned)geo.nch * max_shares * (unsigned)nps),
                               dim3(kTpThreads), groupS_lds, stream, rowptr, colidx, n, (uint32_t)hub_degree, pl, tb,
                               share_hubs, capS, (int)max_shares, U, hub_base);
        });
    const unsigned rows_all = (unsigned)((int64_t)geo.nch * d.nr);
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL(k_tp_scan_t, dim3((segs + 255) / 256), dim3(256), 0, stream, tb);
    });
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL(k_tp_scan_d, dim3((rows_all + 255) / 256), dim3(256), 0, stream, tb);
    });
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL(k_tp_scan, dim3(2), dim3(1024), 0, stream, tb.tstart, (int64_t)segs, tb.sstart,
                           (int64_t)rows_all, (u64 *)nullptr, (int64_t)0);
    });
    L.run(GREM_KERNEL_RELAYOUT, [&] {
        hipLaunchKernelGGL(k_tp_place, dim3((unsigned)(place_wgs * split)), dim3(kPlaceThreads), place_lds,
                           stream, n, pl, tb, U, P.T, P.R, batch, capP, (int)split);
    });
    temp.release_to(tmark);
    if (L.err) { P.T = nullptr; return L.err; }
    return GREM_OK;
}

// ======================================================================================================
// State of one run (Alg. 1's parts, sizes, nbr_counts and the admission tables)
// ======================================================================================================
template <typename LabelT> struct CallState {
    LabelT *Lc = nullptr, *prop = nullptr;
    long long *S = nullptr, *S2 = nullptr, *room = nullptr, *fillSorted = nullptr, *fillC = nullptr;
    uint32_t *cnt = nullptr, *tot = nullptr, *ocnt = nullptr;
    int32_t *fillRank = nullptr;
    unsigned long long *misc = nullptr;
    bool seed_complete = false;        // (host) the seed labels every vertex
};

// 64-bit words behind CallState::misc for the counts of the chunks' long rows and their parts
size_t long_count_words(int64_t n, int64_t cl) {
    const int64_t nchunks = (n + cl - 1) / cl;
    return nchunks <= kLongChunks ? (size_t)((1 + kLongPartSizes) * nchunks + 1) / 2 : 0;
}

template <typename LabelT>
void state_common(Carver &c, CallState<LabelT> &st, int64_t n, int64_t cl, int32_t k) {
    const size_t ntiles = (size_t)((cl + kAdmitTile - 1) / kAdmitTile);
    c.take(st.Lc, (size_t)n);
    c.take(st.prop, (size_t)cl);
    c.take(st.S, (size_t)k);
    c.take(st.S2, (size_t)k);                // the sizes' other copy (the one-launch spill reads one, writes the other)
    c.take(st.cnt, 2 * ntiles * (size_t)k);      // (a slice of fewer rows than a tile has counts of its own)
    c.take(st.tot, 2 * (size_t)k);
    c.take(st.room, (size_t)k);
    c.take(st.ocnt, ntiles);
    c.take(st.fillRank, (size_t)k);
    c.take(st.fillSorted, (size_t)k);
    c.take(st.fillC, (size_t)k + 1);
    c.take(st.misc, 32 + long_count_words(n, cl));
}

// prepass: compact labels and sizes from the seed, its validity; with rowptr also the largest degree
template <typename RowT, typename LabelT>
void launch_prepass(Launcher &L, const RowT *rowptr_or_null, const int32_t *seed, int64_t n, int32_t k, long long P,
                    CallState<LabelT> &st, uint32_t long_degree = 0xFFFFFFFFu, LongCounts lc = LongCounts{}) {
    hipStream_t stream = L.stream;
    L.memset(st.S, 0, (size_t)k * 8);
    const bool counts = lc.nchunks != 0;
    if (counts) lc.count = (uint32_t *)(st.misc + 32);
    L.memset(st.misc, 0, (32 + (counts ? long_count_words(n, lc.chunk) : 0)) * 8);
    int64_t blocks = (n + 255) / 256;
    if (blocks > 256 * 8) blocks = 256 * 8;      // (every workgroup adds its sums at the same few addresses)
    L.run(GREM_KERNEL_PREPASS, [&] {
        hipLaunchKernelGGL((k_prepass<RowT, LabelT>), dim3((unsigned)blocks), dim3(256), 0, stream, rowptr_or_null, seed,
                           n, (int)k, st.Lc, (unsigned long long *)st.S, st.misc, long_degree, lc);
    });
    if (seed)
        L.run(GREM_KERNEL_PREPASS, [&] {
            hipLaunchKernelGGL(k_check_seed_sizes, dim3((k + 255) / 256), dim3(256), 0, stream, st.S, (int)k, P, st.misc);
        });
}

template <typename LabelT>
void launch_spill(Launcher &L, CallState<LabelT> &st, int64_t lo, int64_t hi, int32_t k, unsigned admit_blocks) {
    hipStream_t stream = L.stream;
    L.run(GREM_KERNEL_SPILL_SCAN, [&] {
        hipLaunchKernelGGL(k_spill_scan, dim3(1), dim3(kScanThreads), 0, stream, st.ocnt, (int)admit_blocks, (int)k, st.S,
                           st.fillRank, st.fillSorted, st.fillC, st.misc);
    });
    L.run(GREM_KERNEL_SPILL_FILL, [&] {
        hipLaunchKernelGGL((k_spill_fill<LabelT>), dim3(admit_blocks), dim3(kAdmitThreads), (size_t)k * 4, stream, st.Lc, lo,
                           hi, (int)k, st.ocnt, st.fillRank, st.fillC, (unsigned long long *)st.S, st.misc);
    });
}

template <typename LabelT>
void launch_outputs(Launcher &L, CallState<LabelT> &st, int64_t n, int32_t k, int32_t *labels_out, int64_t *sizes_out) {
    hipStream_t stream = L.stream;
    int64_t blocks = (n + 255) / 256;
    if (blocks > 256 * 32) blocks = 256 * 32;
    if (labels_out)
        L.run(GREM_KERNEL_EXPAND, [&] {
            hipLaunchKernelGGL((k_expand<LabelT>), dim3((unsigned)blocks), dim3(256), 0, stream, st.Lc, n, labels_out);
        });
    if (sizes_out)
        L.run(GREM_KERNEL_EXPAND, [&] {
            hipLaunchKernelGGL(k_copy_sizes, dim3((k + 255) / 256), dim3(256), 0, stream, st.S, (int)k, sizes_out);
        });
}

// ---- two-phase route: per-call arrays beside the common state ---------------------------------------
struct TpState {
    uint32_t *Lx = nullptr, *Hhub = nullptr, *E32 = nullptr, *Ehub = nullptr;
    uint16_t *Rdyn = nullptr, *E16 = nullptr;
    uint8_t *Lc4 = nullptr;            // k <= 16: the labels two per byte, kept by the admission from the second pass on
    uint8_t *hub_old = nullptr;        // the labels of the chunk's hubs, by their place in its list (see k_admit_hubs)
    uint32_t *coarse = nullptr;        // two tables of the tiles' mover counts added up 32 tiles at a time (k_admit_hubs)
};

// twice: two tables of the chunk's hub counts and of the hubs' estimates (the admission that also does the
// hubs' part reads one and writes the other)
void state_two_phase(Carver &c, TpState &t, int64_t n, int32_t k, size_t slots, size_t max_chunk_hubs, size_t total_hubs,
                     bool seeded, bool use16, bool external_E, bool twice) {
    uint8_t *lx = nullptr;
    c.take(lx, (k <= 16 ? slots / 2 : slots) + 16);               // label, 4 bits per tuple (8 when k > 16)
    t.Lx = reinterpret_cast<uint32_t *>(lx);
    c.take(t.Hhub, (twice ? 2 : 1) * (max_chunk_hubs + 1) * (size_t)k);
    c.take(t.Rdyn, seeded && k == 16 ? slots + 8 : 0);            // seeded runs: R with the unassigned neighbours marked
    c.take(t.E16, use16 ? (size_t)n * (size_t)k : 0);
    c.take(t.E32, (!use16 && !external_E) ? (size_t)n * (size_t)k : 0);
    c.take(t.Ehub, (use16 && !external_E) ? (twice ? 2 : 1) * (total_hubs + 1) * (size_t)k : 0);
    c.take(t.Lc4, k <= 16 ? (size_t)n / 2 + 16 : 0);
    c.take(t.hub_old, twice ? max_chunk_hubs + 16 : 0);
    c.take(t.coarse, twice ? 2 * (size_t)(kAdmitTilesMax / kCoarseTiles) * (size_t)k : 0);
}

// The admission kernel does the hubs' blend and proposal itself when every chunk has few hubs and few
// tiles and the hubs' estimates live in a table of their own (16-bit estimates, no caller's array).
bool admission_takes_hubs(const PlanData &P, bool use16, bool external_E) {
    const int64_t tiles = ((int64_t)P.geo.chunk + kAdmitTile - 1) / kAdmitTile;
    return use16 && !external_E && P.max_chunk_hubs <= (unsigned long long)kAdmitHubsMax && tiles <= kAdmitTilesMax;
}

// Alg. 1's loop on a plan.  `prepared`: the common state with the prepass run and the seed validated by
// the caller; otherwise this function does both (one read-back when there is a seed).
// fixed_labels: nothing is decided.  The seed is a labelling that stays as it is (R = 0, estimates_out
// given): after the initial look-up of every label, each chunk runs its counting launches only, and
// estimates_out receives cnt_nbrs (Alg. 2) of every vertex under that labelling.
template <typename RowT>
int run_two_phase(const PlanData &P, int32_t k, double slack, int32_t R, const int32_t *seed, int32_t *labels_out,
                  int64_t *sizes_out, uint32_t *estimates_out, Arena &mem, Launcher &L, CallState<uint8_t> *prepared,
                  bool fixed_labels = false) {
    hipStream_t stream = L.stream;
    const RowT *rowptr = (const RowT *)P.rowptr;
    const int64_t n = P.n;
    const TpGeom &geo = P.geo;
    const TpTables &tb = P.tb;
    const SweepPlan &pl = P.pl;
    const int64_t cl = (int64_t)geo.chunk;
    const long long cap = grem_capacity(n, k, slack);
    const bool external_E = estimates_out != nullptr;
    const int hub_degree = P.hub_degree;
    if (R >= 32 || (P.maxdeg << R) >= (1ull << 32)) return GREM_ERR_RANGE;
    if (external_E && (((uintptr_t)estimates_out) & 15u) != 0) return GREM_ERR_ARG;
    if (fixed_labels && (!seed || !external_E || R != 0)) return GREM_ERR_ARG;
    // estimates of the regular rows stay below hub_degree * 2^R: 16 bits when that fits
    // (the counts of a fixed labelling go straight to the caller's 32-bit array: no 16-bit copy to expand)
    const bool use16 = !fixed_labels && (((unsigned long long)(hub_degree - 1)) << R) <= 65535ull;

    const bool hubs_in_admission = admission_takes_hubs(P, use16, external_E);

    CallState<uint8_t> st;
    if (prepared) {
        st = *prepared;
    } else {
        if (!carve(mem, [&](Carver &c) { state_common(c, st, n, cl, k); })) return GREM_ERR_NOMEM;
    }
    TpState t;
    if (!carve(mem, [&](Carver &c) {
            state_two_phase(c, t, n, k, P.slots, (size_t)P.max_chunk_hubs, (size_t)P.total_hubs, seed != nullptr, use16,
                            external_E, hubs_in_admission);
        }))
        return GREM_ERR_NOMEM;
    if (!prepared) {
        launch_prepass<RowT, uint8_t>(L, (const RowT *)nullptr, seed, n, k, cap, st);
        if (seed) {
            unsigned long long h[16] = {0};
            if (!L.read_back(h, st.misc, sizeof(h))) return L.err;
            if (h[1] != 0 || h[2] != 0) return GREM_ERR_SEED;
            st.seed_complete = h[5] == 0;
        }
    }
    uint32_t *E32 = external_E ? estimates_out : t.E32;
    uint32_t *Ehub_rows = (use16 && !external_E) ? nullptr : E32;    // hubs: rows of E32 when there is one, else Ehub
    if (k > P.max_k) return GREM_ERR_ARG;
    const bool wide = k > 16;                     // 8-bit labels in Lx, 128 KB of counters per slice
    const size_t score_lds = ((size_t)geo.srows / 2 + (size_t)P.share_hubs * k + 3 * (size_t)k) * 4 +
                             (wide ? (size_t)geo.srows * 64 : 0);
    const int cell_rows = geo.srows < kAdmitTile ? geo.srows : kAdmitTile, cpt = kAdmitTile / cell_rows;
    const size_t lookup_lds = wide ? ((size_t)1 << (geo.cb > 4 ? geo.cb : 4)) : ((size_t)1 << (geo.cb > 5 ? geo.cb - 1 : 4));
    // f(kernel, estimates): the score kernel for the estimates' type, the partitions and the rows per slice (skip:
    // neighbours without a label among 32 partitions)
    auto with_score = [&](bool skip, auto &&f) {
        auto rows = [&](auto sr) {
            constexpr int SR = decltype(sr)::value;
            if (wide) {
                if (skip) { if (use16) f(k_tp_score<uint16_t, 32, false, SR, true>, t.E16); else f(k_tp_score<uint32_t, 32, false, SR, true>, E32); }
                else if (use16) f(k_tp_score<uint16_t, 32, false, SR>, t.E16);
                else f(k_tp_score<uint32_t, 32, false, SR>, E32);
            } else if (k <= 8) {                         // (a row's few counters spread over the LDS banks)
                if (use16) f(k_tp_score<uint16_t, 16, true, SR>, t.E16);
                else f(k_tp_score<uint32_t, 16, true, SR>, E32);
            } else {
                if (use16) f(k_tp_score<uint16_t, 16, false, SR>, t.E16);
                else f(k_tp_score<uint32_t, 16, false, SR>, E32);
            }
        };
        if (geo.srows == 512) rows(std::integral_constant<int, 512>{});
        else if (geo.srows == 1024) rows(std::integral_constant<int, 1024>{});
        else rows(std::integral_constant<int, kSliceRows>{});
    };
    constexpr size_t most_lookup = (size_t)1 << (kMaxColBits - 1);         // (a byte per label: 2^16 columns at most)
    bool lds_ok = wide ? set_lds((const void *)k_tp_lookup<true, false, 8>, lookup_lds, most_lookup)
                       : set_lds((const void *)k_tp_lookup<true, false, 4>, lookup_lds, most_lookup) &&
                             set_lds((const void *)k_tp_lookup<true, true, 4>, lookup_lds, most_lookup);
    const size_t most_score = wide ? kScoreLds32 : kScoreLds16 - (size_t)geo.srows * 32;   // (one kernel per number of rows)
    for (int skip = 0; skip < 2; ++skip)
        with_score(skip != 0, [&](auto kernel, auto *) { lds_ok = lds_ok && set_lds((const void *)kernel, score_lds, most_score); });
    if (!lds_ok) return GREM_ERR_HIP;
    L.memset(t.Hhub, 0, (hubs_in_admission ? 2 : 1) * ((size_t)P.max_chunk_hubs + 1) * (size_t)k * 4);
    const size_t coarse_row = (size_t)(kAdmitTilesMax / kCoarseTiles) * (size_t)k;
    if (hubs_in_admission) L.memset(t.coarse, 0, 2 * coarse_row * 4);

    // Ids in order of degree: a chunk has more than twice its share of the entries, and its columns, as a graph's entries go both ways, too.
    // A sweep then finds each workgroup's block by the blocks' sizes, which costs it some 2 us (25M vertices, 250M entries, permuted: 0.82 -> 0.87 ms;
    // 13.9M by degree, k = 32 0.69 -> 0.42).
    const bool lopsided = *std::max_element(P.chunk_entries.begin(), P.chunk_entries.end()) * (u64)geo.nch > 2 * (u64)P.nnz;
    // look-ups of the labels of chunks [c0, c0 + count)
    auto lookup = [&](int c0, int count, int cmin, bool from_lds, bool mark, const uint8_t *labels4 = nullptr) {
        if (cmin >= geo.nch) return;
        // (whole eights where there are as many: a share has the same place among the XCDs whatever its block, see k_tp_lookup)
        const uint32_t by_work = (uint32_t)std::min<int64_t>(P.nnz / geo.nblk / 8192 + 1, kLookupMany);
        auto per_block = [&](uint32_t all) {
            const uint32_t w = std::max(std::min(all / (uint32_t)geo.nbc, by_work), 1u);
            return w < 8 ? w : w / 8 * 8;
        };
        LookupShares deal{per_block(kLookupFew), 0u, 0u};
        dim3 grid;
        if (count == geo.nch && lopsided) {
            const uint64_t groups = P.slots / 8;
            deal.per = (uint32_t)std::max<uint64_t>(groups / kLookupSweep + 1, 1024);
            grid = dim3(lookup_sweep_grid(groups, (uint32_t)geo.nblk, deal));
        } else {
            // (workgroups beyond the blocks' shares cost 2 us a launch, so that `many` are launched for a chunk of long rows only: as a
            // graph's entries go both ways, its columns are then as long.  128 KB of labels: one workgroup per CU)
            const bool lengthy = count == 1 && geo.cb <= 17 && P.chunk_entries[(size_t)c0] / 8 > (u64)kLookupFew * kLookupLong;
            if (count > 1) {
                // (from global memory: no labels to copy, so as many workgroups as there is work for.  Planned, k = 16, a tenth seeded, chunks of 2^20:
                // 13.9M vertices 4.77 | 4.73 ms, 40M 9.06 | 8.96)
                const uint64_t most = from_lds ? std::min<uint64_t>(kLookupFew / (uint32_t)geo.nbc, kLookupSweep / ((uint64_t)count * geo.nbc)) : kLookupMany / (uint32_t)geo.nbc;
                deal.few = (uint32_t)std::max<uint64_t>(std::min<uint64_t>(most, by_work), 1);
            }
            deal.many = lengthy ? per_block(kLookupMany) : deal.few;
            grid = dim3((uint32_t)geo.nbc * deal.many, (unsigned)count);
        }
        auto go = [&](auto kernel, size_t lds) {
            hipLaunchKernelGGL(kernel, grid, dim3(kTpThreads), lds, stream, P.T, t.Lx, P.R, t.Rdyn, tb,
                               (const uint8_t *)st.Lc, labels4, n, c0, cmin, deal);
        };
        L.run(GREM_KERNEL_LOOKUP, [&] {
            if (wide) {
                go(k_tp_lookup<true, false, 8>, lookup_lds);
            } else {
                if (!from_lds) go(k_tp_lookup<false, true, 4>, 0);
                else if (mark) go(k_tp_lookup<true, true, 4>, lookup_lds);
                else go(k_tp_lookup<true, false, 4>, lookup_lds);
            }
        });
    };
    // A seed that leaves vertices without a label: their entries are told by the label that the look-up stores, except
    // with 16 partitions in four bits, where the first pass reads its row fields from Rdyn and the initial look-up,
    // from global memory, marks the entries there.
    const bool partly = seed != nullptr && !st.seed_complete, marks = partly && k == 16;
    if (seed) {        // the seeds are the labels every first-pass look-up starts from
        const int most = lopsided ? geo.nch : 32768;
        for (int c0 = 0; c0 < geo.nch; c0 += most) lookup(c0, std::min(geo.nch - c0, most), 0, !marks, marks);
    }
    L.mark();
    if (fixed_labels) {                     // counts only: nothing to admit, no new labels to look up
        const bool skip = partly && k == 32;
        auto counts = [&](auto kernel) {
            if (!set_lds((const void *)kernel, score_lds, most_score)) { L.err = GREM_ERR_HIP; return; }
            L.run(GREM_KERNEL_HUBS, [&] {
                hipLaunchKernelGGL(k_tp_clear_hubs, dim3((unsigned)std::min<size_t>((size_t)P.total_hubs * k / 256 + 1, 2048)), dim3(256), 0, stream,
                                   (const int32_t *)pl.hub_row, (size_t)P.total_hubs, (int)k, E32);
            });
            L.run(GREM_KERNEL_SCORE, [&] {
                hipLaunchKernelGGL(kernel, dim3((unsigned)((size_t)geo.nch * (size_t)geo.nsl)), dim3(kTpThreads), score_lds, stream,
                                   marks ? (const uint16_t *)t.Rdyn : (const uint16_t *)P.R, (const uint32_t *)t.Lx, tb, pl, n, cl, (int)k, P.share_hubs, E32);
            });
        };
        auto rows = [&](auto sr) {
            constexpr int SR = decltype(sr)::value;
            if (wide) { if (skip) counts(k_tp_counts<32, false, SR, true>); else counts(k_tp_counts<32, false, SR, false>); }
            else if (k <= 8) counts(k_tp_counts<16, true, SR, false>);
            else counts(k_tp_counts<16, false, SR, false>);
        };
        if (geo.srows == 512) rows(std::integral_constant<int, 512>{});
        else if (geo.srows == 1024) rows(std::integral_constant<int, 1024>{});
        else rows(std::integral_constant<int, kSliceRows>{});
        L.mark();
        return L.err;
    }
    const size_t max_chunk_hubs = (size_t)P.max_chunk_hubs;
    uint32_t prev_hubs = 0;                 // hubs of the chunk before (whose counts the admission clears)
    // first pass, chunks of at most kSpillSmallTiles tiles: the spill is one launch that reads the sizes from one
    // array and writes them to the other; the two take turns from chunk to chunk
    const bool spill_small = (cl + kAdmitTile - 1) / kAdmitTile <= kSpillSmallTiles;
    long long *Snow = st.S;
    for (int pass = 0; pass <= R && !L.err; ++pass) {
        for (int64_t c = 0; c < geo.nch && !L.err; ++c) {
            const int64_t lo = c * cl;
            const int64_t hi = (lo + cl < n) ? lo + cl : n;
            const int64_t len = hi - lo;
            const unsigned admit_blocks = (unsigned)((len + kAdmitTile - 1) / kAdmitTile);
            const unsigned blocks = (unsigned)((len + geo.srows - 1) / geo.srows);
            const int ncells = (int)((len + cell_rows - 1) / cell_rows);
            const int jlim = (pass == 0 && !seed) ? (int)c * geo.nbc : geo.nblk;
            // the estimates are state between passes and, if the caller asked for them, output: the last
            // pass does not store them otherwise
            const int store_e = (pass < R || external_E) ? 1 : 0;
            const uint16_t *rows_now = (marks && pass == 0) ? t.Rdyn : P.R;
            // from the second pass on every vertex has a label before its chunk's admission, which then
            // also leaves the chunk's labels two per byte for the look-ups (chunk starts must be even)
            uint8_t *packed_now = (pass >= 1 && t.Lc4 && (cl & 1) == 0) ? t.Lc4 : nullptr;
            const int64_t step = (int64_t)pass * geo.nch + c;
            uint32_t *Hnow = t.Hhub + (hubs_in_admission ? (size_t)(step & 1) * ((size_t)max_chunk_hubs + 1) * (size_t)k : 0);
            auto score = [&](auto kernel, auto *Eptr) {
                hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kTpThreads), score_lds, stream, rows_now, t.Lx, tb, pl,
                                   (const uint8_t *)st.Lc, Snow, Eptr, Hnow, (uint8_t *)st.prop, st.cnt, st.room, (int)c,
                                   lo, hi, (int)k, jlim, P.share_hubs, P.nvs[(size_t)c], pass, cap, store_e,
                                   hubs_in_admission ? t.hub_old : (uint8_t *)nullptr,
                                   hubs_in_admission ? t.coarse + (size_t)(step & 1) * coarse_row : (uint32_t *)nullptr);
            };
            L.run(GREM_KERNEL_SCORE, [&] { with_score(partly && pass == 0 && k == 32, score); });
            if (hubs_in_admission) {
                // one launch: every workgroup works out the chunk's hubs for itself; two tables of hub counts
                // take turns from chunk to chunk, two tables of hub estimates from pass to pass
                const size_t hrow = (size_t)max_chunk_hubs + 1, erow = (size_t)P.total_hubs + 1;
                const uint32_t nh = P.chunk_hubs[(size_t)c];
                const size_t hub0 = (size_t)P.chunk_hub0[(size_t)c];
                uint32_t *Hother = t.Hhub + (size_t)((step + 1) & 1) * hrow * (size_t)k;
                const uint32_t *Eold = t.Ehub + ((size_t)((pass + 1) & 1) * erow + hub0) * (size_t)k;
                uint32_t *Enew = t.Ehub + ((size_t)(pass & 1) * erow + hub0) * (size_t)k;
                L.run(GREM_KERNEL_APPLY, [&] {
                    const unsigned tpw = admit_blocks <= (unsigned)kAdmitGrid ? 1u : admit_blocks <= 2u * kAdmitGrid ? 2u : 4u;
                    auto go = [&](auto kernel) {
                        hipLaunchKernelGGL(kernel, dim3((admit_blocks + tpw - 1) / tpw), dim3(kAdmitTile), 0, stream, (uint8_t *)st.Lc, (const uint8_t *)st.prop,
                                           lo, hi, (int)k, (const uint32_t *)st.cnt, (int)admit_blocks,
                                           (const long long *)st.room, (unsigned long long *)Snow, st.ocnt, pass, packed_now,
                                           (const int32_t *)(pl.hub_row + hub0), (const uint8_t *)t.hub_old, nh,
                                           (const uint32_t *)Hnow, Hother,
                                           prev_hubs, Eold, Enew, store_e,
                                           (const uint32_t *)(t.coarse + (size_t)(step & 1) * coarse_row),
                                           t.coarse + (size_t)((step + 1) & 1) * coarse_row, ncells);
                    };
                    // (slices of fewer rows than a tile are those of short chunks: one tile per workgroup)
                    if (wide) {
                        if (cpt == 2) go(k_admit_hubs<32, 1, 2>);
                        else if (tpw == 1) go(k_admit_hubs<32, 1, 1>);
                        else if (tpw == 2) go(k_admit_hubs<32, 2, 1>);
                        else go(k_admit_hubs<32, 4, 1>);
                    } else {
                        if (cpt == 2) go(k_admit_hubs<16, 1, 2>);
                        else if (tpw == 1) go(k_admit_hubs<16, 1, 1>);
                        else if (tpw == 2) go(k_admit_hubs<16, 2, 1>);
                        else go(k_admit_hubs<16, 4, 1>);
                    }
                });
                prev_hubs = nh;
            } else {
            // (one workgroup more than the hubs need: it adds up the chunk's mover counts)
            L.run(GREM_KERNEL_HUBS, [&] {
                if (wide)
                    hipLaunchKernelGGL(k_hub_finalize<32>, dim3((unsigned)((max_chunk_hubs + 7) / 8) + 1), dim3(256), 0,
                                       stream, pl, (const uint8_t *)st.Lc, st.room, Ehub_rows, t.Ehub, t.Hhub,
                                       (uint8_t *)st.prop, st.cnt, (int)c, lo, (int)k, pass, store_e, ncells, cell_rows,
                                       st.tot);
                else
                    hipLaunchKernelGGL(k_hub_finalize<16>, dim3((unsigned)((max_chunk_hubs + 15) / 16) + 1), dim3(256), 0,
                                       stream, pl, (const uint8_t *)st.Lc, st.room, Ehub_rows, t.Ehub, t.Hhub,
                                       (uint8_t *)st.prop, st.cnt, (int)c, lo, (int)k, pass, store_e, ncells, cell_rows,
                                       st.tot);
            });
            // admission: the score kernel has counted the movers per tile and taken the sizes' snapshot, and
            // the tiles are few enough that every workgroup adds up the earlier tiles' counts itself
            L.run(GREM_KERNEL_APPLY, [&] {
                const dim3 grid((admit_blocks + kSmallApplyTiles - 1) / kSmallApplyTiles);
                auto go = [&](auto kernel, uint8_t *packed) {
                    hipLaunchKernelGGL(kernel, grid, dim3(kAdmitTile), 0, stream, (uint8_t *)st.Lc, (const uint8_t *)st.prop, lo, hi,
                                       (int)k, st.cnt, st.room, st.tot, (unsigned long long *)Snow, st.ocnt, pass, packed, ncells);
                };
                if (wide) cpt == 2 ? go(k_apply_small<32, 2>, nullptr) : go(k_apply_small<32, 1>, nullptr);
                else cpt == 2 ? go(k_apply_small<16, 2>, packed_now) : go(k_apply_small<16, 1>, packed_now);
            });
            }
            if (pass == 0) {
                if (spill_small) {
                    long long *Snext = Snow == st.S ? st.S2 : st.S;
                    L.run(GREM_KERNEL_SPILL_FILL, [&] {
                        const dim3 grid((admit_blocks + kSmallApplyTiles - 1) / kSmallApplyTiles);
                        if (wide)
                            hipLaunchKernelGGL(k_spill_small<32>, grid, dim3(kAdmitTile), 0, stream, (uint8_t *)st.Lc, lo, hi,
                                               (int)k, (const uint32_t *)st.ocnt, (int)admit_blocks, (const long long *)Snow,
                                               Snext);
                        else
                            hipLaunchKernelGGL(k_spill_small<16>, grid, dim3(kAdmitTile), 0, stream, (uint8_t *)st.Lc, lo, hi,
                                               (int)k, (const uint32_t *)st.ocnt, (int)admit_blocks, (const long long *)Snow,
                                               Snext);
                    });
                    Snow = Snext;
                } else {
                    launch_spill<uint8_t>(L, st, lo, hi, k, admit_blocks);
                }
            }
            // the chunk's new labels, looked up for every row that will read them: rows of later chunks in
            // this pass, rows of this and earlier chunks in the next pass (if there is one)
            lookup((int)c, 1, pass == R ? (int)c + 1 : 0, true, marks && pass == 0, packed_now);
        }
        L.mark();
    }
    st.S = Snow;
    launch_outputs<uint8_t>(L, st, n, k, labels_out, sizes_out);
    if (use16 && external_E) {
        int64_t blocks = (n + 255) / 256;
        if (blocks > 256 * 32) blocks = 256 * 32;
        L.run(GREM_KERNEL_EXPAND, [&] {
            hipLaunchKernelGGL((k_expand_estimates<RowT>), dim3((unsigned)blocks), dim3(256), 0, stream, rowptr, n, (int)k,
                               (uint32_t)hub_degree, t.E16, estimates_out);
        });
    }
    L.mark();
    return L.err;
}

// ---- plain route ------------------------------------------------------------------------------------
// The plain route takes the merged launches of grem_plain.hip.h for k <= 1024 and chunks of at most kPlainTiles
// tiles (every workgroup of the admission adds up the tiles' counts), the launches of grem_kernels.hip.h beyond them
// and where the histograms are forced into E's rows.
bool plain_merged(int32_t k, int64_t cl, int hist_mode) {
    return hist_mode != GREM_HIST_GLOBAL && k <= kPlainMaxK && (cl + kAdmitTile - 1) / kAdmitTile <= kPlainTiles;
}

int plain_long_degree(const Opts &o) { return o.long_row_degree ? o.long_row_degree : kLongDegree; }

// most long rows the merged launches keep a list of; with more the degree from which a row is long is doubled
size_t plain_long_rows(int64_t n) {
    const size_t most = (size_t)n / 256 + 1024;
    return most < (size_t)n ? most : (size_t)n;
}

struct PlainExtra {
    uint32_t *E = nullptr, *long_cnt = nullptr, *long_list = nullptr;
    // merged launches
    uint32_t *cnt = nullptr, *coarse = nullptr;          // two tables of mover counts each
    unsigned long long *rej = nullptr;
    uint32_t *nrows = nullptr, *nparts = nullptr, *off = nullptr, *cur = nullptr, *row = nullptr, *pref = nullptr, *ticket = nullptr;
    unsigned long long *bits = nullptr;                  // packed estimates: which cells are stored
};

// rows per workgroup of the tile kernels by the LDS that their histograms may take
int plain_tile_rows(int32_t k, int lds_bytes) {
    int tv = 256;
    while (tv > 1 && (size_t)tv * k * 4 > (size_t)lds_bytes) tv >>= 1;
    return tv;
}

// ... of the merged launches: the histograms in 16 KB of LDS, and small enough for 2048 workgroups
int merged_tile_rows(int32_t k, int64_t cl) {
    int tv = plain_tile_rows(k, kTileHistBytes);
    while (tv > 8 && (cl + tv - 1) / tv < kTileGrid) tv >>= 1;
    return tv;
}

bool pack_estimates(int64_t n, int32_t k, int64_t cl) {
    return k >= kPackMinK && (size_t)n * (size_t)k * 4 > (k >= kPackManyK ? kPackMinBytes : 2 * kPackMinBytes) &&
           merged_tile_rows(k, cl) * k >= kEstAhead * kScoreThreads;
}

// words of 64 cells that the packed estimates of a chunk's tiles make
size_t packed_words(int32_t k, int64_t cl) {
    const int tv = merged_tile_rows(k, cl);
    return (size_t)((cl + tv - 1) / tv) * (((size_t)tv * k + 63) / 64);
}

void state_plain(Carver &c, PlainExtra &x, int64_t n, int64_t cl, int32_t k, int64_t nchunks, bool external_E, bool merged, bool packed = false) {
    c.take(x.E, external_E ? 0 : (size_t)n * (size_t)k);
    if (!merged) {
        c.take(x.long_cnt, (size_t)nchunks);
        c.take(x.long_list, (size_t)cl);
        return;
    }
    const size_t tiles = (size_t)((cl + kAdmitTile - 1) / kAdmitTile), rows = plain_long_rows(n);
    c.take(x.cnt, 2 * tiles * (size_t)k);
    c.take(x.coarse, tiles * (size_t)k > (size_t)kPlainCells ? 2 * ((tiles + kPlainCoarse - 1) / kPlainCoarse) * (size_t)k : 0);
    c.take(x.rej, tiles * (kAdmitTile / 64));
    c.take(x.nrows, (size_t)nchunks);
    c.take(x.nparts, (size_t)nchunks);
    c.take(x.off, (size_t)nchunks);
    c.take(x.cur, (size_t)nchunks);
    c.take(x.row, rows);
    c.take(x.pref, rows);
    c.take(x.ticket, rows);
    c.take(x.bits, packed ? (size_t)nchunks * packed_words(k, cl) : 0);
}

// Alg. 1's loop in the merged launches.  degrees[i]: rows of at least long_row_degree * 2^i entries and fewer than
// twice as many (the last: and more).  long_counts: the prepass's counts by chunk (LongCounts), or null.
template <typename RowT, typename LabelT>
int run_plain_merged(const RowT *rowptr, const int32_t *colidx, int64_t n, int32_t k, double slack, int64_t cl, int32_t R,
                     const int32_t *seed, int32_t *labels_out, int64_t *sizes_out, uint32_t *estimates_out, const Opts &o,
                     unsigned long long maxdeg, const unsigned long long *degrees, const uint32_t *long_counts, Arena &mem, Launcher &L,
                     CallState<LabelT> &st) {
    hipStream_t stream = L.stream;
    const long long P = grem_capacity(n, k, slack);
    const bool external_E = estimates_out != nullptr;
    const int64_t nchunks = (n + cl - 1) / cl;
    PlainExtra x;
    const bool pack = pack_estimates(n, k, cl) && !external_E && R > 0;
    if (!(pack && carve(mem, [&](Carver &c) { state_plain(c, x, n, cl, k, nchunks, external_E, true, true); })) &&
        !carve(mem, [&](Carver &c) { state_plain(c, x, n, cl, k, nchunks, external_E, true); }))
        return GREM_ERR_NOMEM;
    uint32_t *E = external_E ? estimates_out : x.E;
    if (maxdeg * (unsigned long long)plain_tile_rows(k, kLdsHistBytes) >= (1ull << 31)) return GREM_ERR_RANGE;
    const int tv = merged_tile_rows(k, cl);
    const size_t tile_lds = ((size_t)tv * k + tv + 1 + 2 * (size_t)k) * 4;
    const int tiles_full = (int)((cl + kAdmitTile - 1) / kAdmitTile);
    const size_t cells = (size_t)tiles_full * (size_t)k;
    const size_t coarse_cells = x.coarse ? (size_t)((tiles_full + kPlainCoarse - 1) / kPlainCoarse) * (size_t)k : 0;
    const size_t admit_lds = admit_tiles_lds(k), spill_lds = spill_tiles_lds(k);
    // (at most 64 KB, which every kernel may have: k <= kPlainMaxK)

    // the long rows, chunk by chunk
    std::unique_ptr<uint32_t[]> read;              // (nothing throws: allocated without)
    const uint32_t *nrows = nullptr, *nparts = nullptr, *nrows_dev = x.nrows;
    bool counted = false;                          // by the prepass: nparts are then those beyond each row's first
    unsigned long long degree = (unsigned long long)plain_long_degree(o), rows = 0;
    for (int i = 0; i < kLongClasses; ++i) rows += degrees[i];
    for (int i = 0; i < kLongClasses - 1 && rows > plain_long_rows(n); ++i) { rows -= degrees[i]; degree *= 2; }
    const bool split_long = rows != 0 && rows <= plain_long_rows(n) && degree < (1ull << 32);
    uint32_t part = kLongPart;
    while (part < kLongPartMax && maxdeg / part > 64) part *= 2;
    if (split_long) {
        const unsigned blocks = (unsigned)((n + 255) / 256 < 8192 ? (n + 255) / 256 : 8192);
        L.memset(x.cur, 0, (size_t)nchunks * 4);
        counted = long_counts && degree == (unsigned long long)plain_long_degree(o);
        if (counted) {
            int size = 0;
            while ((kLongPart << size) < part) ++size;
            nrows = long_counts;
            nparts = long_counts + (size_t)(size + 1) * (size_t)nchunks;
            nrows_dev = (uint32_t *)(st.misc + 32);
        } else {
            read.reset(new (std::nothrow) uint32_t[2 * (size_t)nchunks]);
            if (!read) return GREM_ERR_NOMEM;
            nrows = read.get();
            nparts = read.get() + nchunks;
            L.memset(x.nrows, 0, (size_t)nchunks * 4);
            L.memset(x.nparts, 0, (size_t)nchunks * 4);
            L.run(GREM_KERNEL_HUBS, [&] {
                hipLaunchKernelGGL((k_long_count<RowT>), dim3(blocks), dim3(256), 0, stream, rowptr, n, cl, (uint32_t)degree,
                                   part, x.nrows, x.nparts);
            });
        }
        L.run(GREM_KERNEL_HUBS, [&] {
            hipLaunchKernelGGL(k_long_offsets, dim3(1), dim3(kScanThreads), 0, stream, nrows_dev, nchunks, x.off);
        });
        L.run(GREM_KERNEL_HUBS, [&] {
            hipLaunchKernelGGL((k_long_list<RowT>), dim3(blocks), dim3(256), 0, stream, rowptr, n, cl, (uint32_t)degree,
                               (const uint32_t *)x.off, x.cur, x.row, x.ticket);
        });
        L.run(GREM_KERNEL_HUBS, [&] {
            hipLaunchKernelGGL((k_long_parts<RowT>), dim3((unsigned)(nchunks < 1024 ? nchunks : 1024)), dim3(256), 0, stream, rowptr,
                               nchunks, part, nrows_dev, (const uint32_t *)x.off, (const uint32_t *)x.row, x.pref);
        });
        L.run(GREM_KERNEL_HUBS, [&] {
            hipLaunchKernelGGL(k_long_clear, dim3((unsigned)(rows < 2048 ? rows : 2048)), dim3(256), 0, stream, (const uint32_t *)x.row,
                               (uint32_t)rows, E, (int)k);
        });
        if (L.err) return L.err;
        if (!counted) {
            if (hipMemcpyAsync(read.get(), x.nrows, (size_t)nchunks * 4, hipMemcpyDeviceToHost, stream) != hipSuccess) return GREM_ERR_HIP;
            if (!L.read_back(read.get() + nchunks, x.nparts, (size_t)nchunks * 4)) {
                (void)hipStreamSynchronize(stream);            // (the copy before it writes to memory that is about to go)
                return L.err;
            }
        }
    }
    L.memset(x.cnt, 0, 2 * cells * 4);
    L.memset(x.coarse, 0, 2 * coarse_cells * 4);

    L.mark();
    long long *now = st.S, *other = st.S2;
    uint32_t *cnt = x.cnt, *cnt_other = x.cnt + cells, *coarse = x.coarse, *coarse_other = x.coarse ? x.coarse + coarse_cells : nullptr;
    for (int pass = 0; pass <= R && !L.err; ++pass) {
        const int standing = pass > 0 ? kAllLabelled : seed ? kSomeLabelled : kNoneLabelled;
        const int store_e = (pass < R || external_E) ? 1 : 0;
        size_t first = 0;                          // the chunk's first long row
        for (int64_t c = 0; c < nchunks && !L.err; first += split_long ? nrows[c] : 0, ++c) {
            const int64_t lo = c * cl;
            const int64_t hi = (lo + cl < n) ? lo + cl : n;
            const int64_t len = hi - lo;
            const unsigned tiles = (unsigned)((len + kAdmitTile - 1) / kAdmitTile);
            LongParts lr{nullptr, nullptr, nullptr, 0u, 0u, (uint32_t)degree, part};
            if (split_long && nrows[c] != 0) {
                const uint32_t parts = nparts[c] + (counted ? nrows[c] : 0u);
                lr = LongParts{x.row + first, x.pref + first, parts <= kLongTicketParts ? x.ticket + first : (uint32_t *)nullptr,
                               nrows[c], parts, (uint32_t)degree, part};
            }
            auto score = [&](auto kernel, unsigned long long *bits) {
                hipLaunchKernelGGL(kernel, dim3(lr.parts + (unsigned)((len + tv - 1) / tv)), dim3(kScoreThreads), tile_lds, stream, rowptr,
                                   colidx, (const LabelT *)st.Lc, (const long long *)now, other, E, st.prop, cnt, coarse, lo, hi, (int)k,
                                   tv, pass, P, standing == kNoneLabelled ? lo : n, standing, store_e, lr, bits);
            };
            L.run(GREM_KERNEL_SCORE, [&] {
                if (x.bits) score(k_score_tile<RowT, LabelT, true>, x.bits + (size_t)c * packed_words(k, cl));
                else score(k_score_tile<RowT, LabelT, false>, nullptr);
            });
            if (lr.rows != 0 && !lr.ticket)
                L.run(GREM_KERNEL_HUBS, [&] {
                    constexpr unsigned waves = kScoreThreads / 64;
                    hipLaunchKernelGGL((k_long_pick<LabelT>), dim3((lr.rows + waves - 1) / waves), dim3(kScoreThreads), (size_t)k * 4, stream,
                                       lr.row, lr.rows, (const uint32_t *)E, (const LabelT *)st.Lc, (const long long *)now, st.prop, cnt,
                                       coarse, lo, (int)k, pass, P, standing);
                });
            L.run(GREM_KERNEL_APPLY, [&] {
                hipLaunchKernelGGL((k_admit_tiles<LabelT>), dim3(tiles), dim3(kAdmitTile), admit_lds, stream, st.Lc,
                                   (const LabelT *)st.prop, lo, hi, (int)k, P, (const uint32_t *)cnt, (const uint32_t *)coarse, cnt_other,
                                   coarse_other, tiles_full, (const long long *)now, (unsigned long long *)other, x.rej, st.ocnt, standing);
            });
            if (pass == 0)
                L.run(GREM_KERNEL_SPILL_FILL, [&] {
                    hipLaunchKernelGGL((k_spill_tiles<LabelT>), dim3(tiles), dim3(kAdmitTile), spill_lds, stream, st.Lc, lo, (int)k,
                                       (const unsigned long long *)x.rej, (const uint32_t *)st.ocnt, (const long long *)other, now);
                });
            else std::swap(now, other);
            std::swap(cnt, cnt_other);
            std::swap(coarse, coarse_other);
        }
        L.mark();
    }
    st.S = now;
    launch_outputs<LabelT>(L, st, n, k, labels_out, sizes_out);
    L.mark();
    return L.err;
}

// A run that one workgroup does (grem_one.hip.h); nnz: entries of the graph.
bool one_takes(int64_t n, int32_t k, int64_t cl, unsigned long long maxdeg, unsigned long long nnz, const Opts &o) {
    const int64_t nchunks = (n + cl - 1) / cl;
    return o.hist_mode == GREM_HIST_AUTO && o.long_row_degree == 0 && k <= kOneMaxK && n <= kOneMaxN && cl <= kOneMaxChunk &&
           nchunks <= kOneMaxChunks && maxdeg < 65536 && nnz < (1ull << 31) && nnz / (unsigned long long)nchunks + (unsigned long long)(cl * k + cl * k / 2) <= kOneWork &&
           one_lds_bytes(n, cl, k) <= kOneLds;
}

// (false: no memory for it, nothing enqueued)
template <typename RowT>
bool run_one(const RowT *rowptr, const int32_t *colidx, int64_t n, int32_t k, double slack, int64_t cl, int32_t R, int32_t *labels_out,
             int64_t *sizes_out, uint32_t *estimates_out, unsigned long long nnz, unsigned long long maxdeg, Arena &mem, Launcher &L, CallState<uint8_t> &st) {
    uint32_t *E = nullptr, *rec = nullptr;
    const bool external_E = estimates_out != nullptr;
    if (!carve(mem, [&](Carver &c) { c.take(E, external_E || R == 0 ? 0 : (size_t)n * (size_t)k); c.take(rec, (size_t)nnz + 16); })) return false;
    const auto kernel = k <= 2 ? k_one_run<RowT, 2> : k <= 4 ? k_one_run<RowT, 4> : k_one_run<RowT, 8>;
    if (!set_lds((const void *)kernel, one_lds_bytes(n, cl, k), kOneLds)) { L.err = GREM_ERR_HIP; return true; }
    if (external_E) E = estimates_out;
    L.mark();
    if (nnz)
        L.run(GREM_KERNEL_RELAYOUT, [&] {
            hipLaunchKernelGGL((k_one_entries<RowT>), dim3((unsigned)((n + 3) / 4 < 2048 ? (n + 3) / 4 : 2048), (unsigned)((maxdeg + kOnePart - 1) / kOnePart)), dim3(256), 0, L.stream, rowptr, colidx,
                               n, cl, rec);
        });
    L.run(GREM_KERNEL_SCORE, [&] {
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kOneThreads), one_lds_bytes(n, cl, k), L.stream, rowptr, (const uint32_t *)rec, (int)n,
                           (int)k, (int)cl, (int)R, (int)std::min<int64_t>(grem_capacity(n, k, slack), 1 << 30), (const uint8_t *)st.Lc, (const long long *)st.S, E,
                           external_E ? 1 : 0, labels_out, sizes_out);
    });
    for (int i = 0; i <= R + 1; ++i) L.mark();       // (one launch: its passes have no bounds of their own)
    return true;
}

// Alg. 1's loop straight on the CSR.  `st` is prepared (prepass run, seed and degrees validated).
template <typename RowT, typename LabelT>
int run_plain(const RowT *rowptr, const int32_t *colidx, int64_t n, int32_t k, double slack, int64_t cl, int32_t R,
              const int32_t *seed, int32_t *labels_out, int64_t *sizes_out, uint32_t *estimates_out, const Opts &o,
              unsigned long long maxdeg, Arena &mem, Launcher &L, CallState<LabelT> &st) {
    hipStream_t stream = L.stream;
    const long long P = grem_capacity(n, k, slack);
    const bool external_E = estimates_out != nullptr;
    const int64_t nchunks = (n + cl - 1) / cl;
    const bool use_lds = o.hist_mode != GREM_HIST_GLOBAL && k <= kLdsMaxK;
    PlainExtra x;
    if (!carve(mem, [&](Carver &c) { state_plain(c, x, n, cl, k, nchunks, external_E, false); })) return GREM_ERR_NOMEM;
    uint32_t *E = external_E ? estimates_out : x.E;

    // tile shape of the score kernels
    int tv = kGlobalTile;
    if (use_lds) {
        tv = plain_tile_rows(k, kLdsHistBytes);
    }
    if (maxdeg * (unsigned long long)tv >= (1ull << 31)) return GREM_ERR_RANGE;
    const size_t score_lds = use_lds ? ((size_t)tv * k + tv + 1 + k) * 4 : ((size_t)tv + 1 + k) * 4;
    const size_t count_lds = (size_t)k * 4;
    const size_t apply_lds = apply_lds_bytes(k);
    if (!set_lds((const void *)k_apply<LabelT, false>, apply_lds, apply_lds_bytes(GREM_MAX_K))) return GREM_ERR_HIP;

    // rows this long are taken out of their tile and spread over a grid of their own
    const int long_degree = o.long_row_degree ? o.long_row_degree : kLongRowDegree;
    const bool split_long = maxdeg >= (unsigned long long)long_degree;
    const size_t long_lds = (size_t)k * 4;
    // (at most 16 KB)

    L.mark();
    for (int pass = 0; pass <= R && !L.err; ++pass) {
        if (split_long) L.memset(x.long_cnt, 0, (size_t)nchunks * 4);
        for (int64_t c = 0; c < nchunks && !L.err; ++c) {
            const int64_t lo = c * cl;
            const int64_t hi = (lo + cl < n) ? lo + cl : n;
            const int64_t len = hi - lo;
            const int64_t gather_limit = (pass == 0 && !seed) ? lo : n;
            const unsigned admit_blocks = (unsigned)((len + kAdmitTile - 1) / kAdmitTile);
            const LongRows lr{split_long ? (uint32_t)long_degree : 0xFFFFFFFFu, kLongRowPart, x.long_cnt + c,
                              x.long_list};
            const unsigned score_blocks = (unsigned)((len + tv - 1) / tv);
            L.run(GREM_KERNEL_SCORE, [&] {
                if (use_lds)
                    hipLaunchKernelGGL((k_score_lds<RowT, LabelT>), dim3(score_blocks), dim3(kScoreThreads), score_lds,
                                       stream, rowptr, colidx, st.Lc, st.S, E, st.prop, lo, hi, (int)k, tv, pass, P,
                                       gather_limit, lr);
                else
                    hipLaunchKernelGGL((k_score_global<RowT, LabelT>), dim3(score_blocks), dim3(kScoreThreads), score_lds,
                                       stream, rowptr, colidx, st.Lc, st.S, E, st.prop, lo, hi, (int)k, pass, P,
                                       gather_limit, lr);
            });
            if (split_long) {
                L.run(GREM_KERNEL_HUBS, [&] {
                    hipLaunchKernelGGL((k_long_rows<RowT, LabelT>), dim3(kLongRowGrid), dim3(kScoreThreads), long_lds, stream,
                                       rowptr, colidx, st.Lc, E, (int)k, pass, gather_limit, lr);
                });
                L.run(GREM_KERNEL_HUBS, [&] {
                    hipLaunchKernelGGL((k_long_propose<LabelT>), dim3(64), dim3(64), 0, stream, st.Lc, st.S, E, st.prop, lo,
                                       (int)k, pass, P, lr);
                });
            }
            // admission: per-tile mover counts, their prefix over the tiles, ranks
            L.run(GREM_KERNEL_COUNT, [&] {
                hipLaunchKernelGGL((k_count<LabelT>), dim3(admit_blocks), dim3(kAdmitThreads), count_lds, stream, st.Lc,
                                   st.prop, lo, hi, (int)k, st.cnt);
            });
            L.run(GREM_KERNEL_SCAN, [&] {
                hipLaunchKernelGGL(k_scan, dim3(1), dim3(kScanThreads), 0, stream, st.cnt, (int)admit_blocks, (int)k, st.S,
                                   P, st.room);
            });
            L.run(GREM_KERNEL_APPLY, [&] {
                hipLaunchKernelGGL((k_apply<LabelT, false>), dim3(admit_blocks), dim3(kAdmitThreads), apply_lds, stream,
                                   st.Lc, st.prop, lo, hi, (int)k, st.cnt, st.room, (unsigned long long *)st.S, st.ocnt,
                                   pass);
            });
            if (pass == 0) launch_spill<LabelT>(L, st, lo, hi, k, admit_blocks);
        }
        L.mark();
    }
    launch_outputs<LabelT>(L, st, n, k, labels_out, sizes_out);
    L.mark();
    return L.err;
}

// packed: with the bits of packed estimates, without which a run keeps them whole
size_t plain_bytes(int64_t n, int32_t k, int64_t cl, bool external_E, bool packed = true) {
    const int64_t nchunks = (n + cl - 1) / cl;
    PlainExtra x;
    size_t a;
    if (k <= 255) {
        CallState<uint8_t> st;
        a = carve_size([&](Carver &c) { state_common(c, st, n, cl, k); });
    } else {
        CallState<uint16_t> st;
        a = carve_size([&](Carver &c) { state_common(c, st, n, cl, k); });
    }
    // (whichever of the two forms takes more)
    const size_t one = carve_size([&](Carver &c) { state_plain(c, x, n, cl, k, nchunks, external_E, false); });
    const size_t two = plain_merged(k, cl, GREM_HIST_AUTO)
                           ? carve_size([&](Carver &c) { state_plain(c, x, n, cl, k, nchunks, external_E, true, packed && pack_estimates(n, k, cl)); }) : 0;
    return a + (one > two ? one : two);
}

// One partition call: route choice, memory, validation, then one of the two loops.
template <typename RowT, typename LabelT>
int run_partition(const RowT *rowptr, const int32_t *colidx, int64_t n, int32_t k, double slack, int64_t chunk,
                  int32_t R, const int32_t *seed, int32_t *labels_out, int64_t *sizes_out, uint32_t *estimates_out,
                  const Opts &o, hipStream_t stream) {
    const int64_t cl = chunk < n ? chunk : n;             // a chunk longer than the graph is the whole graph
    const long long P = grem_capacity(n, k, slack);
    const bool external_E = estimates_out != nullptr;
    if (o.hist_mode == GREM_HIST_LDS && k > kLdsMaxK) return GREM_ERR_ARG;
    const bool forced = o.hist_mode == GREM_HIST_SWEEP;
    bool try_sweep = false;
    if constexpr (sizeof(LabelT) == 1) {
        const TpGeom geo = tp_geometry(n, cl, o.col_bits, k);
        const bool can = k <= kSweepMaxK && geo.ok && (((uintptr_t)estimates_out) & 15u) == 0;
        if (forced && !can) return GREM_ERR_ARG;
        try_sweep = can && (forced || (o.hist_mode == GREM_HIST_AUTO && n >= kSweepMinN && cl >= kSweepMinChunk));
    } else {
        if (forced) return GREM_ERR_ARG;
    }

    Arena mem;
    mem.stream = stream;
    Launcher L{stream};
    {
        std::lock_guard<std::mutex> lock(g.mu);
        mem.base = (char *)g.ws;
        mem.cap = g.ws_bytes;
        L.level = g.prof_level;
    }
    if (mem.base && mem.cap < plain_bytes(n, k, cl, external_E, false)) return GREM_ERR_NOMEM;
    L.mark();

    CallState<LabelT> st;
    if (!carve(mem, [&](Carver &c) { state_common(c, st, n, cl, k); })) { mem.release_all(); return GREM_ERR_NOMEM; }
    unsigned long long maxdeg = 0;
    int rc = GREM_OK;
    bool done = false;
    if constexpr (sizeof(LabelT) == 1) {
        if (try_sweep) {
            // the plan's first kernels also find the largest degree, so the prepass leaves the rows alone
            launch_prepass<RowT, LabelT>(L, (const RowT *)nullptr, seed, n, k, P, st);
            const Arena::Mark before_plan = mem.mark();
            PlanData plan;
            rc = build_plan<RowT>(plan, rowptr, colidx, n, cl, k, o, mem, mem, L, forced);
            if (rc == GREM_ERR_NOMEM && !forced) {       // (a workspace that holds the plain route's state only)
                rc = GREM_OK;
                plan.T = nullptr;
            }
            if (rc != GREM_OK) { mem.release_all(); return rc; }
            if (plan.have_degrees) {
                maxdeg = plan.maxdeg;
                if (seed) {
                    unsigned long long h[16] = {0};
                    if (!L.read_back(h, st.misc, sizeof(h))) { mem.release_all(); return L.err; }
                    if (h[1] != 0 || h[2] != 0) { mem.release_all(); return GREM_ERR_SEED; }
                    st.seed_complete = h[5] == 0;
                }
                if (R >= 32 || (maxdeg << R) >= (1ull << 32)) { mem.release_all(); return GREM_ERR_RANGE; }
            } else {
                try_sweep = false;                       // the plain route's own prepass finds the degrees
            }
            if (plan.T) {
                rc = run_two_phase<RowT>(plan, k, slack, R, seed, labels_out, sizes_out, estimates_out, mem, L, &st);
                if (rc == GREM_ERR_NOMEM && !forced) rc = GREM_OK;      // nothing of the loop is enqueued yet
                else done = true;
            }
            if (!done) mem.release_to(before_plan);
        }
    }
    if (!done) {
        const bool merged = plain_merged(k, cl, o.hist_mode);
        unsigned long long degrees[kLongClasses] = {0};
        std::unique_ptr<unsigned long long[]> back;
        const uint32_t *long_counts = nullptr;
        if (!try_sweep || merged) {        // (the merged launches want the rows' degrees by class)
            // (a row of fewer entries is no rare one: their counts by chunk are then left for when they are known to be few)
            const bool counts = merged && (uint32_t)plain_long_degree(o) >= (uint32_t)kLongDegree && long_count_words(n, cl) != 0;
            const size_t words = 32 + (counts ? long_count_words(n, cl) : 0);
            back.reset(new (std::nothrow) unsigned long long[words]);
            if (!back) { mem.release_all(); return GREM_ERR_NOMEM; }
            launch_prepass<RowT, LabelT>(L, rowptr, seed, n, k, P, st, (uint32_t)plain_long_degree(o),
                                         counts ? LongCounts{nullptr, cl, (n + cl - 1) / cl, kLongPart} : LongCounts{});
            const unsigned long long *h = back.get();
            if (!L.read_back(back.get(), st.misc, words * 8)) { mem.release_all(); return L.err; }
            if (h[1] != 0 || h[2] != 0) { mem.release_all(); return GREM_ERR_SEED; }
            maxdeg = h[0];
            if (R >= 32 || (maxdeg << R) >= (1ull << 32)) { mem.release_all(); return GREM_ERR_RANGE; }
            for (int i = 0; i < kLongClasses; ++i) degrees[i] = h[16 + i];
            if (counts) long_counts = (const uint32_t *)(h + 32);
            if constexpr (sizeof(LabelT) == 1)
                if (one_takes(n, k, cl, maxdeg, h[3], o) &&
                    run_one<RowT>(rowptr, colidx, n, k, slack, cl, R, labels_out, sizes_out, estimates_out, h[3], maxdeg, mem, L, st)) {
                    mem.release_all();
                    return L.err;
                }
        }
        rc = merged ? run_plain_merged<RowT, LabelT>(rowptr, colidx, n, k, slack, cl, R, seed, labels_out, sizes_out, estimates_out, o,
                                                     maxdeg, degrees, long_counts, mem, L, st)
                    : run_plain<RowT, LabelT>(rowptr, colidx, n, k, slack, cl, R, seed, labels_out, sizes_out, estimates_out, o,
                                     maxdeg, mem, L, st);
    }
    mem.release_all();
    return rc;
}

template <typename RowT>
int dispatch_labels(const RowT *rowptr, const int32_t *colidx, int64_t n, int32_t k, double slack,
                    int64_t chunk, int32_t R, const int32_t *seed, int32_t *labels_out,
                    int64_t *sizes_out, uint32_t *estimates_out, const grem_options *options, void *stream) {
    if (!args_ok(rowptr, colidx, n, k, slack, chunk, R) || !labels_out) return GREM_ERR_ARG;
    Opts o;
    if (!resolve_options(options, &o)) return GREM_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    // a byte per label: 255 marks a vertex without one, which a run that starts without a seed and takes the merged
    // launches of the plain route never looks at
    const int64_t cl = chunk < n ? chunk : n;
    if (k <= 255 || (k == 256 && !seed && plain_merged(k, cl, o.hist_mode)))
        return run_partition<RowT, uint8_t>(rowptr, colidx, n, k, slack, chunk, R, seed, labels_out,
                                            sizes_out, estimates_out, o, s);
    return run_partition<RowT, uint16_t>(rowptr, colidx, n, k, slack, chunk, R, seed, labels_out,
                                         sizes_out, estimates_out, o, s);
}

template <typename RowT>
int run_edge_cut(const RowT *rowptr, const int32_t *colidx, int64_t n, const int32_t *labels,
                 int64_t *out, void *stream) {
    if (!rowptr || !colidx || !labels || !out || n < 1 || n > (int64_t)INT32_MAX) return GREM_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    const int64_t tiles = (n + kCutTile - 1) / kCutTile;
    // (fixed tiles: one per workgroup, at most 2^20 / 256 of them, unless the call is captured or has no memory)
    auto walk = [&](const uint32_t *words, LabelSpan *span) {
        const int64_t most = words ? (int64_t)kCutGrid : 2 * (int64_t)kCutGrid;
        const dim3 grid((unsigned)(tiles < most ? tiles : most));
        hipLaunchKernelGGL((k_edge_cut<RowT>), grid, dim3(kCutTile), 0, s, rowptr, colidx, n, labels, words, span,
                           (unsigned long long *)out);
        return hipGetLastError() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
    };
    // the packed table: from where the labels as they are outgrow the L2, unless the stream is being captured
    // or there is no memory for it (then the walk reads the labels themselves)
    char *block = nullptr;
    if (n >= kCutPackMinN) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusActive;
        if (hipStreamIsCapturing(s, &cap) != hipSuccess) (void)hipGetLastError();
        else if (cap == hipStreamCaptureStatusNone &&
                 hipMallocAsync((void **)&block, align_up(sizeof(LabelSpan)) + align_up((size_t)n), s) != hipSuccess) {
            (void)hipGetLastError();
            block = nullptr;
        }
    }
    if (!block) {
        hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, s, (unsigned long long *)out, 1);
        return walk(nullptr, nullptr);
    }
    LabelSpan *span = (LabelSpan *)block;
    uint32_t *words = (uint32_t *)(block + align_up(sizeof(LabelSpan)));
    hipLaunchKernelGGL(k_label_range_init, dim3(1), dim3(64), 0, s, span, (unsigned long long *)out);
    hipLaunchKernelGGL(k_label_range, dim3(2048), dim3(256), 0, s, labels, n, span);
    hipLaunchKernelGGL(k_pack_labels, dim3(2048), dim3(256), 0, s, labels, n, (const LabelSpan *)span, words);
    int rc = walk(words, span);
    if (hipFreeAsync(block, s) != hipSuccess) rc = GREM_ERR_HIP;
    return rc;
}

}  // namespace

// A plan: the re-laid-out copy and the memory it lives in.
struct grem_plan {
    PlanData data;
    Arena mem;          // persistent allocations
};

extern "C" {

int64_t grem_capacity(int64_t n, int32_t k, double balance_slack) {
    if (n < 1 || k < 1 || !(balance_slack >= 1.0)) return -1;
    const int64_t even = (n + k - 1) / k;
    const double scaled = (double)n * balance_slack;
    const double per = scaled / (double)k;
    const int64_t widened = (int64_t)std::ceil(per);
    return even > widened ? even : widened;
}

size_t grem_workspace_bytes(int64_t n, int32_t k, int64_t chunk) {
    if (n < 1 || n > (int64_t)INT32_MAX || k < 1 || k > GREM_MAX_K || chunk < 1) return 0;
    return plain_bytes(n, k, chunk < n ? chunk : n, false);
}

size_t grem_workspace_bytes_two_phase(int64_t n, int64_t nnz, int32_t k, int64_t chunk, const grem_options *options) {
    if (n < 1 || n > (int64_t)INT32_MAX || nnz < 0 || k < 1 || k > GREM_MAX_K || chunk < 1) return 0;
    Opts o;
    if (!resolve_options(options, &o)) return 0;
    const int64_t cl = chunk < n ? chunk : n;
    const size_t plain = plain_bytes(n, k, cl, false);
    const TpGeom geo = tp_geometry(n, cl, o.col_bits, k);
    if (k > kSweepMaxK || !geo.ok) return plain;
    PlanDims d{};
    d.n = n;
    d.nnz = nnz;
    d.geo = geo;
    d.G = (size_t)geo.nch * (size_t)geo.nsl;
    d.hubs = (size_t)(nnz / o.hub_degree);                   // a hub has at least hub_degree entries
    if (d.hubs > (size_t)n) d.hubs = (size_t)n;
    d.npr = kMaxParts;
    d.nps = kMaxParts;
    {   // a chunk has at most one hub share per 64 * nblk hub entries (and at least one per 1024 hubs), never
        // more than slices
        size_t shares = (size_t)nnz / (64 * (size_t)geo.nblk) + d.hubs / 1024 + 1;
        if (shares > (size_t)geo.nsl) shares = (size_t)geo.nsl;
        d.nr = geo.nsl + (int)shares;
    }
    d.slots = plan_slots(nnz, geo, d.nr);
    SweepPlan pl{};
    TpTables tb{};
    u64 *pm = nullptr;
    uint32_t *T = nullptr;
    uint16_t *R = nullptr;
    CallState<uint8_t> st;
    TpState t;
    size_t total = carve_size([&](Carver &c) { state_common(c, st, n, cl, k); });
    total += carve_size([&](Carver &c) { plan_stage1(c, d, pl, pm); });
    total += carve_size([&](Carver &c) { plan_stage2(c, d, pl); });
    total += carve_size([&](Carver &c) { plan_stage3(c, d, tb, T, R); });
    // the intermediate copy and the per-call state take turns in one region; the state is largest for a
    // seeded run whose estimates need 32 bits
    const size_t temp = align_up((size_t)nnz * 4 + 16) + align_up((size_t)geo.nch * (size_t)d.nr * (size_t)geo.nblk * 4);
    const size_t chunk_hubs = d.hubs < (size_t)cl ? d.hubs : (size_t)cl;
    const size_t s16 = carve_size([&](Carver &c) { state_two_phase(c, t, n, k, d.slots, chunk_hubs, d.hubs, true, true, false, true); });
    const size_t s32 = carve_size([&](Carver &c) { state_two_phase(c, t, n, k, d.slots, chunk_hubs, d.hubs, true, false, false, true); });
    size_t tail = temp;
    if (s16 > tail) tail = s16;
    if (s32 > tail) tail = s32;
    total += tail;
    return total > plain ? total : plain;
}

int grem_set_workspace(void *dev_ptr, size_t bytes) {
    std::lock_guard<std::mutex> lock(g.mu);
    if ((dev_ptr == nullptr) != (bytes == 0)) return GREM_ERR_ARG;
    if (((uintptr_t)dev_ptr & 255u) != 0) return GREM_ERR_ARG;
    g.ws = dev_ptr;
    g.ws_bytes = bytes;
    return GREM_OK;
}

int grem_partition(const int64_t *rowptr, const int32_t *colidx, int64_t n, int32_t k,
                   double balance_slack, int64_t chunk, int32_t refine_passes, int32_t *labels_out,
                   void *stream) {
    return dispatch_labels<int64_t>(rowptr, colidx, n, k, balance_slack, chunk, refine_passes, nullptr,
                                    labels_out, nullptr, nullptr, nullptr, stream);
}

int grem_partition_seeded(const int64_t *rowptr, const int32_t *colidx, int64_t n, int32_t k,
                          double balance_slack, int64_t chunk, int32_t refine_passes,
                          const int32_t *seed_labels, int32_t *labels_out, void *stream) {
    return dispatch_labels<int64_t>(rowptr, colidx, n, k, balance_slack, chunk, refine_passes,
                                    seed_labels, labels_out, nullptr, nullptr, nullptr, stream);
}

int grem_partition_r32(const int32_t *rowptr, const int32_t *colidx, int64_t n, int32_t k,
                       double balance_slack, int64_t chunk, int32_t refine_passes, int32_t *labels_out,
                       void *stream) {
    return dispatch_labels<int32_t>(rowptr, colidx, n, k, balance_slack, chunk, refine_passes, nullptr,
                                    labels_out, nullptr, nullptr, nullptr, stream);
}

int grem_partition_seeded_r32(const int32_t *rowptr, const int32_t *colidx, int64_t n, int32_t k,
                              double balance_slack, int64_t chunk, int32_t refine_passes,
                              const int32_t *seed_labels, int32_t *labels_out, void *stream) {
    return dispatch_labels<int32_t>(rowptr, colidx, n, k, balance_slack, chunk, refine_passes,
                                    seed_labels, labels_out, nullptr, nullptr, nullptr, stream);
}

int grem_partition_opt(const void *rowptr, int32_t rowptr_bits, const int32_t *colidx, int64_t n,
                       int32_t k, double balance_slack, int64_t chunk, int32_t refine_passes,
                       const int32_t *seed_labels, int32_t *labels_out, int64_t *sizes_out,
                       uint32_t *estimates_out, const grem_options *options, void *stream) {
    if (rowptr_bits == 64)
        return dispatch_labels<int64_t>((const int64_t *)rowptr, colidx, n, k, balance_slack, chunk,
                                        refine_passes, seed_labels, labels_out, sizes_out,
                                        estimates_out, options, stream);
    if (rowptr_bits == 32)
        return dispatch_labels<int32_t>((const int32_t *)rowptr, colidx, n, k, balance_slack, chunk,
                                        refine_passes, seed_labels, labels_out, sizes_out,
                                        estimates_out, options, stream);
    return GREM_ERR_ARG;
}

int grem_partition_state(const void *rowptr, int32_t rowptr_bits, const int32_t *colidx, int64_t n,
                         int32_t k, double balance_slack, int64_t chunk, int32_t refine_passes,
                         const int32_t *seed_labels, int32_t *labels_out, int64_t *sizes_out,
                         uint32_t *estimates_out, void *stream) {
    return grem_partition_opt(rowptr, rowptr_bits, colidx, n, k, balance_slack, chunk, refine_passes, seed_labels,
                              labels_out, sizes_out, estimates_out, nullptr, stream);
}

int grem_plan_create(const void *rowptr, int32_t rowptr_bits, const int32_t *colidx, int64_t n, int64_t chunk,
                     const grem_options *options, void *stream, grem_plan **plan_out) {
    if (!plan_out) return GREM_ERR_ARG;
    *plan_out = nullptr;
    if (!rowptr || !colidx || n < 1 || n > (int64_t)INT32_MAX || chunk < 1 || (rowptr_bits != 32 && rowptr_bits != 64))
        return GREM_ERR_ARG;
    Opts o;
    if (!resolve_options(options, &o)) return GREM_ERR_ARG;
    const int64_t cl = chunk < n ? chunk : n;
    if (!tp_geometry(n, cl, o.col_bits, o.plan_max_k).ok) return GREM_ERR_ARG;
    grem_plan *p = new (std::nothrow) grem_plan();
    if (!p) return GREM_ERR_NOMEM;
    hipStream_t s = (hipStream_t)stream;
    p->mem.persistent = true;
    Arena temp;
    temp.stream = s;
    Launcher L{s};
    {
        std::lock_guard<std::mutex> lock(g.mu);
        L.level = g.prof_level;
    }
    L.mark();
    int rc = rowptr_bits == 64
                 ? build_plan<int64_t>(p->data, (const int64_t *)rowptr, colidx, n, cl, 0, o, p->mem, temp, L, true)
                 : build_plan<int32_t>(p->data, (const int32_t *)rowptr, colidx, n, cl, 0, o, p->mem, temp, L, true);
    L.mark();
    temp.release_all();
    if (hipStreamSynchronize(s) != hipSuccess && rc == GREM_OK) rc = GREM_ERR_HIP;
    if (rc != GREM_OK) {
        p->mem.release_all();
        delete p;
        return rc;
    }
    *plan_out = p;
    return GREM_OK;
}

int grem_plan_destroy(grem_plan *plan) {
    if (!plan) return GREM_OK;
    const int rc = hipDeviceSynchronize() == hipSuccess ? GREM_OK : GREM_ERR_HIP;
    plan->mem.release_all();
    delete plan;
    return rc;
}

size_t grem_plan_device_bytes(const grem_plan *plan) { return plan ? plan->mem.total : 0; }

int32_t grem_plan_max_k(const grem_plan *plan) { return plan ? plan->data.max_k : 0; }

size_t grem_plan_call_bytes(const grem_plan *plan, int32_t k, int32_t refine_passes, int32_t seeded,
                            int32_t with_estimates_out) {
    if (!plan || !plan->data.T || k < 1 || k > plan->data.max_k || refine_passes < 0 || refine_passes >= 32) return 0;
    const PlanData &P = plan->data;
    const bool use16 = (((unsigned long long)(P.hub_degree - 1)) << refine_passes) <= 65535ull;
    CallState<uint8_t> st;
    TpState t;
    return carve_size([&](Carver &c) { state_common(c, st, P.n, (int64_t)P.geo.chunk, k); }) +
           carve_size([&](Carver &c) {
               state_two_phase(c, t, P.n, k, P.slots, (size_t)P.max_chunk_hubs, (size_t)P.total_hubs, seeded != 0, use16,
                               with_estimates_out != 0, admission_takes_hubs(P, use16, with_estimates_out != 0));
           });
}

int grem_partition_planned(const grem_plan *plan, int32_t k, double balance_slack, int32_t refine_passes,
                           const int32_t *seed_labels, int32_t *labels_out, int64_t *sizes_out,
                           uint32_t *estimates_out, void *stream) {
    if (!plan || !plan->data.T || !labels_out || k < 1 || k > plan->data.max_k || refine_passes < 0 ||
        !(balance_slack >= 1.0) || std::isinf(balance_slack))
        return GREM_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    Arena mem;
    mem.stream = s;
    Launcher L{s};
    {
        std::lock_guard<std::mutex> lock(g.mu);
        mem.base = (char *)g.ws;
        mem.cap = g.ws_bytes;
        L.level = g.prof_level;
    }
    L.mark();
    const int rc = plan->data.rowptr_bits == 64
                       ? run_two_phase<int64_t>(plan->data, k, balance_slack, refine_passes, seed_labels, labels_out,
                                                sizes_out, estimates_out, mem, L, nullptr)
                       : run_two_phase<int32_t>(plan->data, k, balance_slack, refine_passes, seed_labels, labels_out,
                                                sizes_out, estimates_out, mem, L, nullptr);
    mem.release_all();
    return rc;
}

int64_t grem_plan_n(const grem_plan *plan) { return plan ? plan->data.n : 0; }

namespace {

// cnt_nbrs of every vertex under a labelling that stays as it is, on a plan; `mem` supplies the
// run's state (the caller releases it)
int plan_counts(const grem_plan *plan, int32_t k, const int32_t *labels, uint32_t *counts_out, Arena &mem, Launcher &L) {
    // capacity n: whatever the labelling, no partition is over it
    return plan->data.rowptr_bits == 64
               ? run_two_phase<int64_t>(plan->data, k, (double)k, 0, labels, nullptr, nullptr, counts_out, mem, L, nullptr, true)
               : run_two_phase<int32_t>(plan->data, k, (double)k, 0, labels, nullptr, nullptr, counts_out, mem, L, nullptr, true);
}

void plan_call_setup(Arena &mem, Launcher &L, hipStream_t s) {
    mem.stream = s;
    std::lock_guard<std::mutex> lock(g.mu);
    mem.base = (char *)g.ws;
    mem.cap = g.ws_bytes;
    L.level = g.prof_level;
}

}  // namespace

int grem_plan_neighbour_counts(const grem_plan *plan, int32_t k, const int32_t *labels, uint32_t *counts_out,
                               void *stream) {
    if (!plan || !plan->data.T || !labels || !counts_out || k < 1 || k > plan->data.max_k) return GREM_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    Arena mem;
    Launcher L{s};
    plan_call_setup(mem, L, s);
    L.mark();
    const int rc = plan_counts(plan, k, labels, counts_out, mem, L);
    mem.release_all();
    return rc;
}

int grem_plan_edge_cut(const grem_plan *plan, int32_t k, const int32_t *labels, int64_t *cut_entries_out,
                       void *stream) {
    if (!plan || !plan->data.T || !labels || !cut_entries_out || k < 1 || k > plan->data.max_k) return GREM_ERR_ARG;
    hipStream_t s = (hipStream_t)stream;
    Arena mem;
    Launcher L{s};
    plan_call_setup(mem, L, s);
    L.mark();
    const int64_t n = plan->data.n;
    uint32_t *counts = nullptr;
    if (!carve(mem, [&](Carver &c) { c.take(counts, (size_t)n * (size_t)k); })) return GREM_ERR_NOMEM;
    int rc = plan_counts(plan, k, labels, counts, mem, L);
    if (rc == GREM_OK) {
        int64_t blocks = (n + 255) / 256;
        if (blocks > 256 * 32) blocks = 256 * 32;
        L.run(GREM_KERNEL_EXPAND, [&] {
            hipLaunchKernelGGL(k_zero_u64, dim3(1), dim3(64), 0, s, (unsigned long long *)cut_entries_out, 1);
        });
        L.run(GREM_KERNEL_EXPAND, [&] {
            if (plan->data.rowptr_bits == 64)
                hipLaunchKernelGGL(k_cut_from_counts<int64_t>, dim3((unsigned)blocks), dim3(256), 0, s,
                                   (const int64_t *)plan->data.rowptr, labels, (const uint32_t *)counts, n, (int)k,
                                   (unsigned long long *)cut_entries_out);
            else
                hipLaunchKernelGGL(k_cut_from_counts<int32_t>, dim3((unsigned)blocks), dim3(256), 0, s,
                                   (const int32_t *)plan->data.rowptr, labels, (const uint32_t *)counts, n, (int)k,
                                   (unsigned long long *)cut_entries_out);
        });
        rc = L.err;
    }
    mem.release_all();
    return rc;
}

int grem_edge_cut(const int64_t *rowptr, const int32_t *colidx, int64_t n, const int32_t *labels,
                  int64_t *cut_entries_out, void *stream) {
    return run_edge_cut<int64_t>(rowptr, colidx, n, labels, cut_entries_out, stream);
}

int grem_edge_cut_r32(const int32_t *rowptr, const int32_t *colidx, int64_t n, const int32_t *labels,
                      int64_t *cut_entries_out, void *stream) {
    return run_edge_cut<int32_t>(rowptr, colidx, n, labels, cut_entries_out, stream);
}

int grem_profile_enable(int32_t level) {
    if (level < 0 || level > 2) return GREM_ERR_ARG;
    std::lock_guard<std::mutex> lock(g.mu);
    g.prof_level = level;
    return GREM_OK;
}

int grem_profile_reset(void) {
    std::lock_guard<std::mutex> lock(g.mu);
    for (auto &e : g.events) { g.pool.push_back(e.a); g.pool.push_back(e.b); }
    for (auto &e : g.marks) g.pool.push_back(e);
    g.events.clear();
    g.marks.clear();
    return GREM_OK;
}

int grem_profile_read(int32_t kernel_class, double *total_ms, int64_t *launches) {
    if (kernel_class < 0 || kernel_class >= GREM_KERNEL_CLASSES || !total_ms || !launches)
        return GREM_ERR_ARG;
    std::lock_guard<std::mutex> lock(g.mu);
    double tot = 0.0;
    int64_t cnt = 0;
    for (auto &e : g.events) {
        if (e.cls != kernel_class) continue;
        if (hipEventSynchronize(e.b) != hipSuccess) return GREM_ERR_HIP;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, e.a, e.b) != hipSuccess) return GREM_ERR_HIP;
        tot += ms;
        cnt += 1;
    }
    *total_ms = tot;
    *launches = cnt;
    return GREM_OK;
}

int grem_profile_read_marks(double *ms_out, int32_t capacity) {
    if (!ms_out || capacity < 0) return GREM_ERR_ARG;
    std::lock_guard<std::mutex> lock(g.mu);
    int written = 0;
    for (size_t i = 1; i < g.marks.size() && written < capacity; ++i) {
        if (hipEventSynchronize(g.marks[i]) != hipSuccess) return GREM_ERR_HIP;
        float ms = 0.f;
        if (hipEventElapsedTime(&ms, g.marks[i - 1], g.marks[i]) != hipSuccess) return GREM_ERR_HIP;
        ms_out[written++] = ms;
    }
    return written;
}

const char *grem_status_string(int code) {
    switch (code) {
        case GREM_OK: return "ok";
        case GREM_ERR_ARG: return "bad argument";
        case GREM_ERR_NOMEM: return "workspace allocation failed or workspace too small";
        case GREM_ERR_HIP: return "HIP runtime error";
        case GREM_ERR_RANGE: return "max degree * 2^refine_passes does not fit the estimates";
        case GREM_ERR_SEED: return "invalid seed labels";
        case GREM_ERR_LIMIT: return "input larger than the entry point's fixed-size buffer allows";
        default: return "unknown status";
    }
}

const char *grem_kernel_name(int32_t kernel_class) {
    switch (kernel_class) {
        case GREM_KERNEL_PREPASS: return "prepass";
        case GREM_KERNEL_SCORE: return "score";
        case GREM_KERNEL_COUNT: return "count";
        case GREM_KERNEL_SCAN: return "scan";
        case GREM_KERNEL_APPLY: return "apply";
        case GREM_KERNEL_SPILL_SCAN: return "spill_scan";
        case GREM_KERNEL_SPILL_FILL: return "spill_fill";
        case GREM_KERNEL_EXPAND: return "expand";
        case GREM_KERNEL_RELAYOUT: return "relayout";
        case GREM_KERNEL_LOOKUP: return "lookup";
        case GREM_KERNEL_HUBS: return "hub_finalize";
        default: return "?";
    }
}

}  // extern "C"
