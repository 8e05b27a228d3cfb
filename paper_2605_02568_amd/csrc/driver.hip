// Host driver: argument checks, tile planning, workspace carve-up and the nested tile loop
// of Algorithm 2 (outer loop over query tiles, inner loop over key tiles, per-query running
// state, write-out after the last key tile).  Per key tile: one score kernel that appends the
// surviving candidates to the row buffers, one compaction kernel; per query tile: one init and
// one finalize kernel.  Key tiles that hold no legal key for any query of the query tile are
// not visited (Algorithm 2 visits them; their masked entries can never be selected, so the
// result is the same).

#include <algorithm>
#include <atomic>
#include <mutex>
#include <vector>

#include "si_internal.h"

// Scratch of si_indexer_topk_static, the entry point that allocates nothing: the workspace of the
// single-pass schedule for k <= kStaticMaxK (launch counters, then 256 x 8 row buffers of
// 2k + 384 keys), as one static array in device memory.  Each GPU the library runs on holds its
// own copy from the moment the code object is loaded until the process ends.  In host code the
// name `scratch` is only a handle: the address kernels can use comes from hipGetSymbolAddress,
// once per device (static_scratch below), and only that pointer is ever passed on.
namespace {
constexpr int kStaticMaxK = 1024;
constexpr int kStaticMaxLaunches = 64;  // counters: one 256-byte block
constexpr size_t kStaticScratchBytes =
    256 + static_cast<size_t>(si::kFusedSlots) * si::kQueriesPerBlock *
              (si::kFusedTriggerMul * kStaticMaxK + si::kFusedRowSlack) * sizeof(si::key64_t);
}  // namespace
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace si {

namespace {

thread_local int32_t g_last_hip_error = 0;

inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

si_status hip_fail(hipError_t e) {
    g_last_hip_error = static_cast<int32_t>(e);
    return SI_ERR_HIP;
}

// ---- per-kernel timing (benchmark aid) --------------------------------------------------
struct Profiler {
    std::mutex mu;  // every member below is read and written under it
    bool on = false;
    unsigned long long* phase = nullptr;  // device words of the single-pass kernel's phase clock
    int32_t phase_slots = 0;
    std::vector<hipEvent_t> pool;  // reused events
    size_t used = 0;
    struct Span { int cls; size_t begin, end; };
    std::vector<Span> spans;
    double ms[SI_PROFILE_CLASSES] = {0};
    int64_t launches[SI_PROFILE_CLASSES] = {0};

    hipError_t next_event(size_t* idx) {
        if (used == pool.size()) {
            hipEvent_t ev;
            hipError_t e = hipEventCreate(&ev);
            if (e != hipSuccess) return e;
            pool.push_back(ev);
        }
        *idx = used++;
        return hipSuccess;
    }
    // folds finished spans into the totals and frees the events for reuse
    hipError_t drain() {
        for (const Span& s : spans) {
            hipError_t e = hipEventSynchronize(pool[s.end]);
            if (e != hipSuccess) return e;
            float t = 0.f;
            e = hipEventElapsedTime(&t, pool[s.begin], pool[s.end]);
            if (e != hipSuccess) return e;
            ms[s.cls] += t;
            launches[s.cls] += 1;
        }
        spans.clear();
        used = 0;
        return hipSuccess;
    }
};
Profiler g_prof;

// Brackets one launch with events when profiling is on.
template <typename F>
hipError_t timed(int cls, hipStream_t stream, F&& launch) {
    std::lock_guard<std::mutex> hold(g_prof.mu);
    if (!g_prof.on) return launch();
    if (g_prof.spans.size() >= 8192) {  // bound the number of live events
        hipError_t e = g_prof.drain();
        if (e != hipSuccess) return e;
    }
    size_t b = 0, en = 0;
    hipError_t e = g_prof.next_event(&b);
    if (e != hipSuccess) return e;
    e = g_prof.next_event(&en);
    if (e != hipSuccess) return e;
    e = hipEventRecord(g_prof.pool[b], stream);
    if (e != hipSuccess) return e;
    e = launch();
    if (e != hipSuccess) return e;
    e = hipEventRecord(g_prof.pool[en], stream);
    if (e != hipSuccess) return e;
    g_prof.spans.push_back({cls, b, en});
    return hipSuccess;
}

si_status check_dims(const si_dims* d, int32_t m, int32_t k, int mask_mode) {
    if (!d) return SI_ERR_INVALID_ARG;
    if (d->B < 1 || d->S < 1 || d->H_I < 1 || d->D < 1 || d->T < 1) return SI_ERR_INVALID_ARG;
    if (m < 1 || k < 1) return SI_ERR_INVALID_ARG;
    if (mask_mode != SI_MASK_NONE && mask_mode != SI_MASK_CAUSAL_BLOCK) return SI_ERR_INVALID_ARG;
    if (d->D != 32 && d->D != 64 && d->D != 128) return SI_ERR_UNSUPPORTED_SHAPE;
    if (d->H_I > kMaxHeads || k > kMaxK) return SI_ERR_UNSUPPORTED_SHAPE;
    // the score sweep addresses one batch's keys through a 32-bit buffer range
    if (static_cast<int64_t>(d->T) * d->D * 2 >= (int64_t{1} << 32)) return SI_ERR_UNSUPPORTED_SHAPE;
    return SI_OK;
}

size_t workspace_bytes_for(int64_t B, int64_t c_S, int64_t c_T, int64_t k) {
    return carve_workspace(nullptr, B * c_S, k, std::max<int64_t>(c_T, 1)).bytes;
}

// Key tiles of one query tile: a narrow first tile, then widths that double up to c_T.  The
// first tile cannot be filtered (no k-th best exists yet), so it is kept small; each later
// tile is filtered against the top-k of everything before it.  The result does not depend on
// this schedule.
int64_t next_width(int64_t t0, int64_t c_T, int64_t k) {
    const int64_t first = std::max<int64_t>(2 * k, 1024);
    const int64_t w = t0 == 0 ? first : std::max<int64_t>(t0, first);
    return std::min<int64_t>(w, c_T);
}

// Workspace of the single-pass schedule: one launch counter per query tile, then the row
// buffers of the resident workgroups.
struct FusedLayout {
    int32_t* counters;
    int64_t n_launches;
    RowBuffers slots;
    size_t bytes;
};
int32_t fused_rows_per_launch(int32_t c_S, int32_t S) {
    if (c_S < 1) c_S = kFusedDefaultRows;
    return std::min(c_S, S);
}
FusedLayout carve_fused(void* base, int64_t S, int64_t k, int64_t c_S) {
    FusedLayout L;
    char* p = static_cast<char*>(base);
    L.n_launches = (S + c_S - 1) / c_S;
    size_t off = 0;
    L.counters = reinterpret_cast<int32_t*>(p + off);
    off = align_up(off + static_cast<size_t>(L.n_launches) * sizeof(int32_t), 256);
    L.slots.keys = reinterpret_cast<key64_t*>(p + off);
    L.slots.cap = static_cast<int32_t>(kFusedTriggerMul * k + kFusedRowSlack);
    off = align_up(off + static_cast<size_t>(kFusedSlots) * kQueriesPerBlock * L.slots.cap * sizeof(key64_t), 256);
    L.slots.count = nullptr;
    L.slots.theta = nullptr;
    L.slots.bytes = off;
    L.bytes = off;
    return L;
}

// Immutable facts about a device, looked up once per device and process.
struct DeviceInfo {
    std::atomic<int> compute_units{0};
    std::atomic<void*> static_scratch{nullptr};  // this device's copy of `scratch`
};
constexpr int kMaxDevices = 64;
DeviceInfo g_device[kMaxDevices];

// Workgroups the single-pass kernel is launched with: one wide (8-wave) or two narrow (4-wave)
// workgroups per compute unit of the current device -- either way 2 waves per SIMD, which is what
// their register budget allows -- and at most what the workspace has row buffers for.
hipError_t fused_workgroups(int32_t waves, int32_t* n) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    int cus = (dev >= 0 && dev < kMaxDevices) ? g_device[dev].compute_units.load(std::memory_order_acquire) : 0;
    if (cus == 0) {
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        if (cus < 1) return hipErrorInvalidDevice;
        if (dev >= 0 && dev < kMaxDevices) g_device[dev].compute_units.store(cus, std::memory_order_release);
    }
    const int32_t per_cu = kQueriesPerBlock / waves;
    *n = std::min<int32_t>(cus * per_cu, kFusedSlots * per_cu);
    return hipSuccess;
}

// Keys of the longest row: under the causal mask the cache may hold more keys than the last query sees.
int32_t longest_row(const si_dims& d, int32_t m, int32_t mask_mode) {
    return mask_mode == SI_MASK_CAUSAL_BLOCK ? std::min(d.T, d.S / m) : d.T;
}

// Workgroup shape of the single-pass schedule when the caller does not choose (see SweepShape in
// score_sweep.h).  Per work item the merges, the final cut + sort and the write-out cost a time
// that depends on k but not on the item's key range, with the matrix pipe idle; two narrow
// workgroups per compute unit overlap one's such phases with the other's sweep, at the price of
// staging every key chunk for 4 queries instead of 8 and of a lone sweeping wave per SIMD that
// cannot hide its own stalls.  Measured on MI355X (time of the narrow shape over that of the wide one): prompts, S = 4 T, causal,
// k = 512, 4096 / 8192 / 16384 / 24576 / 32768 keys per query: 64 heads of 128 0.87 / 0.96 / 1.00 / 1.01 / 1.02, 32 of 128 0.95 /
// 1.02 / 0.99 / 1.03 / 1.02, 33 of 64 0.95 / 0.99 / 0.99 / 0.99 / 1.00, 4 of 32 0.95 / 0.95 / 0.97 / 0.99 / 1.00.  Without a mask all
// items are equally long and the two workgroups of a unit stay in step: 8192 queries of 4096 / 8192 / 16384 / 32768 keys, the same
// heads: 1.00 / 1.03 / 1.09 / 1.04, 0.97 / 1.04 / 1.05 / 1.07, 0.99 / 1.03 / 1.06 / 1.12, 1.03 / 1.02 / 1.03 / 1.07.
constexpr int64_t kNarrowMaxKeys = 16384;
constexpr int64_t kNarrowMaxKeysInStep = 4096;
// Rounds of equal items the chip works through, a round of wide workgroups being 1: a round of two narrow ones per unit takes
// 1.06, one with at most one per unit 0.65 (3000 queries of 9000 keys, 20 x 100 of 9000: wide 471 and 421 us, narrow 410 and 374).
double wide_rounds(const si_dims& d) {
    const int64_t wide = (static_cast<int64_t>(d.S) + 7) / 8 * d.B;
    return static_cast<double>((wide + kFusedSlots - 1) / kFusedSlots);
}
double narrow_rounds(const si_dims& d) {
    const int64_t narrow = (static_cast<int64_t>(d.S) + 3) / 4 * d.B;
    const int64_t rest = narrow % (2 * kFusedSlots);
    const double last = rest == 0 ? 0.0 : rest <= kFusedSlots ? 0.65 : 1.06;
    return 1.06 * static_cast<double>(narrow / (2 * kFusedSlots)) + last;
}
int32_t fused_shape_for(const si_dims& d, int32_t m, int32_t mask_mode) {
    const int32_t longest = longest_row(d, m, mask_mode);
    if (mask_mode == SI_MASK_NONE && longest > kNarrowMaxKeysInStep && longest <= kNarrowMaxKeys) return wide_rounds(d) < narrow_rounds(d) ? 8 : 4;
    return longest <= kNarrowMaxKeys ? 4 : 8;
}

// Device address of the current device's copy of `scratch`: asked from the runtime on the first
// call on that device (with that device current), remembered afterwards.
hipError_t static_scratch(void** ptr) {
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool tracked = dev >= 0 && dev < kMaxDevices;
    void* p = tracked ? g_device[dev].static_scratch.load(std::memory_order_acquire) : nullptr;
    if (p == nullptr) {
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (p == nullptr) return hipErrorInvalidSymbol;
        if (tracked) g_device[dev].static_scratch.store(p, std::memory_order_release);
    }
    *ptr = p;
    return hipSuccess;
}

// The single-pass schedule on a carved workspace: one counter-clearing kernel, then one launch
// per c_S queries.  Arguments have been checked.
si_status run_fused(const void* q, const void* K, const float* w, const si_dims& d, int32_t m, int32_t k,
                    int32_t mask_mode, int32_t c_S, int32_t waves, const FusedLayout& L, int32_t* out_idx,
                    float* out_score, hipStream_t hs) {
    if (waves == 0) waves = fused_shape_for(d, m, mask_mode);
    int32_t n_wg = 0;
    hipError_t e = fused_workgroups(waves, &n_wg);
    if (e != hipSuccess) return hip_fail(e);
    e = timed(kProfInit, hs, [&] {
        return launch_zero_ints(L.counters, static_cast<int32_t>(L.n_launches), hs);
    });
    if (e != hipSuccess) return hip_fail(e);
    int64_t launch = 0;
    for (int64_t s0 = 0; s0 < d.S; s0 += c_S, ++launch) {
        const int32_t rows = static_cast<int32_t>(std::min<int64_t>(c_S, d.S - s0));
        e = timed(waves == 8 ? kProfFused : kProfFusedNarrow, hs, [&] {
            // (timed holds the profiler's lock: the phase clock's buffer is read under it)
            unsigned long long* phase = g_prof.phase_slots >= n_wg ? g_prof.phase : nullptr;
            if (phase != nullptr && !(d.D == 128 && d.H_I > 32 && k <= 1024)) phase = nullptr;
            return launch_fused(q, K, w, d, m, mask_mode, k, static_cast<int32_t>(s0), rows, L.slots,
                                waves, n_wg, L.counters + launch, out_idx, out_score, phase,
                                g_prof.phase_slots, hs);
        });
        if (e != hipSuccess) return hip_fail(e);
    }
    return SI_OK;
}

// ---- few query rows: key axis split over the chip (rows.hip) -------------------------------
// Workgroups per row of a selection over n entries: enough for the chip's compute units, at least
// kMinPart entries each.
constexpr int32_t kMinPart = 4096;
// Group maxima of a row of n entries from row_maxima_kernel: 64 per 2048 << lg entries.
int64_t row_maxima_count(int64_t n, int32_t lg) { return (n + (int64_t{2048} << lg) - 1) / (int64_t{2048} << lg) * 64; }
int32_t row_parts_for(int64_t R, int64_t n) {
    const int64_t by_rows = kFusedSlots / std::max<int64_t>(R, 1);
    return static_cast<int32_t>(std::max<int64_t>(1, std::min<int64_t>(by_rows, n / kMinPart)));
}
// Carves what a selection of R rows of n entries with n_maxima group maxima and a list of list_cap keys each needs behind `off`
// bytes of the workspace; returns the bytes used.
size_t carve_selection(void* base, size_t off, int64_t R, int64_t n, int32_t n_parts, int64_t n_maxima, int32_t list_cap,
                       RowSelection* sel) {
    *sel = RowSelection{};
    sel->n_parts = n_parts;
    sel->part_len = static_cast<int32_t>((n + n_parts - 1) / n_parts);
    if (n_parts == 1) return off;
    char* p = static_cast<char*>(base);
    off = align_up(off, 256);
    sel->n_maxima = static_cast<int32_t>(n_maxima);
    sel->maxima = reinterpret_cast<float*>(p + off);
    off = align_up(off + static_cast<size_t>(R) * n_maxima * sizeof(float), 256);
    sel->list_cap = list_cap;
    sel->lists = reinterpret_cast<key64_t*>(p + off);
    off = align_up(off + static_cast<size_t>(R) * list_cap * sizeof(key64_t), 256);
    sel->held = reinterpret_cast<unsigned long long*>(p + off);
    return off + static_cast<size_t>(R) * sizeof(unsigned long long);
}
// The selection of caller-supplied rows by several workgroups per row, if the rows are long enough and what they exchange fits
// the workspace: maxima of groups of 32 entries and a list of kRowListCap(k) keys, or, as many workspaces hold less than that, of
// groups twice, four times .. as large and a list of what is left.  Measured on MI355X (us, one workgroup -> several, 1 and 64
// rows): 24576 scores, k = 20 11 -> 13, 12 -> 14, k = 300 13 -> 14, 13 -> 14; 32768 scores, k = 20 13 -> 14, 13 -> 15, k = 300
// 15 -> 13, 15 -> 15, k = 512 17 -> 13, 17 -> 15; 45056 scores, k = 20 16 -> 14, 17 -> 15, k = 512 21 -> 14, 22 -> 16.  Larger groups
// let more through and two or three workgroups a row share little: 32768 scores, k = 20 in a small workspace 13 -> 16, 14 -> 17;
// 128 rows, k = 300 16 -> 18; 45056, k = 20, small workspace 16 -> 16, 17 -> 18.
constexpr int64_t kCallerPartsMin = 49152;
int64_t caller_parts_min(int32_t n_parts, int32_t k) {  // with groups of 32 entries and a list of kRowListCap(k)
    if (n_parts < 3) return kCallerPartsMin;
    return n_parts == 3 ? 40960 : k < 256 ? 36864 : 32768;
}
// Keys the joint list must have room for.  Of the maxima of M groups of normal scores the k-th largest lets about 1.07 k keys pass
// with M = 8 k, 1.16 k with 4 k, 1.4 k with 2 k; M is what the kernel folds them to (with that left out, a list of 5300 keys,
// k = 4096, 1 x 1048576 overflowed, which sends the row's last workgroup through the row alone: 169 us instead of 34).
int64_t caller_list_min(int64_t n_maxima, int64_t k) {
    const int64_t groups = std::min<int64_t>(n_maxima, int64_t{kPartsThreads} * kPartsMaxima(static_cast<int>(k)));
    const int64_t sixteenths = groups >= 8 * k ? 20 : groups >= 4 * k ? 24 : 28;
    return std::max<int64_t>(512, k * sixteenths / 16);
}
void carve_caller_rows(void* base, size_t bytes, int64_t R, int64_t n, int32_t k, RowSelection* sel) {
    const int32_t n_parts = row_parts_for(R, n);
    if (n_parts > 1 && n >= caller_parts_min(n_parts, k)) {
        const int64_t of_32 = row_maxima_count(n, 0);
        if (of_32 >= 2 * static_cast<int64_t>(k) && carve_selection(base, 0, R, n, n_parts, of_32, kRowListCap(k), sel) <= bytes) return;
    }
    if (n_parts > 1 && n >= kCallerPartsMin) {
        for (int32_t lg = 0; lg <= 5; ++lg) {
            const int64_t n_maxima = row_maxima_count(n, lg);
            if (n_maxima < 2 * static_cast<int64_t>(k)) break;
            const int64_t row_bytes = n_maxima * static_cast<int64_t>(sizeof(float)) + static_cast<int64_t>(sizeof(unsigned long long));
            const int64_t for_lists = static_cast<int64_t>(bytes) - R * row_bytes - 3 * 256;
            const int64_t room = for_lists / (R * static_cast<int64_t>(sizeof(key64_t)));
            const int32_t cap = static_cast<int32_t>(std::min<int64_t>(kRowListCap(k), room));
            if (cap < caller_list_min(n_maxima, k)) continue;
            if (carve_selection(base, 0, R, n, n_parts, n_maxima, cap, sel) > bytes) continue;
            sel->maxima_lg = lg;
            return;
        }
    }
    carve_selection(base, 0, R, n, 1, 0, 0, sel);
}

// The dense schedule: the scores of `rows` query rows per batch as fp32 rows in the workspace, then the
// selection over them.
struct RowsLayout {
    int32_t rows;     // query rows per batch and tile
    int32_t batches;  // batches per tile: all, unless the rows of a tile are whole
    int32_t n_cols;  // length of a score row: the legal keys of the longest row, at least 1
    float* scores;
    RowSelection sel;
    size_t bytes;
};
// Fewer query rows than this per batch: a wave's keys serve its one query (score_rows_kernel); from here
// on the sweep, whose 8 waves share the staged keys: 64 batches, 64 heads of 128, 8192 keys, whole call, 7 queries by the
// former 95 us, 8 by the latter 80.
constexpr int32_t kSharedKeysRows = 8;
RowsLayout carve_rows(void* base, const si_dims& d, int32_t n_cols, int32_t k, int32_t rows, int32_t batches) {
    RowsLayout L;
    const int64_t R = static_cast<int64_t>(batches) * rows;
    L.rows = rows;
    L.batches = batches;
    L.n_cols = n_cols;
    L.scores = static_cast<float*>(base);
    // Group maxima for the selection's bound, which needs at least 2k groups to be of use: of 32 or 8
    // consecutive keys from score_rows_kernel, 64 per 2048 entries from row_maxima_kernel.
    const int32_t lg = rows >= kSharedKeysRows ? 0 : n_cols / 32 >= 4 * static_cast<int64_t>(k) ? 5 : 3;
    const int64_t n_maxima = lg == 0 ? row_maxima_count(n_cols, 0) : (static_cast<int64_t>(n_cols) + (1 << lg) - 1) >> lg;
    const int32_t n_parts = rows == d.S && n_maxima >= 2 * static_cast<int64_t>(k) ? row_parts_for(R, n_cols) : 1;
    L.bytes = carve_selection(base, static_cast<size_t>(R) * n_cols * sizeof(float), R, n_cols, n_parts, n_maxima, kRowListCap(k), &L.sel);
    L.sel.group_lg = lg;
    return L;
}

// Whether si_indexer_topk takes the dense schedule, and its layout.  Measured on MI355X (64 heads of 128,
// us, single pass -> dense; all with the same bits):
//   one query, 262144 keys, k = 1024                       4180 ->  33
//   64 / 512 / 2048 queries, 16384 keys each, k = 512       254 ->  33,  260 -> 133,  495 -> 463
//   prompts, causal, k = 512: 2049 / 4096 / 8192 queries     48 ->  33,   80 ->  60,  205 -> 171
//                             16384 / 32768 queries         649 -> 576,  2219 -> 2235 (in another run 2131 -> 2085)
//                             65536 queries, 16384 keys    7847 -> 8001
// The single pass leaves compute units idle below 2048 queries (8 per unit) and pays its merges and
// write-outs with the matrix cores idle; the dense schedule writes and reads every score once more,
// which grows with the key range.  So: dense up to kDenseMaxKeys keys per query, or where there are few
// rows; with fewer than kSharedKeysRows queries per batch, see decoding_layout.  All rows must fit the workspace at once, with
// k <= kFusedMaxK; beyond, where the alternative is the tiled schedule, tiles of at least 1024 rows will do (16384 queries and
// keys, k = 4096: 4701 -> 2671).
// Only up to kDenseMaxKeysCheap where the single pass has less to do per row (k <= 1024; longer lists it sorts by the
// network): with k below 256 its merges and write-outs are short, and with few heads the ReLU makes one score in 2^heads
// exactly 0, which the single pass drops at its threshold and a selection has to cut from its list (most for the short
// rows of a causal prompt, which enter the list whole).  Single pass -> dense, us: 64 heads of 128, causal, k = 64: 16384
// queries of 4096 keys 599 -> 564, 20000 of 5000 821 -> 874, 32768 of 8192 1992 -> 2138 (k = 512: 649 -> 576, 880 -> 899,
// 2131 -> 2085); causal, k = 512, 4096 and 8192 keys: 1 head of 128 536 -> 406, 1557 -> 1944, 4 heads of 32 375 -> 260,
// 1075 -> 1153, 8 heads of 64 340 -> 262, 1053 -> 1051; 9000 queries of 8192 keys, no mask, k = 512: 1 head 769 -> 931, 2
// heads 626 -> 569, 4 heads 544 -> 420; 32768 of 8192, k = 2048: 1 head 2734 -> 1812, 4 heads 2131 -> 1267.
constexpr int32_t kDenseMaxKeys = 8192;
constexpr int32_t kDenseMaxKeysTiled = 32768;
constexpr int32_t kDenseMaxKeysCheap = 4096;
int32_t dense_max_keys(const si_dims& d, int32_t k, int32_t mask_mode) {
    if (k > kFusedMaxK) return kDenseMaxKeysTiled;
    const bool few_heads = d.H_I < (mask_mode == SI_MASK_CAUSAL_BLOCK ? 8 : 2);
    return k <= kFusedMaxRankedK && (k < 256 || few_heads) ? kDenseMaxKeysCheap : kDenseMaxKeys;
}
// (Rows of up to 2048 keys mostly take one kernel instead: short_rows below.)
// Few rows: where the single pass leaves compute units idle, 8 queries each.  With very long rows, where its merges are rare and
// writing and reading the scores weighs more, only where it leaves many idle.  Time of dense over that of the single pass, all
// head shapes (median, rows 1281 to 1408 / 1409 to 1536 / 1537 to 1792 / 1921 to 2048): k <= 1024, keys 32769 to 65536 0.91 / 0.96 /
// 0.99 / 1.01, to 98304 0.87 / 1.02 / 1.03 / 1.05, to 131072 0.87 / 1.03 / 1.05 / 1.07, to 262144 0.93 / 1.07 / 1.07 / 1.08; k > 1024 to
// 65536 0.82 / 0.89 / 0.90 / 0.94, to 131072 0.85 / 0.97 / 0.97 / 0.99, to 262144 0.93 / 1.01 / 1.02 / 1.02.
constexpr int32_t kFewRows = kFusedSlots * kQueriesPerBlock;
struct FewRowsLine {
    int32_t keys, rows;  // beyond so many keys up to so many rows
};
constexpr FewRowsLine kFewRowsShortLists = {98304, 1408}, kFewRowsLongLists = {65536, 1536};
int32_t few_rows(int32_t longest, int32_t k) {
    if (k > kFusedMaxK) return kFewRows;
    const FewRowsLine line = k <= kFusedMaxRankedK ? kFewRowsShortLists : kFewRowsLongLists;
    return longest > line.keys ? line.rows : kFewRows;
}
// Batches whose queries fill the last group of eight badly: workgroups of four queries take them all in one round where those of
// eight, which write dense scores, need a second one.  133 x 11 queries of 8528 keys, 64 heads of 128, k = 28 234 us single pass, 369
// dense; over all head shapes, 2049 to 16384 keys, dense takes 1.11 to 1.43 of its time (medians), with k > 1024 0.64 to 1.17.
bool single_pass_has_one_round(const si_dims& d, int32_t longest, int32_t k) {
    const int64_t B = d.B, S = d.S;
    return k <= kFusedMaxRankedK && longest <= kNarrowMaxKeys && B * ((S + 7) / 8) > kFusedSlots && B * ((S + 3) / 4) <= 2 * kFusedSlots;
}
// Decoding (1 .. 7 queries of any number of batches): the dense schedule, at once or in tiles of as many batches as the workspace has
// room for, where that takes less time than the single pass, in which a workgroup takes the keys to one or a few queries of its batch.
// Both times (us) by sums fitted to 23779 calls on MI355X (1 to 20000 batches, 64 to 250000 keys, all head shapes, 1 to 20 tiles;
// eight in ten within 18 %):
//   dense        15, 17 for every further tile, the keys' trip at 6.3 TB/s for every four queries, the work per score, and a row's
//                selection by
//                the length of its list;
//   single pass  a step of 64 keys a round of workgroups, more with matrix work and with more workgroups fetching keys, and per
//                round the merges and the write-out; lists it sorts by the network (k > 1024) cost narrow workgroups a step more
//                (left out, the narrow shape's sum was 0.70 of its time there, and 117 x 7 queries of 4060 keys, k = 1227 went to it:
//                104 -> 135).
// The choice costs 0.6 % on average over the better of the two; 2.5 % of the calls lose more than a tenth.  (us, single pass -> dense:
// 287 x 3 queries of 39218 keys, 64 heads of 32, 938 -> 341; 276 x 3 of 65014 1323 -> 522; 503 x 6 of 3395, 4 heads of 32, 213 -> 92;
// 240 x 4 of 7900, 33 heads of 128, and 93 x 7 of 11952 in four tiles are the single pass's, 194 against 317 the latter.)
double dense_few_us(const si_dims& d, int32_t n_cols, int32_t k, int64_t tiles) {
    const double rows = static_cast<double>(d.B) * d.S;
    const double key_mb = static_cast<double>(d.B) * n_cols * d.D * 2 * 1e-6;
    const double blocks = (d.H_I + 31) / 32, matrix = blocks * d.D / 256.0;
    return 17.0 * static_cast<double>(tiles) - 2.4 + 0.153 * ((d.S + 3) / 4) * key_mb + (10.5 * matrix + 1.26 * blocks) * rows * n_cols * 1e-6 +
           rows * (0.0012 + 4.5e-6 * std::min(k, n_cols));
}
double single_pass_few_us(const si_dims& d, int32_t n_cols, int32_t k, int32_t shape) {
    const double blocks = (d.H_I + 31) / 32, matrix = blocks * d.D / 256.0, steps = n_cols / 64.0;
    const double workgroups = static_cast<double>(d.B) * ((d.S + shape - 1) / shape);
    const bool network = k > kFusedMaxRankedK;
    if (shape == 8) {
        const double trip = 0.34 * std::min(1.0, workgroups / kFusedSlots) * d.D / 128;
        return wide_rounds(d) * (steps * (0.143 + 0.578 * matrix + 0.15 * blocks + trip + (network ? 0.09 : 0.0)) + 0.028 * k + 24.6);
    }
    const double trip = 0.34 * std::min(1.0, workgroups / (2 * kFusedSlots)) * d.D / 128;
    const double queries = 0.14 * std::min(d.S, 4) / 4;
    return narrow_rounds(d) * (steps * (0.416 + 0.97 * matrix + 0.03 * blocks + queries + trip + (network ? 0.94 : 0.0)) + 0.0026 * k + 7.1) + 12.6;
}
bool decoding_layout(void* workspace, size_t workspace_bytes, const si_dims& d, int32_t n_cols, int32_t k, bool single_pass,
                     int32_t fused_shape, RowsLayout* L) {
    const auto fits = [&](int64_t batches) {
        return carve_rows(nullptr, d, n_cols, k, d.S, static_cast<int32_t>(batches)).bytes <= workspace_bytes;
    };
    int64_t nb = d.B;
    if (!fits(nb)) {
        // Down from as many as the scores alone have room for: the fewer rows a tile has, the more workgroups share each of them, and
        // the joint lists those need can make a smaller tile the larger one (up from one batch, 300 x 1 queries of 38062 keys, k = 595
        // came to 126 batches a tile instead of 169).
        nb = static_cast<int64_t>(workspace_bytes / (static_cast<size_t>(d.S) * n_cols * sizeof(float)));
        nb = std::min<int64_t>(d.B, nb);
        while (nb > 0 && !fits(nb)) --nb;
        if (nb < 1) return false;
        const int64_t least = (d.B + nb - 1) / nb, even = (d.B + least - 1) / least;
        if (fits(even)) nb = even;
    }
    const int64_t tiles = (d.B + nb - 1) / nb;
    if ((single_pass || tiles > 1) && dense_few_us(d, n_cols, k, tiles) >= single_pass_few_us(d, n_cols, k, fused_shape)) return false;
    *L = carve_rows(workspace, d, n_cols, k, d.S, static_cast<int32_t>(nb));
    return L->bytes <= workspace_bytes;
}
// single_pass: the workspace holds the single pass's buffers as well.
bool dense_layout(void* workspace, size_t workspace_bytes, const si_dims& d, int32_t m, int32_t k, int32_t mask_mode,
                  bool single_pass, RowsLayout* L) {
    const int64_t R = static_cast<int64_t>(d.B) * d.S;
    const int32_t longest = longest_row(d, m, mask_mode);
    const int32_t n_cols = std::max(longest, 1);
    if (R >= (1 << 20) || d.B > 65535) return false;  // the launches' grids
    if (d.S < kSharedKeysRows && k <= kFusedMaxK)
        return decoding_layout(workspace, workspace_bytes, d, n_cols, k, single_pass, fused_shape_for(d, m, mask_mode), L);
    if (single_pass && single_pass_has_one_round(d, longest, k)) return false;
    const bool few = R <= few_rows(longest, k);
    if (!few && longest > dense_max_keys(d, k, mask_mode)) return false;
    *L = carve_rows(workspace, d, n_cols, k, d.S, d.B);
    if (L->bytes <= workspace_bytes) return true;
    if (k <= kFusedMaxK) return false;
    const int64_t rows = static_cast<int64_t>(workspace_bytes / (static_cast<size_t>(d.B) * n_cols * sizeof(float))) / 8 * 8;
    if (rows * d.B < 1024 || rows < kSharedKeysRows || rows >= d.S) return false;
    *L = carve_rows(workspace, d, n_cols, k, static_cast<int32_t>(rows), d.B);
    return L->bytes <= workspace_bytes;
}

si_status run_rows(const void* q, const void* K, const float* w, const si_dims& all, int32_t m, int32_t k,
                   int32_t mask_mode, const RowsLayout& L, int32_t* out_idx, float* out_score, hipStream_t hs) {
    const bool shared = L.rows >= kSharedKeysRows;
    for (int32_t b0 = 0; b0 < all.B; b0 += L.batches) {
        si_dims d = all;
        d.B = std::min(L.batches, all.B - b0);
        const int64_t row0 = static_cast<int64_t>(b0) * d.S;
        const char* const qb = static_cast<const char*>(q) + row0 * d.H_I * d.D * 2;
        const char* const Kb = static_cast<const char*>(K) + static_cast<int64_t>(b0) * d.T * d.D * 2;
        const float* const wb = w + row0 * d.H_I;
        for (int32_t s0 = 0; s0 < d.S; s0 += L.rows) {
            const RowTile tile{s0, std::min(L.rows, d.S - s0), d.S};
            hipError_t e = timed(kProfScore, hs, [&] {
                return shared ? launch_score_tile(qb, Kb, wb, d, m, mask_mode, s0, 0, tile.rows, L.n_cols, tile.rows, L.n_cols, L.scores, hs)
                              : launch_score_rows(qb, Kb, wb, d, m, mask_mode, L.n_cols, L.sel, L.scores, hs);
            });
            if (e != hipSuccess) return hip_fail(e);
            if (shared && L.sel.n_parts > 1) {
                e = timed(kProfInit, hs, [&] {
                    return launch_row_maxima(L.scores, d.B * d.S, L.n_cols, nullptr, d.S, m, mask_mode, L.sel, hs);
                });
                if (e != hipSuccess) return hip_fail(e);
            }
            e = timed(kProfFinalize, hs, [&] {
                return launch_select_rows(L.scores, d.B * tile.rows, L.n_cols, nullptr, tile, m, mask_mode, k, L.sel,
                                          out_idx + row0 * k, out_score + row0 * k, hs);
            });
            if (e != hipSuccess) return hip_fail(e);
            if (d.S - s0 <= L.rows) break;  // (s0 + rows could pass the range of an int)
        }
        if (all.B - b0 <= L.batches) break;
    }
    return SI_OK;
}

// Whether a row's best k end among scores of exactly 0, of which the ReLU makes one in 2^heads: then the bins of either selection do not
// separate them, and the exact one that follows runs longer in the kernel that also sweeps, with two waves per SIMD, than in the one
// that only selects, with three or four, once there are rows for it (1792: launch_select_rows).  Time of one kernel over dense, 1 / 2 /
// 3 heads (medians): 513 to 1024 wanted, below 4096 rows 1.07 / 1.06 / 0.98, from there 1.22 / 1.21 / 1.18 (7912 rows of 884 keys, 1 head of
// 128, k = 639 186 us, dense 151); 257 to 512 wanted 1.05 / 1.02 / 0.86 and 1.15 / 1.12 / 0.90; up to 256 1.00 / 0.91 / 0.88 and 1.09 /
// 0.90 / 0.89; from 4 heads on 0.8 to 0.97; fewer rows 0.6 to 1.05.
bool ends_among_zeros(const si_dims& d, int32_t longest, int32_t k) {
    const int64_t wanted = std::min(k, longest);
    const int32_t heads = wanted > 512 ? 3 : wanted > 256 ? 2 : wanted > 128 ? 1 : 0;
    return d.H_I <= heads && static_cast<int64_t>(d.B) * d.S >= 1792 && ((longest - wanted) << d.H_I) < longest;
}
// Whether the dense schedule's two steps go into one kernel that keeps a row's scores on chip (short_rows.hip): rows of up to
// 1024 keys, or of up to 2048 where there are enough of them that whole rows, one a wave, occupy the chip; with few long rows only
// the kernel that splits the key axis does.  Measured on MI355X (us, dense / single pass / one kernel; the same bits): prompts,
// causal, k = 512, 64 heads of 128, 4096 / 8192 queries of 1024 / 2048 keys 56 / 76 / 50, 156 / 191 / 143; 2 x 8191 queries, 33 heads of
// 64, k = 300 187 / 234 / 180.  No mask, over 64 heads of 128, 33 of 64, 16 of 128 and 4 of 32, time ratio: 8 to 512 rows of 128 to 768
// keys 0.61 to 0.89, of 1024 0.85 to 1.03, of 1536 and 2048 0.84 to 1.55; 768 and more rows of any length 0.6 to 1.04.  Lists of 513 to
// 1024, all head shapes, medians: 8 to 767 rows of up to 1024 keys 0.74 to 0.81, of 1025 to 1536 0.89 to 1.05, of more 0.93 to 1.19; more
// rows 0.70 to 0.92.  dense_fits: the workspace holds dense scores.
bool short_rows(const si_dims& d, int32_t m, int32_t k, int32_t mask_mode, bool dense_fits) {
    const int32_t longest = longest_row(d, m, mask_mode);
    if (d.S < kSharedKeysRows || longest > kShortMaxKeys || std::min(k, longest) > kShortMaxK) return false;
    if (d.S > kShortMaxQueries || d.B > 65535) return false;  // the launch's grid
    if (dense_fits && ends_among_zeros(d, longest, k)) return false;
    return longest <= 1024 || static_cast<int64_t>(d.B) * d.S >= 768;
}
si_status run_short_rows(const void* q, const void* K, const float* w, const si_dims& d, int32_t m, int32_t k,
                         int32_t mask_mode, int32_t* out_idx, float* out_score, hipStream_t hs) {
    const hipError_t e = timed(kProfScore, hs, [&] {
        return launch_short_rows(q, K, w, d, m, mask_mode, k, longest_row(d, m, mask_mode), out_idx, out_score, hs);
    });
    return e == hipSuccess ? SI_OK : hip_fail(e);
}
}  // namespace

// Per query row of a tile: a key buffer of 2k + c_T slots (a row is cut back to k as soon as
// it holds 2k, and one key tile adds at most c_T), a count and a threshold.
RowBuffers carve_workspace(void* base, int64_t rows_, int64_t k, int64_t c_T) {
    RowBuffers rb;
    const size_t rows = static_cast<size_t>(rows_);
    rb.cap = static_cast<int32_t>(2 * k + c_T);
    size_t off = 0;
    char* p = static_cast<char*>(base);
    rb.keys = reinterpret_cast<key64_t*>(p + off);
    off = align_up(off + rows * static_cast<size_t>(rb.cap) * sizeof(key64_t), 256);
    rb.count = reinterpret_cast<int32_t*>(p + off);
    off = align_up(off + rows * sizeof(int32_t), 256);
    rb.theta = reinterpret_cast<float*>(p + off);
    off = align_up(off + rows * sizeof(float), 256);
    rb.bytes = off;
    return rb;
}

}  // namespace si

using namespace si;

extern "C" {

size_t si_workspace_bytes(const si_dims* dims, int32_t k, int32_t c_S, int32_t c_T) {
    if (!dims || dims->B < 1 || dims->S < 1 || dims->T < 1 || k < 1 || c_S < 1 || c_T < 1) return 0;
    const int64_t cs = std::min<int64_t>(c_S, dims->S);
    const int64_t ct = std::min<int64_t>(c_T, dims->T);
    return workspace_bytes_for(dims->B, cs, ct, k);
}

si_status si_plan_tiles(const si_dims* dims, int32_t m, int32_t k, si_mask_mode mask_mode,
                        size_t hbm_budget_bytes, si_plan* out) {
    si_status st = check_dims(dims, m, k, mask_mode);
    if (st != SI_OK) return st;
    if (!out) return SI_ERR_INVALID_ARG;
    // Measured on MI355X (flash_1m, 8 GB budget): larger tiles win on both axes.  Fewer, longer
    // launches lose less to the drain at every kernel boundary, and every key tile costs one
    // pass of the compaction kernel over all rows.  The workgroups of a launch walk the key
    // tile in step, so the part of K in use at any moment is small whatever c_T is.  Rule:
    // the largest key tile (up to 32768) for which a query tile at least as long (up to 32768)
    // still fits the budget; failing that, the smallest query tile and a shrinking key tile.
    const int64_t B = dims->B;
    const int64_t s_cap = std::min<int64_t>(dims->S, std::max<int64_t>(kQueriesPerBlock, 32768 / B));
    auto fit_rows = [&](int64_t c_T) {  // longest query tile (multiple of 8, or all of S) within the budget
        int64_t lo = 0, hi = s_cap;     // workspace grows with c_S: bisect
        while (lo < hi) {
            const int64_t mid = (lo + hi + 1) / 2;
            if (workspace_bytes_for(B, mid, c_T, k) <= hbm_budget_bytes) lo = mid; else hi = mid - 1;
        }
        if (lo < dims->S) lo = lo / kQueriesPerBlock * kQueriesPerBlock;
        return lo;
    };
    static const int64_t key_tiles[] = {32768, 24576, 16384, 12288, 8192, 6144, 4096, 3072, 2048, 1024,
                                        512, 256, 128, 64, 32};
    int64_t best_S = 0, best_T = 0;
    for (int64_t cand : key_tiles) {
        const int64_t c_T = std::min<int64_t>(cand, dims->T);
        const int64_t c_S = fit_rows(c_T);
        if (c_S >= std::min<int64_t>(c_T, s_cap)) {  // balanced tile found
            best_S = c_S;
            best_T = c_T;
            break;
        }
        if (c_S >= kQueriesPerBlock || c_S == dims->S) {  // remember the widest key tile that fits at all
            if (best_S == 0 || c_S * c_T > best_S * best_T) {
                best_S = c_S;
                best_T = c_T;
            }
        }
    }
    if (best_S == 0) return SI_ERR_WORKSPACE_TOO_SMALL;
    out->c_S = static_cast<int32_t>(best_S);
    out->c_T = static_cast<int32_t>(best_T);
    out->workspace_bytes = workspace_bytes_for(B, best_S, best_T, k);
    return SI_OK;
}

si_status si_score_tile(const void* q, const void* K, const float* w, const si_dims* dims,
                        int32_t m, si_mask_mode mask_mode, int32_t s0, int32_t t0,
                        int32_t c_S, int32_t c_T, float* tile, void* stream) {
    si_status st = check_dims(dims, m, 1, mask_mode);
    if (st != SI_OK) return st;
    if (!q || !K || !w || !tile) return SI_ERR_INVALID_ARG;
    if (s0 < 0 || t0 < 0 || c_S < 1 || c_T < 1 || s0 >= dims->S || t0 >= dims->T) return SI_ERR_INVALID_ARG;
    const int32_t rows = std::min<int64_t>(c_S, static_cast<int64_t>(dims->S) - s0);
    const int32_t width = std::min<int64_t>(c_T, static_cast<int64_t>(dims->T) - t0);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    hipError_t e = timed(kProfScore, hs, [&] {
        return launch_score_tile(q, K, w, *dims, m, mask_mode, s0, t0, rows, width, c_S, c_T, tile, hs);
    });
    return e == hipSuccess ? SI_OK : hip_fail(e);
}

si_status si_indexer_topk_tiled(const void* q, const void* K, const float* w,
                                const si_dims* dims, int32_t m, int32_t k,
                                si_mask_mode mask_mode, int32_t c_S, int32_t c_T,
                                int32_t* out_idx, float* out_score, void* workspace,
                                size_t workspace_bytes, void* stream) {
    si_status st = check_dims(dims, m, k, mask_mode);
    if (st != SI_OK) return st;
    if (!q || !K || !w || !out_idx || !out_score || !workspace) return SI_ERR_INVALID_ARG;
    if (c_S < 1 || c_T < 1) return SI_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return SI_ERR_INVALID_ARG;
    const si_dims d = *dims;
    c_S = std::min(c_S, d.S);
    c_T = std::min(c_T, d.T);
    const RowBuffers rb = carve_workspace(workspace, static_cast<int64_t>(d.B) * c_S, k, c_T);
    if (rb.bytes > workspace_bytes) return SI_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t hs = static_cast<hipStream_t>(stream);

    for (int64_t s0 = 0; s0 < d.S; s0 += c_S) {
        const int32_t rows = static_cast<int32_t>(std::min<int64_t>(c_S, d.S - s0));
        hipError_t e = timed(kProfInit, hs, [&] { return launch_init_rows(rb, d.B * c_S, hs); });
        if (e != hipSuccess) return hip_fail(e);
        // keys visible to the last query of this tile (Section 4.2); later key tiles are skipped
        int64_t t_hi = d.T;
        if (mask_mode == SI_MASK_CAUSAL_BLOCK) t_hi = std::min<int64_t>(d.T, (s0 + rows) / m);
        for (int64_t t0 = 0; t0 < t_hi;) {
            const int32_t width = static_cast<int32_t>(std::min<int64_t>(next_width(t0, c_T, k), d.T - t0));
            e = timed(kProfScore, hs, [&] {
                return launch_score_filter(q, K, w, d, m, mask_mode, k, static_cast<int32_t>(s0),
                                           static_cast<int32_t>(t0), rows, width, c_S, rb, hs);
            });
            if (e != hipSuccess) return hip_fail(e);
            e = timed(kProfCompact, hs, [&] { return launch_compact(rb, d.B, rows, c_S, k, 2 * k, hs); });
            if (e != hipSuccess) return hip_fail(e);
            t0 += width;
        }
        e = timed(kProfFinalize, hs, [&] {
            return launch_finalize(rb, d.B, rows, c_S, k, d.S, s0, out_idx, out_score, hs);
        });
        if (e != hipSuccess) return hip_fail(e);
    }
    return SI_OK;
}

si_status si_indexer_topk(const void* q, const void* K, const float* w, const si_dims* dims,
                          int32_t m, int32_t k, si_mask_mode mask_mode, int32_t* out_idx,
                          float* out_score, void* workspace, size_t workspace_bytes,
                          void* stream) {
    // The single-pass schedule whenever it applies (k <= 2048) and its small workspace fits;
    // otherwise the tiled schedule with the plan for this budget.  A workspace that neither accepts is
    // refused, also where the dense schedule would need less.
    const size_t fused_bytes = si_fused_workspace_bytes(dims, k, 0);
    const bool fused = fused_bytes != 0 && fused_bytes <= workspace_bytes;
    si_plan plan;
    if (!fused) {
        si_status st = si_plan_tiles(dims, m, k, mask_mode, workspace_bytes, &plan);
        if (st != SI_OK) return st;
    }
    RowsLayout dense;
    if (check_dims(dims, m, k, mask_mode) == SI_OK && q && K && w && out_idx && out_score && workspace &&
        reinterpret_cast<uintptr_t>(workspace) % 256 == 0) {
        const bool fits = dense_layout(workspace, workspace_bytes, *dims, m, k, mask_mode, fused, &dense);
        if ((fits || fused) && short_rows(*dims, m, k, mask_mode, fits))
            return run_short_rows(q, K, w, *dims, m, k, mask_mode, out_idx, out_score, static_cast<hipStream_t>(stream));
        if (fits)
            return run_rows(q, K, w, *dims, m, k, mask_mode, dense, out_idx, out_score, static_cast<hipStream_t>(stream));
    }
    if (fused)
        return si_indexer_topk_fused(q, K, w, dims, m, k, mask_mode, 0, out_idx, out_score, workspace,
                                     workspace_bytes, stream);
    return si_indexer_topk_tiled(q, K, w, dims, m, k, mask_mode, plan.c_S, plan.c_T, out_idx,
                                 out_score, workspace, workspace_bytes, stream);
}

size_t si_fused_workspace_bytes(const si_dims* dims, int32_t k, int32_t c_S) {
    if (!dims || dims->S < 1 || k < 1 || k > kFusedMaxK) return 0;
    c_S = fused_rows_per_launch(c_S, dims->S);
    return carve_fused(nullptr, dims->S, k, c_S).bytes;
}

si_status si_indexer_topk_fused_shape(const void* q, const void* K, const float* w, const si_dims* dims,
                                      int32_t m, int32_t k, si_mask_mode mask_mode, int32_t c_S,
                                      int32_t queries_per_workgroup, int32_t* out_idx, float* out_score,
                                      void* workspace, size_t workspace_bytes, void* stream) {
    si_status st = check_dims(dims, m, k, mask_mode);
    if (st != SI_OK) return st;
    if (k > kFusedMaxK) return SI_ERR_UNSUPPORTED_SHAPE;
    if (!q || !K || !w || !out_idx || !out_score || !workspace) return SI_ERR_INVALID_ARG;
    if (queries_per_workgroup != 0 && queries_per_workgroup != 4 && queries_per_workgroup != 8)
        return SI_ERR_INVALID_ARG;
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return SI_ERR_INVALID_ARG;
    c_S = fused_rows_per_launch(c_S, dims->S);
    const FusedLayout L = carve_fused(workspace, dims->S, k, c_S);
    if (L.bytes > workspace_bytes) return SI_ERR_WORKSPACE_TOO_SMALL;
    return run_fused(q, K, w, *dims, m, k, mask_mode, c_S, queries_per_workgroup, L, out_idx, out_score,
                     static_cast<hipStream_t>(stream));
}

si_status si_indexer_topk_fused(const void* q, const void* K, const float* w, const si_dims* dims,
                                int32_t m, int32_t k, si_mask_mode mask_mode, int32_t c_S,
                                int32_t* out_idx, float* out_score, void* workspace,
                                size_t workspace_bytes, void* stream) {
    return si_indexer_topk_fused_shape(q, K, w, dims, m, k, mask_mode, c_S, 0, out_idx, out_score,
                                       workspace, workspace_bytes, stream);
}

int32_t si_fused_shape_for(const si_dims* dims, int32_t m, int32_t k, si_mask_mode mask_mode) {
    if (check_dims(dims, m, k, mask_mode) != SI_OK || k > kFusedMaxK) return 0;
    return fused_shape_for(*dims, m, mask_mode);
}

si_status si_indexer_topk_static(const void* q, const void* K, const float* w, const si_dims* dims,
                                 int32_t m, int32_t k, si_mask_mode mask_mode, int32_t* out_idx,
                                 float* out_score, void* stream) {
    si_status st = check_dims(dims, m, k, mask_mode);
    if (st != SI_OK) return st;
    if (!q || !K || !w || !out_idx || !out_score) return SI_ERR_INVALID_ARG;
    // beyond what the static array was sized for: refuse, never spill over
    if (k > kStaticMaxK) return SI_ERR_UNSUPPORTED_SHAPE;
    const int32_t c_S = fused_rows_per_launch(0, dims->S);
    if ((static_cast<int64_t>(dims->S) + c_S - 1) / c_S > kStaticMaxLaunches) return SI_ERR_UNSUPPORTED_SHAPE;
    void* base = nullptr;
    hipError_t e = static_scratch(&base);
    if (e != hipSuccess) return hip_fail(e);
    const FusedLayout L = carve_fused(base, dims->S, k, c_S);
    if (L.bytes > kStaticScratchBytes) return SI_ERR_UNSUPPORTED_SHAPE;  // (cannot happen within the two limits)
    return run_fused(q, K, w, *dims, m, k, mask_mode, c_S, 0, L, out_idx, out_score,
                     static_cast<hipStream_t>(stream));
}

si_status si_topk_from_scores(const float* scores, int32_t R, int32_t n_cols,
                              const int32_t* legal, int32_t k, int32_t c_T, int32_t* out_idx,
                              float* out_score, void* workspace, size_t workspace_bytes,
                              void* stream) {
    if (!scores || !out_idx || !out_score || !workspace) return SI_ERR_INVALID_ARG;
    if (R < 1 || n_cols < 1 || k < 1 || c_T < 1) return SI_ERR_INVALID_ARG;
    if (k > kMaxK) return SI_ERR_UNSUPPORTED_SHAPE;
    if (reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return SI_ERR_INVALID_ARG;
    c_T = std::min(c_T, n_cols);
    if (carve_workspace(workspace, R, k, c_T).bytes > workspace_bytes) return SI_ERR_WORKSPACE_TOO_SMALL;
    hipStream_t hs = static_cast<hipStream_t>(stream);
    RowSelection sel;
    carve_caller_rows(workspace, workspace_bytes, R, n_cols, k, &sel);
    hipError_t e;
    if (sel.n_parts > 1) {
        e = timed(kProfInit, hs, [&] { return launch_row_maxima(scores, R, n_cols, legal, 1, 1, SI_MASK_NONE, sel, hs); });
        if (e != hipSuccess) return hip_fail(e);
    }
    e = timed(kProfFilterScores, hs, [&] {
        return launch_select_rows(scores, R, n_cols, legal, RowTile{0, 1, 1}, 1, SI_MASK_NONE, k, sel, out_idx,
                                  out_score, hs);
    });
    return e == hipSuccess ? SI_OK : hip_fail(e);
}

uint64_t si_materialize_bytes(const si_dims* dims) {
    if (!dims) return 0;
    return static_cast<uint64_t>(dims->B) * static_cast<uint64_t>(dims->S) *
           static_cast<uint64_t>(dims->H_I) * static_cast<uint64_t>(dims->T) * 4ull;
}

si_status si_profile_enable(int32_t on) {
    std::lock_guard<std::mutex> hold(g_prof.mu);
    g_prof.on = on != 0;
    return SI_OK;
}

si_status si_profile_phases(uint64_t* device_words, int32_t n_workgroups) {
    if (device_words != nullptr && n_workgroups < 1) return SI_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> hold(g_prof.mu);
    g_prof.phase = reinterpret_cast<unsigned long long*>(device_words);
    g_prof.phase_slots = device_words ? n_workgroups : 0;
    return SI_OK;
}

int32_t si_wall_clock_khz(void) {
    int dev = 0, khz = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&khz, hipDeviceAttributeWallClockRate, dev) != hipSuccess) return 0;
    return khz;
}

si_status si_profile_reset(void) {
    std::lock_guard<std::mutex> hold(g_prof.mu);
    hipError_t e = g_prof.drain();
    if (e != hipSuccess) return hip_fail(e);
    for (int i = 0; i < SI_PROFILE_CLASSES; ++i) {
        g_prof.ms[i] = 0.0;
        g_prof.launches[i] = 0;
    }
    return SI_OK;
}

si_status si_profile_read(double* ms_per_class, int64_t* launches_per_class) {
    if (!ms_per_class || !launches_per_class) return SI_ERR_INVALID_ARG;
    std::lock_guard<std::mutex> hold(g_prof.mu);
    hipError_t e = g_prof.drain();
    if (e != hipSuccess) return hip_fail(e);
    for (int i = 0; i < SI_PROFILE_CLASSES; ++i) {
        ms_per_class[i] = g_prof.ms[i];
        launches_per_class[i] = g_prof.launches[i];
    }
    return SI_OK;
}

const char* si_strerror(si_status status) {
    switch (status) {
        case SI_OK: return "ok";
        case SI_ERR_INVALID_ARG: return "invalid argument";
        case SI_ERR_UNSUPPORTED_SHAPE: return "unsupported shape (D in {32,64,128}, H_I <= 64, k <= 4096, T*D*2 < 2^32)";
        case SI_ERR_WORKSPACE_TOO_SMALL: return "workspace too small for this tiling";
        case SI_ERR_HIP: return "HIP runtime error (see si_last_hip_error)";
    }
    return "unknown status";
}

int32_t si_last_hip_error(void) { return g_last_hip_error; }

int32_t si_version(void) { return 100; }

}  // extern "C"
