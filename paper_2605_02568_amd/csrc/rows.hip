// The path for few query rows (decoding: one or a few positions of each request against its whole
// cache) and the selection of the best k of dense score rows, which it shares with
// si_topk_from_scores.
//
// With few rows the single-pass schedule leaves the chip idle: a workgroup takes 8 (4) consecutive
// queries of one batch through their whole key range, so one query uses one wave of one compute unit
// and its 262144 keys are one serial chain of 2048 key chunks (4.2 ms measured at one row, against
// 14 us that reading the keys takes).  Here the key axis is split over the chip instead:
//   score_rows_kernel    one wave = one query x a few 32-key blocks, scores to a dense fp32 row.  Bound by
//                        the trip of the keys from memory.
//   select_rows_kernel   one workgroup = one row.
//   select_parts_kernel  several workgroups per row, for rows long enough and few enough.  The scores
//                        come with the maxima of groups of consecutive keys, from which every
//                        workgroup derives the same bound for the whole row (topk_group.h): together
//                        the parts keep little more than k keys, and the last one to arrive sorts.
// Every score comes from the same instruction sequence as in score_sweep.h (MFMA steps in order of d
// on one accumulator, the head sum in register order, one exchange between the half-waves), and the
// selection is exact under the total order of Section 4.1, so the result is bit-identical to the other
// schedules'.

#include <algorithm>

#include "score_sweep.h"
#include "topk_group.h"

namespace si {

constexpr int kRowWaveThreads = 256;

// A wave's keys travel HBM -> LDS -> operand registers through two 8 KiB blocks (D = 128) of its own, so
// there is no barrier: whole key rows per load (read straight into the operand layout, a row would be
// fetched in 32-byte pieces by eight loads, and the 32 KB L1 does not hold the blocks of 8 waves from the
// first to the last: 60 us instead of 42 at 32 x 2 rows of 16411 keys, 64 heads of 128).  Two workgroups
// per compute unit fit the LDS; their 8 waves keep 64 KB in flight.  Measured: 128 x 1 rows of 65536 keys,
// 2.1 GB, 438 us = 4.9 TB/s (a large copy reaches 4.6); 1 row of 262144 keys, 67 MB, 14 us = 4.8 TB/s.
template <int D, int HB>
__global__ __launch_bounds__(kRowWaveThreads) __attribute__((amdgpu_waves_per_eu(2)))
void score_rows_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ K, const float* __restrict__ w,
                       int B, int S, int H, int T, int n_cols, int m, int mask_mode, int queries, int blocks_per_wave,
                       int n_slabs, float* __restrict__ scores, float* __restrict__ maxima, int group_lg,
                       unsigned long long* __restrict__ counters, int n_counters) {
#if defined(__HIP_DEVICE_COMPILE__)
    constexpr int KS = D / 16;
    constexpr int kRowBytes = D * 2;
    constexpr int kBlockBytes = 32 * kRowBytes;
    constexpr int kLoads = kBlockBytes / 1024;
    constexpr int kRowBuffers = 2;  // one block multiplied, one on its way
    __shared__ __attribute__((aligned(1024))) unsigned char lds_all[4 * kRowBuffers * kBlockBytes];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int col = lane & 31;
    const int half = lane >> 5;
    // the selection's counters are cleared here: it runs after this kernel
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_counters; i += kRowWaveThreads) counters[i] = 0ull;

    // Workgroup -> (batch, key slab, query group): the workgroups that read the same keys are 8 apart,
    // that is on the same XCD, so that its L2 fetches the keys once.
    const int n_groups = (S + queries - 1) / queries;
    const int xcd = blockIdx.x & 7, rest = blockIdx.x >> 3;
    const int slab_of_all = (rest / n_groups) * 8 + xcd;  // b * n_slabs + slab
    const int group = rest % n_groups;
    if (slab_of_all >= B * n_slabs) return;  // (fewer than 8 past the end)
    const int b = slab_of_all / n_slabs;
    const int per_group = 4 / queries;  // waves of the workgroup that share a query
    const int t = group * queries + wave % queries;
    if (t >= S) return;
    const int slab = (slab_of_all % n_slabs) * per_group + wave / queries;
    const int n_keys = min(n_cols, legal_count(t, T, m, mask_mode));
    int key0 = slab * blocks_per_wave * 32;
    if (key0 >= n_keys) return;
    const int key_end = min(n_keys, key0 + blocks_per_wave * 32);
    const int64_t row = static_cast<int64_t>(b) * S + t;
    const __bf16* Kb = K + static_cast<int64_t>(b) * T * D;

    typedef __attribute__((address_space(3))) void lds_void;
    unsigned char* lds = lds_all + wave * (kRowBuffers * kBlockBytes);
    // keys [KEY0, KEY0 + 32) to buffer BUF; key rows past the last one land as zero
#define SI_FETCH(KEY0, BUF)                                                                                  \
    {                                                                                                         \
        const __amdgpu_buffer_rsrc_t rsrc_ = chunk_rsrc<D>(Kb, T, (KEY0));                                    \
        _Pragma("unroll") for (int i = 0; i < kLoads; ++i)                                                    \
            __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc_, (lds_void*)(lds + (BUF) * kBlockBytes + i * 1024), \
                                                     16, chunk_lane_offset<D>(i, lane), 0, 0, 0);             \
    }
    SI_FETCH(key0, 0)
    bf16x8 a[HB][KS];
    float wr[HB][16];
    load_query<D, HB>(q, w, row, H, lane, a, wr);
    const int swz = (col / (256 / kRowBytes)) % (D / 8);
    int kaddr[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kaddr[ks] = col * kRowBytes + (((ks * 2 + half) ^ swz) * 16);
    float* out = scores + row * n_cols;
    const int64_t n_max = (static_cast<int64_t>(n_cols) + (1 << group_lg) - 1) >> group_lg;
    const floatx16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int buf = 0; key0 < key_end; key0 += 32, buf ^= 1) {
        // The other buffer's readers are done (its operands are in registers), so the next block starts
        // its trip; then everything but that block must have landed.
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        SI_FETCH(key0 + 32, buf ^ 1)
        __builtin_amdgcn_s_waitcnt(0x0F70 | kLoads);
        asm volatile("" ::: "memory");
        bf16x8 kc[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) kc[ks] = *reinterpret_cast<const bf16x8*>(lds + buf * kBlockBytes + kaddr[ks]);
        floatx16 acc[HB];
#pragma unroll
        for (int hb = 0; hb < HB; ++hb)
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                acc[hb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[hb][ks], kc[ks], ks == 0 ? zero16 : acc[hb], 0, 0, 0);
        float s = 0.0f;
#pragma unroll
        for (int e = 0; e < 16 * HB; ++e) s = fmaf(wr[e / 16][e % 16], relu(acc[e / 16][e % 16]), s);
        s = both_halves<8>(s);
        const bool live = key0 + col < key_end;
        if (half == 0 && live) out[key0 + col] = s;
        if (maxima != nullptr) {  // of 8 or 32 consecutive keys; NaN counts as nothing, like -inf
            float g = live ? fmaxf(s, -__builtin_huge_valf()) : -__builtin_huge_valf();
            g = fmaxf(g, __shfl_xor(g, 1));
            g = fmaxf(g, __shfl_xor(g, 2));
            g = fmaxf(g, __shfl_xor(g, 4));
            if (group_lg == 5) {
                g = fmaxf(g, __shfl_xor(g, 8));
                g = fmaxf(g, __shfl_xor(g, 16));
            }
            if (half == 0 && live && (col & ((1 << group_lg) - 1)) == 0) maxima[row * n_max + ((key0 + col) >> group_lg)] = g;
        }
    }
#undef SI_FETCH
    __builtin_amdgcn_s_waitcnt(0x0F70);  // the block past the end has landed too
#else
    (void)q; (void)K; (void)w; (void)B; (void)S; (void)H; (void)T; (void)n_cols; (void)m; (void)mask_mode; (void)queries;
    (void)blocks_per_wave; (void)n_slabs; (void)scores; (void)maxima; (void)group_lg; (void)counters; (void)n_counters;
#endif
}

// Maxima of groups of 32 << lg entries of score rows, the caller's or the dense schedule's (entries 64 apart, so that every load
// of a wave is one run of 64; any split into groups gives a bound): group 64 c + l of a row is entries
// (2048 << lg) c + l + 64 i.  Entries past the legal count do not count.  A wave takes 32 entries a group, all on their way before
// the first is used; a workgroup's waves are SHARE to 64 groups, each 2048 entries apart (one wave alone for 64 groups of 1024:
// 14 x 76484 scores, k = 36, whole selection 46 us, here 14).
template <int SHARE>
__global__ __launch_bounds__(SHARE == 1 ? 256 : 64 * SHARE) void row_maxima_kernel(
    const float* __restrict__ scores, int R, int n_cols, const int32_t* __restrict__ legal_rows, int S, int m, int mask_mode, int chunks,
    int lg, float* __restrict__ maxima, unsigned long long* __restrict__ counters, int n_counters) {
    constexpr int kWaves = SHARE == 1 ? 4 : SHARE;
    __shared__ float s_part[SHARE == 1 ? 1 : SHARE][64];
    if (blockIdx.x == 0)
        for (int i = threadIdx.x; i < n_counters; i += 64 * kWaves) counters[i] = 0ull;
    const int wave = threadIdx.x >> 6;
    const int64_t task = SHARE == 1 ? static_cast<int64_t>(blockIdx.x) * kWaves + wave : static_cast<int64_t>(blockIdx.x);
    const int lane = threadIdx.x & 63;
    const int row = static_cast<int>(task / chunks), c = static_cast<int>(task % chunks);
    if (row >= R) return;  // (with SHARE > 1 there are no more workgroups than tasks)
    const int n = legal_rows != nullptr ? min(legal_rows[row], n_cols) : legal_count(row % S, n_cols, m, mask_mode);
    const float* sc = scores + static_cast<int64_t>(row) * n_cols;
    float g = -__builtin_huge_valf();
    for (int part = SHARE == 1 ? 0 : wave; part < (1 << lg); part += SHARE) {
        const int64_t from = ((static_cast<int64_t>(c) << lg) + part) * 2048;
        const float* const first = sc + from + lane;
        const int left = static_cast<int>(max(int64_t{0}, min(static_cast<int64_t>(n) - from, int64_t{2048}))) - lane;
        float v[32];
#pragma unroll
        for (int i = 0; i < 32; ++i) v[i] = i * 64 < left ? first[i * 64] : -__builtin_huge_valf();
#pragma unroll
        for (int i = 0; i < 32; ++i) g = fmaxf(g, v[i]);
    }
    if constexpr (SHARE > 1) {
        s_part[wave][lane] = g;
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int i = 1; i < SHARE; ++i) g = fmaxf(g, s_part[i][lane]);
    }
    maxima[(static_cast<int64_t>(row) * chunks + c) * 64 + lane] = g;
}

template <int THREADS>
__device__ __forceinline__ void write_row(const key64_t* keys, int c, int k, int64_t row, int32_t* out_idx,
                                          float* out_score) {
    const list_rank_t* const ranks = reinterpret_cast<const list_rank_t*>(keys);  // GroupList::finish has been there
    const int64_t out = row * k;
    for (int j = threadIdx.x; j < k; j += THREADS) {
        if (j < c) {
            const rank_t key = ranks[j];
            out_idx[out + j] = rank_index(key);
            out_score[out + j] = rank_score(key);
        } else {  // Section 4.2: pad
            out_idx[out + j] = -1;
            out_score[out + j] = -__builtin_huge_valf();
        }
    }
}

// Rows of at most THREADS * VPT scores and the best min(k, n_cols) <= KCAP of each: the whole row in
// registers, group_rank_select, one workgroup per row (rows and arguments as for select_rows_kernel).  Where the
// bins do not separate the scores, group_exact_select in the same LDS.  Bound by the chains of a row's
// dependent LDS steps; few threads per row keep the steps without barriers and many rows in flight.  One wave per row
// against the list with 256 threads (us, list -> here): 16384 rows of 256 scores, k = 64 110 -> 25; 1024, k = 512 133 ->
// 47; 2047, k = 300 151 -> 65; two waves: 4096 rows of 4096, k = 1024 41.  512 threads: 4096 rows of 8192, k = 4096 235 ->
// 93; 16384, k = 2048 300 -> 122.  With integer compares in the sorts and a test per bin the same took 44, 63, 83, 48, 118 and 149.  Counting only the entries above a guess of the k-th best (from mean and
// deviation) changed nothing: the atomics are not what a row waits for.  Rows half of which are equal scores (us, cutting
// an LDS list -> group_exact_select): 16384 of 1024, k = 512 434 -> 126; 2000 of 2048, k = 1024 199 -> 58;
// 4096 of 4096, k = 1024 326 -> 89; 1024 of 16384, k = 4096 413 -> 100.  A fifth wave per SIMD of the one-wave form
// fits only some SIMDs of a compute unit and costs 5 % (16384 rows of 1024, k = 512: 62 -> 67): four at most.
template <int THREADS, int VPT, int KCAP, int BINS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(THREADS == 64 ? (KCAP == 512 ? 4 : 3) : VPT == 16 ? 6 : 4, THREADS == 64 ? 4 : 8)))
void select_short_rows_kernel(const float* __restrict__ scores, int n_cols, const int32_t* __restrict__ legal_rows,
                              RowTile tile, int m, int mask_mode, int k, int32_t* __restrict__ out_idx,
                              float* __restrict__ out_score) {
    constexpr int kSlots = KCAP + kWaveRankMaxBin + (KCAP + kWaveRankMaxBin) / 8;  // sort_slots
    static_assert((KCAP & (KCAP - 1)) == 0, "the network sorts in place");
    __shared__ __attribute__((aligned(16))) rank_t s_keys[kSlots];
    __shared__ __attribute__((aligned(16))) union {
        RankScratch<THREADS, BINS> rank;
        GroupScratch<THREADS, 1> exact;
    } s;
    const int row = static_cast<int>(blockIdx.x);
    const int t = tile.s0 + row % tile.rows;
    int n = legal_rows != nullptr ? min(legal_rows[row], n_cols) : legal_count(t, n_cols, m, mask_mode);
    n = __builtin_amdgcn_readfirstlane(n);
    const float* sc = scores + static_cast<int64_t>(row) * n_cols;
    const int left = n - static_cast<int>(threadIdx.x);
    float v[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) v[i] = i * THREADS < left ? sc[threadIdx.x + i * THREADS] : -__builtin_huge_valf();
    float some = n > 0 ? sc[0] : 0.0f;
    if (!(some - some == 0.0f)) some = 0.0f;
#pragma unroll
    for (int i = 0; i < VPT; ++i)
        v[i] = v[i] > -__builtin_huge_valf() ? v[i] : -__builtin_huge_valf();  // (NaN: none)
    const int kk = min(k, n_cols);  // <= KCAP
    const int64_t out = (static_cast<int64_t>(row / tile.rows) * tile.S + t) * k;
    int c = 0;
    const bool ranked = group_rank_select<THREADS, VPT, BINS>(v, n, some, kk, s_keys, s.rank, &c);
    if (!ranked) {
        __syncthreads();  // the scratch changes hands
        c = group_exact_select<THREADS>(v, kk, s_keys, s.exact);
    }
    const SortSlot slot;
    for (int j = threadIdx.x; j < k; j += THREADS) {
        if (j < c) {
            const rank_t key = s_keys[slot(j)];
            out_idx[out + j] = rank_index(key);
            out_score[out + j] = rank_score(key);
        } else {  // Section 4.2: pad
            out_idx[out + j] = -1;
            out_score[out + j] = -__builtin_huge_valf();
        }
    }
}

// Bound by the vector instructions (some 15 per 64 scores) and the chains of dependent LDS steps of a workgroup's phases; what
// hides the latter is several workgroups per compute unit: 512 threads, three of them (80 registers).  Measured (us): 2048 rows
// of 32771 scores, k = 512 60 = 4.5 TB/s; with rows of 5/8 that length 59; 700 rows 30; 1024 threads and two per unit were
// half as fast.  Scores as ordered images from the start, a ballot and a rank for every 64 and generic loads with an
// address pair each (which the allocator took 102 registers for, or spilled): 87, 69 and 43.
// Row r of scores [R, n_cols] has legal_rows[r] legal entries, or where legal_rows is null those of query
// position tile.s0 + r mod tile.rows; its result is row (r / tile.rows) * tile.S + that position of the
// outputs.  One workgroup per row.
template <int THREADS, int CAP, int OCC>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(OCC)))
void select_rows_kernel(const float* __restrict__ scores, int n_cols,
                                                              const int32_t* __restrict__ legal_rows, RowTile tile,
                                                              int m, int mask_mode, int k,
                                                              int32_t* __restrict__ out_idx,
                                                              float* __restrict__ out_score) {
    __shared__ __attribute__((aligned(16))) key64_t s_keys[CAP];
    __shared__ GroupScratch<THREADS> s;
    const int row = static_cast<int>(blockIdx.x);
    const int t = tile.s0 + row % tile.rows;
    int n = legal_rows != nullptr ? min(legal_rows[row], n_cols) : legal_count(t, n_cols, m, mask_mode);
    n = __builtin_amdgcn_readfirstlane(n);
    GroupList<THREADS, CAP> list;
    list.init(s_keys, &s);
    const float* sc = scores + static_cast<int64_t>(row) * n_cols;
    list.stream(sc, n, k);
    list.finish(k);
    write_row<THREADS>(s_keys, list.count, k, static_cast<int64_t>(row / tile.rows) * tile.S + t, out_idx, out_score);
}

// Raises the list's floor by n_mx group maxima, folded to N per thread: eight times k of them or more, so that little more than k
// keys pass, but no more than that takes, for every value costs the workgroup's waves an instruction in each pass.
template <int N, int THREADS, typename List>
__device__ __forceinline__ bool bound_by_maxima(List& list, const float* mx, int n_mx, int k) {
    float most[N];
#pragma unroll
    for (int i = 0; i < N; ++i) most[i] = -__builtin_huge_valf();
    for (int64_t j0 = 0; j0 < n_mx; j0 += THREADS * N) {
        const int left = static_cast<int>(min(n_mx - j0, int64_t{THREADS * N})) - static_cast<int>(threadIdx.x);
        float v[N];
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = i * THREADS < left ? mx[j0 + threadIdx.x + i * THREADS] : -__builtin_huge_valf();
#pragma unroll
        for (int i = 0; i < N; ++i) most[i] = fmaxf(most[i], v[i]);
    }
    uint32_t g[N];
#pragma unroll
    for (int i = 0; i < N; ++i) g[i] = candidate(most[i]);
    return list.bound_by(g, k);
}

// Several workgroups per row: workgroup r * n_parts + p sends the keys of entries [p, p + 1) * part_len of row
// r that are above the row's bound to lists[r][0 .. list_cap), list_cap <= CAP; the low half of held[r] counts them, the high half
// the parts that are done (zero before the launch; one word, so that the last arrival learns the count by the way).  The last part sorts the list; if it overflowed
// (many equal or oddly spread scores), that workgroup goes through the whole row by itself.
// 1024 threads: with few workgroups only the length of the chain counts (one row of 262144, k = 1024; 10 ns ticks of the wall
// clock: loads 180, bound 240, filter 200, arrival and list 120, sort 330, write 30; 512 threads 0.7 to 2 us more, for 16 rows and
// more the same).  What made it 16.5 us: a wait behind each of the eight loads of maxima and of the scores, and passes over 16
// values a thread of which 2 to 8 existed.
// The exchange between workgroups uses device-scope loads and stores (which pass the XCDs' own L2s) and a
// wait for the stores before the arrival is counted, instead of a fence, which
// writes back the whole L2 (5 to 10 us measured).
template <int THREADS, int CAP, bool FROM_SCORES>
__global__ __launch_bounds__(THREADS) void select_parts_kernel(
    const float* __restrict__ scores, int n_cols, const int32_t* __restrict__ legal_rows, int S, int m,
    int mask_mode, int k, int n_parts, int part_len, const float* __restrict__ maxima, int n_maxima, int group_lg, int list_cap, key64_t* lists,
    unsigned long long* held, int32_t* __restrict__ out_idx, float* __restrict__ out_score) {
    __shared__ __attribute__((aligned(16))) key64_t s_keys[CAP];
    __shared__ GroupScratch<THREADS> s;
    const int row = static_cast<int>(blockIdx.x) / n_parts;
    const int part = static_cast<int>(blockIdx.x) % n_parts;
    int n = legal_rows != nullptr ? min(legal_rows[row], n_cols) : legal_count(row % S, n_cols, m, mask_mode);
    n = __builtin_amdgcn_readfirstlane(n);
    GroupList<THREADS, CAP> list;
    list.init(s_keys, &s);
    const float* sc = scores + static_cast<int64_t>(row) * n_cols;
    key64_t* const row_list = lists + static_cast<int64_t>(row) * list_cap;
    unsigned long long* const row_held = held + row;

    // The part's first chunk and the row's maxima (as many as a thread has values) are requested together, before anything is
    // used: a load that is waited for at once costs a trip of its own (one row of 262144, k = 1024: 2 us).
    const int64_t beg = static_cast<int64_t>(part) * part_len, end = min(static_cast<int64_t>(n), beg + part_len);
    float f[kSelectValues];
    const auto load_chunk = [&](int64_t c0) {
        const int left = static_cast<int>(max(end - c0, int64_t{0})) - static_cast<int>(threadIdx.x);
        const float* const chunk = sc + c0;
#pragma unroll
        for (int i = 0; i < kSelectValues; ++i)
            f[i] = i * THREADS < left ? chunk[threadIdx.x + i * THREADS] : -__builtin_huge_valf();
    };
    // The row's first workgroup takes it alone where sharing it gains nothing: a caller's row of which one chunk counts, and one with
    // fewer groups than a bound takes, all of whose entries would be sent (us, 1 row, k = 89, of 89027 scores 22000 count: 19 -> 13).
    // Only with maxima from row_maxima_kernel (FROM_SCORES): decoding, whose rows are never so, takes 0.1 to 0.3 us longer with the tests.
    bool alone = FROM_SCORES && legal_rows != nullptr && n <= THREADS * kSelectValues, equals = false;
    if (!alone) {  // the row's bound; the groups are folded to at most kSelectValues per thread
        load_chunk(beg);
        const float* mx = maxima + static_cast<int64_t>(row) * n_maxima;
        // groups of 2^group_lg consecutive entries past the legal ones were not written; of the others all were
        const int n_mx = FROM_SCORES ? n_maxima : min(n_maxima, (n + (1 << group_lg) - 1) >> group_lg);
        if (kPartsMaxima(k) == 4) equals = bound_by_maxima<4, THREADS>(list, mx, n_mx, k);
        else equals = bound_by_maxima<8, THREADS>(list, mx, n_mx, k);
        if constexpr (FROM_SCORES) alone = list.floor == -__builtin_huge_valf() && n > list_cap;
    }
    if constexpr (FROM_SCORES) alone = __builtin_amdgcn_readfirstlane(alone ? 1 : 0) != 0;
    if (alone && part != 0) return;
    if (!alone) {
        for (int64_t c0 = beg; c0 < end; c0 += THREADS * kSelectValues) {
            const int first = static_cast<int>(c0) + static_cast<int>(threadIdx.x);
            const int live = static_cast<int>((end - c0 + THREADS - 1) / THREADS);
            if (c0 > beg) load_chunk(c0);
            int before = 0;
            const int total = list.above(f, live, &before);
            if (total == 0) continue;  // uniform
            if (threadIdx.x == 0)
                s.flag = static_cast<int>(__hip_atomic_fetch_add(row_held, static_cast<unsigned long long>(total), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
            __syncthreads();
            list.each_above(f, live, s.flag + before, first, [&](int p, key64_t key) {
                if (p < list_cap) __hip_atomic_store(&row_list[p], key, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            });
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this thread's keys have arrived
        __syncthreads();
        if (threadIdx.x == 0) {
            const unsigned long long before = __hip_atomic_fetch_add(row_held, 1ull << 32, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s.flag = static_cast<int>(before >> 32) == n_parts - 1 ? static_cast<int>(before) : -1;  // all keys have been counted
        }
        __syncthreads();
        const int total = __builtin_amdgcn_readfirstlane(s.flag);
        if (total < 0) return;  // uniform: another workgroup of this row arrives later
        if (total <= list_cap) {
            for (int j = threadIdx.x; j < total; j += THREADS)
                s_keys[j] = __hip_atomic_load(&row_list[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            list.count = total;
        } else if (equals && total > CAP && list.floor > -__builtin_huge_valf() && list.finish_with_equals(sc, n, k)) {
            // Equal scores at the bound get a pass of their own: rows whose best are all 0, 50 x 49152, k = 300 57 -> 22 us (one
            // workgroup for each row from the start: 48), 1 x 262144, k = 1024 92 -> 50; distinct scores as before.  Only
            // where the list in LDS would overflow as well: where it does not, the plain pass is the shorter one.
            write_row<THREADS>(s_keys, list.count, k, row, out_idx, out_score);
            return;
        } else {
            alone = true;
        }
    }
    if (alone) list.stream(sc, n, k);
    list.finish(k);
    write_row<THREADS>(s_keys, list.count, k, row, out_idx, out_score);
}

hipError_t launch_score_rows(const void* q, const void* K, const float* w, const si_dims& d, int32_t m,
                             int32_t mask_mode, int32_t n_cols, const RowSelection& sel, float* scores, hipStream_t stream) {
    // a workgroup's four waves: four queries, or two queries times two slabs of keys, or one times four
    const int queries = d.S >= 3 ? 4 : d.S;
    const int n_groups = (d.S + queries - 1) / queries;
    const int64_t key_blocks = (static_cast<int64_t>(n_cols) + 31) / 32;
    // one round of the chip's 2048 resident waves where 24 blocks per wave are enough for it, else 16 (32 x 2 rows of 16411 keys:
    // 17 in one round, 16 leave 32 workgroups for a second one)
    const int64_t total = key_blocks * d.B * n_groups * queries;
    const int64_t one_round = std::max<int64_t>(1, (total + 2047) / 2048);
    const int per_wave = static_cast<int>(one_round <= 24 ? one_round : 16);
    const int64_t per_group = static_cast<int64_t>(per_wave) * (4 / queries);
    const int64_t n_slabs = (key_blocks + per_group - 1) / per_group;
    const int64_t grid = (n_slabs * d.B + 7) / 8 * 8 * n_groups;
    if (grid >= (int64_t{1} << 31)) return hipErrorInvalidValue;
    const __bf16* qp = static_cast<const __bf16*>(q);
    const __bf16* Kp = static_cast<const __bf16*>(K);
    const int HB = (d.H_I + 31) / 32;
#define SI_LAUNCH(DD, HH)                                                                                        \
    hipLaunchKernelGGL((score_rows_kernel<DD, HH>), dim3(static_cast<unsigned>(grid)), dim3(kRowWaveThreads), 0, \
                       stream, qp, Kp, w, d.B, d.S, d.H_I, d.T, n_cols, m, mask_mode, queries, per_wave,                 \
                       static_cast<int>(n_slabs), scores, sel.maxima, sel.group_lg, sel.held, sel.n_parts > 1 ? d.B * d.S : 0)
    if (d.D == 128 && HB == 2) SI_LAUNCH(128, 2);
    else if (d.D == 128 && HB == 1) SI_LAUNCH(128, 1);
    else if (d.D == 64 && HB == 2) SI_LAUNCH(64, 2);
    else if (d.D == 64 && HB == 1) SI_LAUNCH(64, 1);
    else if (d.D == 32 && HB == 2) SI_LAUNCH(32, 2);
    else if (d.D == 32 && HB == 1) SI_LAUNCH(32, 1);
    else return hipErrorInvalidValue;
#undef SI_LAUNCH
    return hipGetLastError();
}

hipError_t launch_row_maxima(const float* scores, int32_t R, int32_t n_cols, const int32_t* legal_rows, int32_t S,
                             int32_t m, int32_t mask_mode, const RowSelection& sel, hipStream_t stream) {
    const int64_t per_chunk = int64_t{2048} << sel.maxima_lg;
    const int chunks = static_cast<int>((n_cols + per_chunk - 1) / per_chunk);
    if (sel.n_maxima != chunks * 64 || sel.maxima_lg < 0 || sel.maxima_lg > 5) return hipErrorInvalidValue;
    const int64_t tasks = static_cast<int64_t>(R) * chunks;
#define SI_LAUNCH(SHARE)                                                                                                   \
    hipLaunchKernelGGL((row_maxima_kernel<SHARE>), dim3(static_cast<unsigned>(SHARE == 1 ? (tasks + 3) / 4 : tasks)),      \
                       dim3(SHARE == 1 ? 256 : 64 * SHARE), 0, stream, scores, R, n_cols, legal_rows, S, m, mask_mode,    \
                       chunks, sel.maxima_lg, sel.maxima, sel.held, R)
    if (sel.maxima_lg == 0) SI_LAUNCH(1);
    else if (sel.maxima_lg == 1) SI_LAUNCH(2);
    else if (sel.maxima_lg == 2) SI_LAUNCH(4);
    else if (sel.maxima_lg == 3) SI_LAUNCH(8);
    else SI_LAUNCH(16);
#undef SI_LAUNCH
    return hipGetLastError();
}

hipError_t launch_select_rows(const float* scores, int32_t R, int32_t n_cols, const int32_t* legal_rows,
                              const RowTile& tile, int32_t m, int32_t mask_mode, int32_t k, const RowSelection& sel,
                              int32_t* out_idx, float* out_score, hipStream_t stream) {
    if (k < 1 || k > kMaxK) return hipErrorInvalidValue;
    // a list holds at least k + one key per thread (GroupList::stream) and the sorted 2^ceil(log2 k)
    static_assert(kRowListCap(1024) == 4096 && kRowListCap(2049) == 8192, "the launches below");
    if (sel.n_parts > 1) {
        if (tile.s0 != 0 || tile.rows != tile.S) return hipErrorInvalidValue;  // whole problems only
        if (static_cast<int64_t>(sel.n_parts) * sel.part_len < n_cols || !sel.maxima || !sel.lists || !sel.held ||
            sel.list_cap < k || sel.list_cap > kRowListCap(k))
            return hipErrorInvalidValue;
        const dim3 grid(static_cast<unsigned>(R * sel.n_parts));
#define SI_LAUNCH(CC, FF)                                                                                         \
    hipLaunchKernelGGL((select_parts_kernel<kPartsThreads, CC, FF>), grid, dim3(kPartsThreads), 0, stream, scores, n_cols, legal_rows, tile.S, m, \
                       mask_mode, k, sel.n_parts, sel.part_len, sel.maxima, sel.n_maxima, sel.group_lg, sel.list_cap, sel.lists, sel.held, out_idx, \
                       out_score)
        if (sel.group_lg == 0) {
            if (k <= 2048) SI_LAUNCH(4096, true); else SI_LAUNCH(8192, true);
        } else {
            if (k <= 2048) SI_LAUNCH(4096, false); else SI_LAUNCH(8192, false);
        }
#undef SI_LAUNCH
        return hipGetLastError();
    }
    // At most 2^22 rows per launch (a launch has fewer than 2^32 threads); only rows that stand for
    // themselves, not for positions of a batch, can be that many.
    constexpr int32_t kRowsPerLaunch = 1 << 22;
    if (R > kRowsPerLaunch && tile.S != 1) return hipErrorInvalidValue;
    for (int64_t r0 = 0; r0 < R; r0 += kRowsPerLaunch) {
        const dim3 grid(static_cast<unsigned>(std::min<int64_t>(kRowsPerLaunch, R - r0)));
        const float* sc = scores + r0 * n_cols;
        const int32_t* lg = legal_rows ? legal_rows + r0 : nullptr;
#define SI_LAUNCH(TT, CC, OO)                                                                                      \
    hipLaunchKernelGGL((select_rows_kernel<TT, CC, OO>), grid, dim3(TT), 0, stream, sc, n_cols, lg, tile, m, mask_mode, \
                       k, out_idx + r0 * k, out_score + r0 * k)
#define SI_SHORT(TT, VV, CC, BB)                                                                                       \
    hipLaunchKernelGGL((select_short_rows_kernel<TT, VV, CC, BB>), grid, dim3(TT), 0, stream, sc, n_cols, lg, tile, m, \
                       mask_mode, k, out_idx + r0 * k, out_score + r0 * k)
        // In registers, by one wave (two beyond 2048 scores) where there are enough rows to fill the chip that
        // way (1024 scores, k = 512: 1800 rows 21.3 -> 16.1 us, but 1024 rows 12.3 -> 15.0), or no blocks to sort one
        // after the other (k <= 16: 1024 rows of 256 10.5 -> 8.9).  By 512 threads for long lists, which the LDS list
        // holds once or twice only (1024 rows of 8192: k = 2048 37 -> 31, k = 512 24 -> 26).  Else the list: for few
        // short rows its 256 threads are the shorter chain, for k up to 1024 of many scores its bound
        // leaves fewer keys to count.
        const int32_t kk = std::min(k, n_cols);
        const bool many = grid.x >= 1792;
        if (n_cols <= 512 && (many || kk <= 16)) SI_SHORT(64, 8, 512, 1024);
        else if (many && n_cols <= 1024 && kk <= 512) SI_SHORT(64, 16, 512, 2048);
        else if (many && n_cols <= 1024) SI_SHORT(64, 16, 1024, 2048);
        else if (many && n_cols <= 2048 && kk <= 512) SI_SHORT(64, 32, 512, 2048);
        else if (many && n_cols <= 2048 && kk <= 1024) SI_SHORT(64, 32, 1024, 2048);
        else if (many && n_cols <= 4096 && kk <= 1024) SI_SHORT(128, 32, 1024, 2048);
        else if (n_cols <= 4096 && kk <= 1024) SI_LAUNCH(256, 2048, 5);
        else if (n_cols <= 8192 && kk > 1024 && kk <= 2048) SI_SHORT(512, 16, 2048, 4096);
        else if (n_cols <= 16384 && kk > 1024) SI_SHORT(512, 32, 4096, 8192);
        else if (kk <= 2048) SI_LAUNCH(512, 4096, 6);
        else SI_LAUNCH(512, 8192, 4);
#undef SI_SHORT
#undef SI_LAUNCH
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace si
