// Workgroup-level selection: the best k of a stream of 64-bit (score, ~index) keys, kept in LDS by
// all waves of one workgroup.  Used where a row is too long, or the rows too few, for the wave-level
// routines of topk_wave.h to fill the chip: what counts here is the length of the chain of dependent
// steps, not the number of instructions.
//
// The list invariant is that of the row buffers: it holds the k best keys of the prefix visited so
// far plus every later key above `floor`, a lower bound of the k-th best.  What makes one pass over
// the data enough in the usual case is where the first bound comes from: the elements are split into
// M >= 2k groups of equal size, and the k-th largest of the M group maxima is a lower bound of the
// k-th largest element (k groups reach it).  With M = 2k and iid scores about 1.4 k elements pass it,
// with M = 8k about 1.07 k, for one maximum per element and a radix step over M values, where a
// histogram over all elements would cost an LDS atomic each.  Scores in an unfavourable order only
// cost time: a chunk that does not fit is cut against its own bound, and if it still does not fit it
// is taken in steps of one element per thread with a cut whenever the list is full.
#pragma once

#include "topk_wave.h"
#include "wave_ops.h"

namespace si {

constexpr int kRankBins = 2048;
constexpr int kRankMaxBin = 64;  // fuller bins than this: the bitonic network is the better sort

// (BINS = 1 where group_rank_sort is not called)
template <int THREADS, int BINS = kRankBins>
struct GroupScratch {
    static constexpr int kWavesPerGroup = THREADS / 64;
    union {
        int hist[3][256];
        int bins[BINS];
    };
    uint32_t low[kWavesPerGroup], high[kWavesPerGroup];
    float lo[kWavesPerGroup], hi[kWavesPerGroup], sum[kWavesPerGroup];
    int wave_sum[kWavesPerGroup], wave_most[kWavesPerGroup];
    int flag;
};

// A group of 64 threads is one wave of its workgroup, and the only one that uses the scratch it is given: LDS accesses of a
// wave are executed in order, so that its barrier only holds the compiler back.
template <int THREADS>
__device__ __forceinline__ int group_thread() { return static_cast<int>(THREADS == 64 ? threadIdx.x & 63 : threadIdx.x); }
template <int THREADS>
__device__ __forceinline__ int group_wave() { return THREADS == 64 ? 0 : static_cast<int>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)); }
template <int THREADS>
__device__ __forceinline__ void group_barrier() {
    if constexpr (THREADS == 64) {
        asm volatile("" ::: "memory");
        __builtin_amdgcn_wave_barrier();
        asm volatile("" ::: "memory");
    } else {
        __syncthreads();
    }
}

// Sum over the workgroup of a wave-uniform value; *before = sum over the waves below this one.
template <int THREADS, int BINS>
__device__ inline int group_sum(int wave_value, int* before, GroupScratch<THREADS, BINS>& s) {
    constexpr int W = THREADS / 64;
    const int wave = group_wave<THREADS>();
    const int lane = threadIdx.x & 63;
    group_barrier<THREADS>();  // earlier readers of wave_sum are done
    if (lane == 0) s.wave_sum[wave] = wave_value;
    group_barrier<THREADS>();
    const int incl = wave_prefix_sum(lane < W ? s.wave_sum[lane] : 0);
    *before = wave == 0 ? 0 : lane_value(incl, wave - 1);
    return lane_value(incl, W - 1);
}

// A lower bound of the k-th largest of the workgroup's values (N per thread, 0 = none; more than k are
// present): returns `thr` such that exactly *above + *bin values are >= thr, *above of them above the last
// window, with k <= *above + *bin, and <= limit unless thr is itself the k-th largest value (and *bin its
// multiplicity).  Histogram descent, up to 8 bits per pass, on the distance from the smallest value: the
// values are the upper tail of a distribution, close together but often on both sides of a power of
// two, where a descent by common prefix would spend its first pass on a few exponent codes.  With NARROW a
// bin of more than kCrowdedBin values is narrowed to its own range before the next pass: equal values end the
// descent at once, where every further pass would have them queue for one histogram word (the lists do without:
// its registers cost select_rows_kernel 20 %).  One barrier per pass: the three histograms take turns, and the one that a pass clears was last read two
// barriers ago.
constexpr int kCrowdedBin = 128;
template <int THREADS, bool NARROW = false, int N, int BINS>
__device__ inline uint32_t group_kth(const uint32_t (&x)[N], int k, int limit, GroupScratch<THREADS, BINS>& s,
                                     int* above, int* bin) {
    constexpr int W = THREADS / 64;
    const int lane = threadIdx.x & 63;
    const int wave = group_wave<THREADS>();
    uint32_t lo = 0xFFFFFFFFu, hi = 0u;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        lo = min(lo, x[i] - 1u);  // 0 wraps to the top
        hi = max(hi, x[i]);
    }
    lo = wave_min(lo);
    hi = wave_max(hi);
    group_barrier<THREADS>();  // earlier readers of the scratch are done
    if (lane == 0) {
        s.low[wave] = lo;
        s.high[wave] = hi;
    }
    for (int i = group_thread<THREADS>(); i < 256; i += THREADS) s.hist[0][i] = 0;
    group_barrier<THREADS>();
    uint32_t base = wave_min(lane < W ? s.low[lane] : 0xFFFFFFFFu) + 1u;
    uint32_t range = wave_max(lane < W ? s.high[lane] : 0u) - base;  // undecided values: [base, base + range]
    int bits = range == 0u ? 0 : 32 - __builtin_clz(range);
    int need = k, in_bin = 0;
    for (int p = 0;; p = p == 2 ? 0 : p + 1) {
        const int shift = max(bits - 8, 0);
        const uint32_t bins = 1u << (bits - shift);
        int* hist = s.hist[p];
        int* next = s.hist[p == 2 ? 0 : p + 1];
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const uint32_t d = (x[i] - base) >> shift;
            if (x[i] >= base && (NARROW ? x[i] - base <= range : d < bins)) atomicAdd(&hist[d], 1);
        }
        for (int i = group_thread<THREADS>(); i < 256; i += THREADS) next[i] = 0;
        group_barrier<THREADS>();
        // every wave walks the bins by itself (lane l owns bins 255-4l .. 252-4l, from the top)
        int h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = hist[255 - 4 * lane - j];
        const int local = h[0] + h[1] + h[2] + h[3];
        const int incl = wave_prefix_sum(local);
        int cum = incl - local;
        const bool crossing = cum < need && need <= incl;
        int digit = 0, new_need = 0, new_bin = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (crossing && cum < need && need <= cum + h[j]) {
                digit = 255 - 4 * lane - j;
                new_need = need - cum;
                new_bin = h[j];
            }
            cum += h[j];
        }
        const int src = __builtin_ctzll(__ballot(crossing));
        digit = lane_value(digit, src);
        need = lane_value(new_need, src);
        in_bin = lane_value(new_bin, src);
        base += static_cast<uint32_t>(digit) << shift;
        bits = shift;
        if (k - need + in_bin <= limit || shift == 0) break;
        range = min(range - (static_cast<uint32_t>(digit) << shift), (1u << shift) - 1u);
        if (NARROW && in_bin > kCrowdedBin) {
            lo = 0xFFFFFFFFu;
            hi = 0u;
#pragma unroll
            for (int i = 0; i < N; ++i) {
                const bool in = x[i] >= base && x[i] - base <= range;
                lo = min(lo, in ? x[i] : 0xFFFFFFFFu);
                hi = max(hi, in ? x[i] : 0u);
            }
            lo = wave_min(lo);
            hi = wave_max(hi);
            if (lane == 0) {  // (the scratch was last read before the latest barrier)
                s.low[wave] = lo;
                s.high[wave] = hi;
            }
            group_barrier<THREADS>();
            base = wave_min(lane < W ? s.low[lane] : 0xFFFFFFFFu);
            range = wave_max(lane < W ? s.high[lane] : 0u) - base;
            if (range == 0u) break;
            bits = 32 - __builtin_clz(range);
        }
    }
    *above = k - need;
    *bin = in_bin;
    return base;
}

// The same contract as wave_radix_kth for a whole workgroup: a key `thr` with exactly *kept of the keys
// (N per thread, 0 = none) >= thr, k <= *kept <= max(k, limit); more than k keys must be present.
template <int THREADS, int N, int BINS>
__device__ inline key64_t group_radix_kth(const key64_t (&keys)[N], int k, int limit, GroupScratch<THREADS, BINS>& s,
                                          int* kept) {
    uint32_t x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = static_cast<uint32_t>(keys[i] >> 32);
    int above = 0, bin = 0;
    const uint32_t hi = group_kth<THREADS>(x, k, limit, s, &above, &bin);
    key64_t thr = static_cast<key64_t>(hi) << 32;
    if (above + bin > max(k, limit)) {  // equal scores: the index words decide
        const int need = k - above, over = limit - above;
#pragma unroll
        for (int i = 0; i < N; ++i) x[i] = x[i] == hi ? static_cast<uint32_t>(keys[i]) : 0u;
        int higher = 0;
        thr |= group_kth<THREADS>(x, need, over, s, &higher, &bin);
        above += higher;
    }
    *kept = above + bin;
    return thr;
}

// ---- sort -----------------------------------------------------------------------------------
// A slot of a list in LDS holds a key first and, once sorted, that key's rank: an access as a rank may alias one as a key.
typedef rank_t __attribute__((may_alias)) list_rank_t;
// Bitonic network over P keys (a power of two >= 4) in LDS by the whole workgroup, largest first; the
// four-keys-per-thread form of wave_sort_descending (two strides per LDS round trip).
template <int THREADS, int NB>
__device__ inline void group_sort_pass(list_rank_t* s, int P, int b, int size) {
    constexpr int E = 1 << NB;
    for (int u = threadIdx.x; u < (P >> NB); u += THREADS) {
        const int base = (u & ((1 << b) - 1)) | ((u >> b) << (b + NB));
        const uint32_t sign = (base & size) == 0 ? 0u : 0x80000000u;
        rank_t v[E];
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = flip(s[base | (j << b)], sign);
#pragma unroll
        for (int d = E >> 1; d > 0; d >>= 1)
#pragma unroll
            for (int i = 0; i < (E >> 1); ++i) {
                const int lo = 2 * i - (i & (d - 1));
                exchange(v[lo], v[lo + d]);
            }
#pragma unroll
        for (int j = 0; j < E; ++j) s[base | (j << b)] = flip(v[j], sign);
    }
    __syncthreads();
}
template <int THREADS>
__device__ inline void group_sort_descending(list_rank_t* s, int P) {
    for (int lg = 1; (1 << lg) <= P; ++lg) {
        for (int top = lg; top > 0;) {
            const int nb = (top & 1) ? 1 : 2;  // an odd stride first, then pairs
            top -= nb;
            if (nb == 2) group_sort_pass<THREADS, 2>(s, P, top, 1 << lg);
            else group_sort_pass<THREADS, 1>(s, P, top, 1 << lg);
        }
    }
}

// Turns list[0 .. c) into ranks, best first, by ranking: the keys are counted into bins of equal score width, laid
// out in bin order, and each key counts the better ones of its own bin (a few: the bins outnumber the
// keys that matter).  About a dozen dependent LDS steps, where the network has some 30 with a barrier
// each (sorting 1024 keys, 1024 threads: 24 k cycles measured for the network).  Bins only group keys;
// order comes from comparing whole keys, so the result is exact whatever the rounding of the bin number
// (which is monotone in the score).  The bins span [lowest, min(highest, lowest + 8 times the mean's
// distance from it)], so that a few far outliers, which share the first bin, do not squeeze the rest.
// Only the first k places are filled in.  Returns false, with the list as it was, where this does not
// apply: equal or infinite scores, or a bin with more than kRankMaxBin keys.
template <int THREADS, int CAP>
__device__ inline bool group_rank_sort(key64_t* list, int c, int k, GroupScratch<THREADS>& s) {
    constexpr int W = THREADS / 64, N = CAP / THREADS, BPT = kRankBins / THREADS;
    static_assert(kRankBins % THREADS == 0 && CAP % THREADS == 0, "even split over the threads");
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const float inf = __builtin_huge_valf();
    key64_t kb[N];
    float v[N];
    list_rank_t* const ranks = reinterpret_cast<list_rank_t*>(list);
    float lo = inf, hi = -inf, sum = 0.0f;  // sum of the distances from some key: no cancellation later
    __syncthreads();  // the list is complete, earlier readers of the scratch are done
    const float some = key_score(list[0]);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int j = static_cast<int>(threadIdx.x) + i * THREADS;
        kb[i] = j < c ? list[j] : 0ull;
    }
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i * THREADS < c) {  // (uniform, here and below: a list fills a third of its slots or less)
            v[i] = key_score(kb[i]);
            lo = fminf(lo, kb[i] != 0ull ? v[i] : inf);
            hi = fmaxf(hi, kb[i] != 0ull ? v[i] : -inf);
            sum += kb[i] != 0ull ? v[i] - some : 0.0f;
        }
    lo = wave_min(lo);
    hi = wave_max(hi);
    sum = wave_sum(sum);
    if (lane == 0) {
        s.lo[wave] = lo;
        s.hi[wave] = hi;
        s.sum[wave] = sum;
    }
#pragma unroll
    for (int i = 0; i < BPT; ++i) s.bins[threadIdx.x + i * THREADS] = 0;
    __syncthreads();
    lo = wave_min(lane < W ? s.lo[lane] : inf);
    hi = wave_max(lane < W ? s.hi[lane] : -inf);
    sum = wave_sum(lane < W ? s.sum[lane] : 0.0f);
    const float span = fminf(hi - lo, 8.0f * (sum / static_cast<float>(c) + (some - lo)));
    const float scale = static_cast<float>(kRankBins - 1) / span;
    if (!(span > 0.0f && scale < inf && scale > 0.0f)) return false;  // (uniform; also an infinite or NaN span)
    const float from = lo + span;
    int bin[N];
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i * THREADS < c) {
            bin[i] = static_cast<int>(rank_bin<kRankBins>(v[i], from, scale));
            if (kb[i] != 0ull) atomicAdd(&s.bins[bin[i]], 1);
        }
    __syncthreads();
    // counts -> first places
    int h[BPT], local = 0, most = 0;
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        h[i] = s.bins[threadIdx.x * BPT + i];
        local += h[i];
        most = max(most, h[i]);
    }
    const int incl = wave_prefix_sum(local);
    most = wave_max(most);
    if (lane == 63) {
        s.wave_sum[wave] = incl;
        s.wave_most[wave] = most;
    }
    __syncthreads();
    most = wave_max(lane < W ? s.wave_most[lane] : 0);
    const int waves_incl = wave_prefix_sum(lane < W ? s.wave_sum[lane] : 0);
    if (most > kRankMaxBin) return false;  // uniform
    int start = incl - local + (wave == 0 ? 0 : lane_value(waves_incl, wave - 1));
#pragma unroll
    for (int i = 0; i < BPT; ++i) {
        s.bins[threadIdx.x * BPT + i] = start;
        start += h[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i * THREADS < c && kb[i] != 0ull) ranks[atomicAdd(&s.bins[bin[i]], 1)] = rank_of(kb[i]);
    __syncthreads();
    int place[N];  // bins[b] is the end of bin b now, which is the start of bin b + 1
#pragma unroll
    for (int i = 0; i < N; ++i) {
        place[i] = CAP;
        if (i * THREADS >= c) continue;
        int p = kb[i] != 0ull && bin[i] > 0 ? s.bins[bin[i] - 1] : 0;
        const int end = kb[i] != 0ull ? s.bins[bin[i]] : 0;
        place[i] = kb[i] != 0ull ? p : CAP;
        const rank_t mine = rank_of(kb[i]);
        if (p < k)
            for (; p < end; ++p) place[i] += ranks[p] > mine ? 1 : 0;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < N; ++i)
        if (i * THREADS < c && place[i] < k) ranks[place[i]] = rank_of(kb[i]);
    __syncthreads();
    return true;
}

// Places in index order of the entries that satisfy pred(i) (entry tid + i * THREADS; registers first, then threads):
// the number of them before this wave's run of register i is lane_value(*before, index_order_lane<..>(i)).
// Returns their total.  counts: VPT * THREADS / 64 ints of LDS that nobody else uses meanwhile (more than one wave).
template <int THREADS, int VPT>
__device__ __forceinline__ int index_order_lane(int i) {
    constexpr int W = THREADS / 64, kPer = VPT * W > 64 ? VPT * W / 64 : 1;
    return (i * W + group_wave<THREADS>()) / kPer;
}
template <int THREADS, int VPT, typename Pred>
__device__ __forceinline__ int index_order(Pred&& pred, int* counts, int* before) {
    constexpr int W = THREADS / 64, E = VPT * W, kPer = E > 64 ? E / 64 : 1;
    static_assert(E % kPer == 0 && (W == 1 || E >= 64) && VPT <= 64, "whole lanes");
    const int lane = threadIdx.x & 63;
    int c = 0;  // lane i: this wave's count of register i
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const int n = static_cast<int>(__popcll(__ballot(pred(i))));
        c = lane == i ? n : c;
    }
    if constexpr (W == 1) {
        const int incl = wave_prefix_sum(c);
        *before = incl - c;
        return lane_value(incl, 63);
    } else {
        const int wave = group_wave<THREADS>();
        group_barrier<THREADS>();  // earlier readers are done
        if (lane < VPT) counts[lane * W + wave] = c;
        group_barrier<THREADS>();
        int h[kPer], local = 0;
#pragma unroll
        for (int j = 0; j < kPer; ++j) {
            h[j] = local;
            local += counts[lane * kPer + j];
        }
        const int incl = wave_prefix_sum(local);
        int mine = h[0];
#pragma unroll
        for (int j = 1; j < kPer; ++j) mine = (wave & (kPer - 1)) == j ? h[j] : mine;
        *before = incl - local + mine;
        return lane_value(incl, 63);
    }
}

// ---- the list of the best keys ----------------------------------------------------------------
// In LDS: CAP slots of which `count` are in use (a uniform register value).
constexpr int kSelectValues = 16;  // scores per thread and chunk

// The ordered image of a score, 0 where it is no candidate: one is greater than -inf (never NaN), as everywhere in the library.
__device__ __forceinline__ uint32_t candidate(float v) {
    return v > -__builtin_huge_valf() ? score_to_ordered(__float_as_uint(v + 0.0f)) : 0u;
}

template <int THREADS, int CAP, int BINS = kRankBins>
struct GroupList {
    static_assert(CAP % THREADS == 0, "the list must split evenly over the threads");
    static constexpr int VPT = kSelectValues;
    static constexpr int kLiveBlock = 4;  // values skipped together
    key64_t* keys;
    GroupScratch<THREADS, BINS>* s;
    int count;
    float floor;  // a score must be greater than this to be of interest (NaN never is)

    __device__ inline void init(key64_t* keys_, GroupScratch<THREADS, BINS>* s_) {
        keys = keys_;
        s = s_;
        count = 0;
        floor = -__builtin_huge_valf();
    }

    // Cuts the list to its best k (.. limit) keys.  Requires count > k.  Entries visited later have
    // larger indices, so they must beat the cut's score.
    __device__ inline void cut(int k, int limit) {
        __syncthreads();  // appended keys are visible
        key64_t kb[CAP / THREADS];
#pragma unroll
        for (int i = 0; i < CAP / THREADS; ++i) {
            const int j = static_cast<int>(threadIdx.x) + i * THREADS;
            kb[i] = j < count ? keys[j] : 0ull;
        }
        int kept = 0;
        const key64_t thr = group_radix_kth<THREADS>(kb, k, limit, *s, &kept);
        int mine = 0;
#pragma unroll
        for (int i = 0; i < CAP / THREADS; ++i) mine += static_cast<int>(__popcll(__ballot(kb[i] >= thr && kb[i] != 0ull)));
        int pos = 0;
        group_sum<THREADS>(mine, &pos, *s);  // its barriers stand between the reads above and the writes
#pragma unroll
        for (int i = 0; i < CAP / THREADS; ++i) {
            const bool keep = kb[i] >= thr && kb[i] != 0ull;
            const unsigned long long mask = __ballot(keep);
            if (keep) keys[pos + lanes_below(mask)] = kb[i];
            pos += static_cast<int>(__popcll(mask));
        }
        count = kept;
        floor = fmaxf(floor, key_score(thr));
        __syncthreads();
    }

    static __device__ __forceinline__ int lanes_below(unsigned long long mask) {
        return __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask >> 32),
                                         __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask), 0u));
    }

    // Raises the floor to just below the k-th largest of M group maxima, N per thread (ordered images, 0 = empty
    // group).  No bound comes from fewer than k groups.  Returns (uniformly) whether the k-th largest is the equal of others: more
    // than k + k / 32 maxima reach it.
    template <int N>
    __device__ inline bool bound_by(const uint32_t (&g)[N], int k) {
        int mine = 0;
#pragma unroll
        for (int i = 0; i < N; ++i) mine += static_cast<int>(__popcll(__ballot(g[i] != 0u)));
        int before = 0;
        const int total = group_sum<THREADS>(mine, &before, *s);
        if (total <= k) return false;
        int above = 0, bin = 0;
        const int limit = k + k / 32;
        const uint32_t thr = group_kth<THREADS>(g, k, limit, *s, &above, &bin);
        uint32_t below = ordered_to_score(thr - 1u);  // (the values are not 0, so thr is not)
        if (below == 0x80000000u) below = 0x80000001u;  // 0 counts as greater than the float below it, which -0 is not
        floor = fmaxf(floor, __uint_as_float(below));
        return above + bin > limit;
    }
    // The same from a chunk's scores, two or eight groups per thread so that M >= 2k if that can be;
    // slots far apart share a group, so that a chunk that is only partly filled still has as many groups.
    __device__ inline void bound(const float (&f)[VPT], int k) {
        static_assert(VPT == 16, "eight pairs per thread");
        float m[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) m[i] = fmaxf(f[i], f[i + 8]);
        if (k <= THREADS) {
            uint32_t g2[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) g2[i] = candidate(fmaxf(fmaxf(m[i], m[i + 2]), fmaxf(m[i + 4], m[i + 6])));
            bound_by(g2, k);
        } else {
            uint32_t g[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) g[i] = candidate(m[i]);
            bound_by(g, k);
        }
    }

    // Number of the workgroup's scores above the floor; *before = those in front of this thread's, which follow one another: a
    // thread counts and writes its own, one prefix sum over the threads in between, where a ballot and a rank per run of 64 take
    // half as much again.  Only the first `live` (uniform) values of a thread can be there.
    __device__ __forceinline__ int above(const float (&f)[VPT], int live, int* before) {
        int mine = 0;
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            if (i % kLiveBlock == 0 && i >= live) break;
            mine += f[i] > floor ? 1 : 0;
        }
        const int incl = wave_prefix_sum(mine);
        const int total = group_sum<THREADS>(lane_value(incl, 63), before, *s);
        *before += incl - mine;
        return total;
    }
    // f(position, key) for each of this thread's, positions from `pos` on; its value i is entry first + i * THREADS.
    template <typename F>
    __device__ __forceinline__ void each_above(const float (&v)[VPT], int live, int pos, int first, F&& f) const {
#pragma unroll
        for (int i = 0; i < VPT; ++i) {
            if (i % kLiveBlock == 0 && i >= live) break;
            if (v[i] > floor) {
                f(pos, make_key(v[i], static_cast<uint32_t>(first + i * THREADS)));
                ++pos;
            }
        }
    }

    // Visits entries [0, n) of a row of scores.  A chunk is read again after a cut instead of kept across it, whose
    // registers would otherwise set the kernel's number of waves.
    __device__ inline void stream(const float* __restrict__ scores, int n, int k) {
        for (int64_t c0 = 0; c0 < n; c0 += THREADS * VPT) {
            const int first = static_cast<int>(c0) + static_cast<int>(threadIdx.x);
            const int left = n - static_cast<int>(c0) - static_cast<int>(threadIdx.x);
            bool bounded = false, trimmed = false;
            for (;;) {
                // Opaque, so that neither the loads nor the index words (a register each) are moved out of the loop; in the global
                // address space, which the compiler would not know of a pointer that has been through asm.
                typedef __attribute__((address_space(1))) const float global_float;
                global_float* chunk = (global_float*)(scores + c0);
                asm volatile("" : "+s"(chunk));
                int first_now = first;
                asm volatile("" : "+v"(first_now));
                float f[VPT];
#pragma unroll
                for (int i = 0; i < VPT; ++i)
                    f[i] = i * THREADS < left ? chunk[threadIdx.x + i * THREADS] : -__builtin_huge_valf();
                // the first chunk of a long row starts with its own bound; later ones usually pass few keys
                if (c0 == 0 && floor == -__builtin_huge_valf() && n > CAP && !bounded) {
                    bound(f, k);
                    bounded = true;
                }
                int before = 0;
                int total = above(f, VPT, &before);
                const bool can_trim = !trimmed && count > k;
                if (count + total > CAP && !can_trim && !bounded) {
                    bound(f, k);
                    bounded = true;
                    total = above(f, VPT, &before);
                }
                if (count + total <= CAP) {
                    each_above(f, VPT, count + before, first_now, [&](int p, key64_t key) { keys[p] = key; });
                    count += total;
                    break;
                }
                if (can_trim) {
                    cut(k, compact_limit(k));
                    trimmed = true;
                    continue;
                }
                // one score per thread at a time: always fits after a cut
#pragma unroll 1
                for (int i = 0; i < VPT; ++i) {
                    if (count + THREADS > CAP) cut(k, CAP - THREADS < compact_limit(k) ? k : compact_limit(k));
                    const float one = i * THREADS < left ? chunk[threadIdx.x + i * THREADS] : -__builtin_huge_valf();
                    const bool keep = one > floor;
                    const unsigned long long mask = __ballot(keep);
                    int pos = 0;
                    const int more = group_sum<THREADS>(static_cast<int>(__popcll(mask)), &pos, *s);
                    if (keep) keys[count + pos + lanes_below(mask)] = make_key(one, static_cast<uint32_t>(first + i * THREADS));
                    count += more;
                }
                break;
            }
        }
    }

    // The best k of a row that at least k entries of reach the float above `floor`: ranks in place of keys[0 .. k), best first.
    // For rows of mostly equal scores, of which more than the list holds reach it: the entries above it go to the list, of those
    // that equal it the first that make up k, in index order, to its far end, and are never sorted.  Returns false (uniformly), with an empty
    // list and the same floor, where the entries above are too many for that; `floor` must not be -inf.
    __device__ inline bool finish_with_equals(const float* __restrict__ scores, int n, int k) {
        const float below = floor;
        // (0 follows the negative float next to it)
        const uint32_t next = score_to_ordered(__float_as_uint(below)) + 1u;
        const float least = __uint_as_float(next == 0x7FFFFFFFu ? 0u : ordered_to_score(next));
        list_rank_t* const ranks = reinterpret_cast<list_rank_t*>(keys);
        int equals = 0;
        floor = least;
        __syncthreads();  // earlier readers of the list and the scratch are done
        for (int64_t c0 = 0; c0 < n; c0 += THREADS * VPT) {
            const int first = static_cast<int>(c0) + static_cast<int>(threadIdx.x);
            const int left = n - static_cast<int>(c0) - static_cast<int>(threadIdx.x);
            const int live = (n - static_cast<int>(c0) + THREADS - 1) / THREADS;
            float f[VPT];
#pragma unroll
            for (int i = 0; i < VPT; ++i)
                f[i] = i * THREADS < left ? scores[c0 + threadIdx.x + i * THREADS] : -__builtin_huge_valf();
            int before = 0;
            const int total = above(f, live, &before);
            if (count + total + equals > CAP) {
                count = 0;
                floor = below;
                return false;
            }
            each_above(f, live, count + before, first, [&](int p, key64_t key) { keys[p] = key; });
            count += total;
            if (equals < k - count) {  // (more of them will not be wanted)
                const int more = index_order<THREADS, VPT>([&](int i) { return f[i] == least; }, s->hist[0], &before);
                const int taken = min(more, k - count - equals);
                if (count + equals + taken > CAP) {
                    count = 0;
                    floor = below;
                    return false;
                }
#pragma unroll
                for (int i = 0; i < VPT; ++i) {
                    const unsigned long long mask = __ballot(f[i] == least);
                    const int place = lane_value(before, index_order_lane<THREADS, VPT>(i)) + lanes_below(mask);
                    if (f[i] == least && place < taken)
                        ranks[CAP - 1 - equals - place] = make_rank(least, static_cast<uint32_t>(first + i * THREADS));
                }
                equals += taken;
            }
        }
        finish(k);  // (its sorts touch at most the power of two from k up, half the list)
        for (int j = static_cast<int>(threadIdx.x); j < k - count; j += THREADS) ranks[count + j] = ranks[CAP - 1 - j];
        count = k;
        __syncthreads();
        return true;
    }

    // The list's best k, best first, as ranks in place of keys[0 .. min(count, k)); count becomes that number.
    __device__ inline void finish(int k) {
        if (count > 0 && !group_rank_sort<THREADS, CAP>(keys, count, k, *s)) finish_by_network(k);
        count = min(count, k);
        __syncthreads();
    }
    __device__ inline void finish_by_network(int k) {
        if (count > k) cut(k, k);
        int P = 4;
        while (P < count) P <<= 1;
        list_rank_t* const ranks = reinterpret_cast<list_rank_t*>(keys);
        __syncthreads();
        for (int i = static_cast<int>(threadIdx.x); i < P; i += THREADS) ranks[i] = i < count ? rank_of(keys[i]) : no_rank();
        __syncthreads();
        group_sort_descending<THREADS>(ranks, P);
    }
};

// ---- rows that fit the workgroup's registers ------------------------------------------------------
template <int THREADS, int BINS>
struct RankScratch {
    static constexpr int kWavesPerGroup = THREADS / 64;
    uint32_t bins[BINS / 2];  // two 16-bit counts per word; first, for its alignment
    float lo[kWavesPerGroup], hi[kWavesPerGroup], sum[kWavesPerGroup];
    int count[kWavesPerGroup], wave_sum[kWavesPerGroup];
    int cut_bin, cut_begin, cut_end, too_full;  // (the cut: where there are several waves)
    int bad[2];
};

// wave_rank_select for a workgroup, straight from a row of scores in registers: v[i] of a thread is entry
// tid + i * THREADS of n, -inf where there is none (or none that can be selected; never NaN).  The
// best *c = min(k, candidates) go to s[SortSlot()(0)], [SortSlot()(1)], ..., best first, then no_rank() up
// to a multiple of 16.  One LDS atomic per entry and one per key of a bin that can hold the best k, where a
// list of whole keys would be written, read back and cut.  Returns false (uniformly) with nothing decided
// where bins do not separate the scores: equal or infinite ones, or more than kWaveRankMaxBin in a bin that matters.
// `some` is any finite number near the scores.  s: sort_slots(k rounded up to 16, + kWaveRankMaxBin) keys.
template <int THREADS, int VPT, int BINS>
__device__ inline bool group_rank_select(const float (&v)[VPT], int n, float some, int k, rank_t* s,
                                         RankScratch<THREADS, BINS>& r, int* c) {
    constexpr int W = THREADS / 64;
    constexpr int kMine = BINS / 2 / THREADS;  // words of a thread
    constexpr int kBlock = VPT < 4 ? VPT : 4;  // registers handled or skipped together
    static_assert(THREADS * VPT < 65536 && kMine % 4 == 0 && VPT % kBlock == 0, "16-bit counts, whole words and blocks");
    const int lane = threadIdx.x & 63;
    const int wave = group_wave<THREADS>();
    const int tid = group_thread<THREADS>();
    const float inf = __builtin_huge_valf();
    const SortSlot slot;
    uintx4* const mine = reinterpret_cast<uintx4*>(r.bins + tid * kMine);
#pragma unroll
    for (int i = 0; i < kMine / 4; ++i) mine[i] = uintx4{0u, 0u, 0u, 0u};
    if (W > 1 && tid == 0) r.too_full = r.bad[0] = r.bad[1] = 0;

    float lo = inf, hi = -inf, sum = 0.0f;
    int count = 0;
#pragma unroll
    for (int i0 = 0; i0 < VPT; i0 += kBlock)
        if (i0 * THREADS < n) {
#pragma unroll
            for (int i = i0; i < i0 + kBlock; ++i) {
                const bool valid = v[i] > -inf;
                lo = fminf(lo, valid ? v[i] : inf);
                hi = fmaxf(hi, v[i]);
                sum += valid ? v[i] - some : 0.0f;
                count += static_cast<int>(__popcll(__ballot(valid)));
            }
        }
    lo = wave_min(lo);
    hi = wave_max(hi);
    sum = wave_sum(sum);
    if (W > 1) {
        if (lane == 0) {
            r.lo[wave] = lo;
            r.hi[wave] = hi;
            r.sum[wave] = sum;
            r.count[wave] = count;
        }
        group_barrier<THREADS>();
        lo = wave_min(lane < W ? r.lo[lane] : inf);
        hi = wave_max(lane < W ? r.hi[lane] : -inf);
        sum = wave_sum(lane < W ? r.sum[lane] : 0.0f);
        count = lane_value(wave_prefix_sum(lane < W ? r.count[lane] : 0), 63);
    } else {
        group_barrier<THREADS>();
    }
    const int want = min(k, count);
    *c = want;
    if (count == 0) return true;
    const float span = fminf(hi - lo, 8.0f * (sum / static_cast<float>(count) + (some - lo)));
    const float scale = static_cast<float>(BINS - 1) / span;
    if (!(span > 0.0f && scale < inf && scale > 0.0f)) return false;  // (also an infinite or NaN span)
    const float from = lo + span;
#pragma unroll
    for (int i0 = 0; i0 < VPT; i0 += kBlock)
        if (i0 * THREADS < n) {
#pragma unroll
            for (int i = i0; i < i0 + kBlock; ++i) {
                const uint32_t bin = rank_bin<BINS>(v[i], from, scale);
                if (v[i] > -inf) atomicAdd(&r.bins[bin >> 1], 1u << (16 * (bin & 1)));
            }
        }
    group_barrier<THREADS>();
    // counts -> first places, and the bin across place k
    RankCut cut;
    const int local = rank_count<kMine>(mine, &cut.most);
    const int incl = wave_prefix_sum(local);
    int place = incl - local;
    if (W > 1) {
        if (lane == 63) r.wave_sum[wave] = incl;
        __syncthreads();
        const int waves_incl = wave_prefix_sum(lane < W ? r.wave_sum[lane] : 0);
        place += wave == 0 ? 0 : lane_value(waves_incl, wave - 1);
    }
    bool full = __ballot(place + local < want && cut.most > kWaveRankMaxBin) != 0ull;
    const unsigned long long across = __ballot(place < want && want <= place + local);  // one thread of the workgroup
    if (across != 0ull) {
        const int src = __builtin_ctzll(across);
        rank_find_cut<kMine>(r.bins + wave * (64 * kMine), src, lane_value(place, src), want, &cut);
        full = full || cut.full;
        if (W > 1) {
            r.cut_bin = cut.bin + wave * (128 * kMine);
            r.cut_begin = cut.begin;
            r.cut_end = cut.end;
        }
    }
    if (W == 1 && full) return false;
    if (W > 1 && full) r.too_full = 1;
    rank_places<kMine>(mine, place);
    group_barrier<THREADS>();
    if (W > 1) {
        if (r.too_full != 0) return false;
        cut.bin = r.cut_bin;
        cut.begin = r.cut_begin;
        cut.end = r.cut_end;
    }
#pragma unroll
    for (int i0 = 0; i0 < VPT; i0 += kBlock)
        if (i0 * THREADS < n) {
#pragma unroll
            for (int i = i0; i < i0 + kBlock; ++i) {
                const uint32_t bin = rank_bin<BINS>(v[i], from, scale);
                if (v[i] > -inf && static_cast<int>(bin) <= cut.bin) {
                    const int sh = 16 * (bin & 1);
                    const int at = static_cast<int>((atomicAdd(&r.bins[bin >> 1], 1u << sh) >> sh) & 0xFFFFu);
                    s[slot(at)] = make_rank(v[i], static_cast<uint32_t>(tid + i * THREADS));  // at < want + kWaveRankMaxBin
                }
            }
        }
    group_barrier<THREADS>();
    const int padded = (want + 15) / 16 * 16;
    if (wave == 0) rank_trim(s, cut, want, padded);
    group_barrier<THREADS>();
    for (int shift = 0, pass = 0;; shift ^= 8, ++pass) {
        for (int base = 16 * tid + shift; base + 16 <= padded; base += 16 * THREADS) sort_16_at(s, base);
        group_barrier<THREADS>();
        if (pass == 0 && padded > 16) continue;
        // sorted if the borders between the blocks just sorted agree; the two flags take turns, the one
        // cleared here was last read before this pass
        bool fine = true;
        for (int border = 16 * tid + (shift != 0 ? 8 : 16); border < padded; border += 16 * THREADS)
            fine = fine && s[slot(border - 1)] >= s[slot(border)];
        if (W == 1) {
            if (__ballot(!fine) == 0ull) break;
        } else {
            if (tid == 0) r.bad[(pass + 1) & 1] = 0;
            if (!fine) r.bad[pass & 1] = 1;
            group_barrier<THREADS>();
            if (r.bad[pass & 1] == 0) break;
        }
    }
    return true;
}

// The same result where the bins do not separate the scores (equal ones: with few heads the ReLU makes many that are
// exactly 0): the k-th best by histogram descent over the registers, equal scores at the border by their index, then a
// bitonic network, which a list that is already in order skips (the keys are emitted in index order, so one of equal
// scores is).  Returns the number of keys.  s: sort_slots of the power of two >= k (at least 16).
template <int THREADS, int VPT>
__device__ inline int group_exact_select(const float (&v)[VPT], int k, rank_t* s, GroupScratch<THREADS, 1>& g) {
    static_assert(VPT * (THREADS / 64) <= 256, "the counts fit a histogram");
    const int lane = threadIdx.x & 63;
    const int tid = group_thread<THREADS>();
    const auto below = [](unsigned long long mask) {
        return static_cast<int>(__builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask >> 32),
                                                          __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask), 0u)));
    };
    uint32_t x[VPT];
    int mine = 0, before = 0;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        x[i] = candidate(v[i]);
        mine += static_cast<int>(__popcll(__ballot(x[i] != 0u)));
    }
    const int count = group_sum<THREADS>(mine, &before, g);
    uint32_t thr = 1u;  // scores from thr on are kept
    if (count > k) {
        int above = 0, bin = 0;
        thr = group_kth<THREADS, true>(x, k, k, g, &above, &bin);
        if (above + bin > k) {  // thr is the k-th best itself: the first k - above entries that have it
            const int need = k - above;
            index_order<THREADS, VPT>([&](int i) { return x[i] == thr; }, g.hist[0], &before);
#pragma unroll
            for (int i = 0; i < VPT; ++i) {
                const bool equal = x[i] == thr;
                const int rank = lane_value(before, index_order_lane<THREADS, VPT>(i)) + below(__ballot(equal));
                if (equal && rank >= need) x[i] = 0u;
            }
        }
    }
    const int c = index_order<THREADS, VPT>([&](int i) { return x[i] >= thr; }, g.hist[0], &before);
    const SortSlot slot;
#pragma unroll
    for (int i = 0; i < VPT; ++i) {
        const bool keep = x[i] >= thr;
        const int at = lane_value(before, index_order_lane<THREADS, VPT>(i)) + below(__ballot(keep));
        if (keep) s[slot(at)] = make_rank(v[i], static_cast<uint32_t>(tid + i * THREADS));
    }
    int P = 16;
    while (P < c) P <<= 1;
    for (int i = c + tid; i < P; i += THREADS) s[slot(i)] = no_rank();
    if (tid == 0) g.flag = 0;
    group_barrier<THREADS>();
    bool unsorted = false;
    for (int i = tid + 1; i < c; i += THREADS) unsorted = unsorted || s[slot(i - 1)] < s[slot(i)];
    if (__ballot(unsorted) != 0ull && lane == 0) g.flag = 1;
    group_barrier<THREADS>();
    if (g.flag != 0) {
        if constexpr (THREADS == 64) wave_sort_descending(s, P);
        else sort_descending_by<3, THREADS>(s, P);
    }
    return c;
}

}  // namespace si
