// Wave-level building blocks of the per-tile select, the merge and the write-out (Algorithm 2):
// radix selection of the k-th largest key, order-preserving compaction, and a bitonic sort, each
// run by one 64-lane wave on one query row without workgroup barriers.  Keys are the 64-bit
// (score, ~index) words of si_internal.h, whose unsigned order is the total order of Section 4.1.
#pragma once

#include "si_internal.h"
#include "wave_ops.h"

namespace si {

constexpr int kKeysInFlight = 16;  // global loads a lane issues before it uses them

// A mid-stream cut keeps the best k .. compact_limit(k) keys of a row (only the last cut has to
// be exact).
__host__ __device__ inline int compact_limit(int k) { return k + k / 16; }

// ---- the form keys are sorted in --------------------------------------------------------------
// A double with the score's own bits in the high word and, in the low one, ~index where the score is positive, the index where it is
// negative: the order of doubles is then the order of keys (Section 4.1), and an exchange is one v_max_f64 and one v_min_f64, 12
// cycles in a chain, where a 64-bit integer compare and four selects take 44, and with a second wave on the SIMD 135
// (one workgroup of 1 and of 8 waves).  No key is a double NaN or infinity: that takes a float of 0x7FF00000 and more in
// magnitude, a NaN; zero and denormal scores make denormal doubles, which these instructions keep.
typedef double rank_t;
__device__ __forceinline__ rank_t rank_from_words(uint32_t high, uint32_t low) {
    return __builtin_bit_cast(rank_t, (static_cast<unsigned long long>(high) << 32) | low);
}
__device__ __forceinline__ uint32_t rank_high(rank_t r) { return static_cast<uint32_t>(__builtin_bit_cast(unsigned long long, r) >> 32); }
__device__ __forceinline__ uint32_t rank_low(rank_t r) { return static_cast<uint32_t>(__builtin_bit_cast(unsigned long long, r)); }
__device__ __forceinline__ uint32_t sign_mask(uint32_t bits) { return static_cast<uint32_t>(static_cast<int32_t>(bits) >> 31); }
__device__ __forceinline__ rank_t make_rank(float score, uint32_t idx) {
    const uint32_t bits = __float_as_uint(score + 0.0f);
    return rank_from_words(bits, ~idx ^ sign_mask(bits));
}
__device__ __forceinline__ rank_t rank_of(key64_t key) {
    const uint32_t bits = ordered_to_score(static_cast<uint32_t>(key >> 32));
    return rank_from_words(bits, static_cast<uint32_t>(key) ^ sign_mask(bits));
}
__device__ __forceinline__ float rank_score(rank_t r) { return __uint_as_float(rank_high(r)); }
__device__ __forceinline__ int32_t rank_index(rank_t r) { return static_cast<int32_t>(~(rank_low(r) ^ sign_mask(rank_high(r)))); }
// Below every key: the empty slot.
__device__ __forceinline__ rank_t no_rank() { return rank_from_words(0xFF800000u, 0xFFFFFFFFu); }
__device__ __forceinline__ void exchange(rank_t& better, rank_t& worse) {
    const rank_t x = better, y = worse;
#if defined(__HIP_DEVICE_COMPILE__)
    asm("v_max_f64 %0, %1, %2" : "=v"(better) : "v"(x), "v"(y));
    asm("v_min_f64 %0, %1, %2" : "=v"(worse) : "v"(x), "v"(y));
#else
    (void)x; (void)y;
#endif
}
// x or -x: an ascending run is a descending one of the negated keys.
__device__ __forceinline__ rank_t flip(rank_t x, uint32_t sign) { return rank_from_words(rank_high(x) ^ sign, rank_low(x)); }

// ---- wave-level selection -----------------------------------------------------------------
// One wave works on one row without workgroup barriers: its 64 lanes stream the row's keys from
// global memory (the row buffer is L2 resident), build a 256-bin histogram in the wave's own
// slice of LDS, and walk the bins with a wave prefix sum.

// A row's keys as seen by one wave.  Lane l is responsible for keys l, l+64, l+128, ...
// RegKeys holds them in registers (rows of up to 64*R keys: read from memory once);
// StreamKeys re-reads them from global memory on every sweep (any length).
// RegKeys skips blocks of 512 keys past the end of the row: R covers the longest row of the largest k of a
// kernel, and at k = 512 a row fills 17 to 22 of 38 registers.  Whole blocks only: a branch per 64 keys costs
// more than it saves (compaction +30 %).  With the lane moves of wave_ops.h in place of LDS permutes, 65536
// queries at k = 512 went from 7972 to 7686 us, 2 x 8191 at k = 300 from 366 to 318.
// SKIP = false: no test per block, for rows that fill most of their registers.
template <int R, bool SKIP = true>
struct RegKeys {
    static constexpr int kBlock = 8;
    key64_t kb[R];
    int n;
    // The lane number, opaque to the compiler: what depends on it is computed where it is used, and not kept -- spilled, one
    // address per key, each of whose reloads waited for the key before it -- across the loops of a persistent kernel.
    static __device__ __forceinline__ int fresh_lane() {
        int lane = threadIdx.x & 63;
        asm volatile("" : "+v"(lane));
        return lane;
    }
    __device__ inline void load(const key64_t* buf, int n_) {
        n = min(n_, 64 * R);
        const int lane = fresh_lane();
#pragma unroll
        for (int i = 0; i < R; ++i) kb[i] = lane < n - 64 * i ? buf[lane + 64 * i] : 0ull;
    }
    // f(key, valid, first_lane_index): called for successive blocks of 64 keys, in key order
    template <typename F>
    __device__ inline void sweep(F&& f) const {
        sweep_numbered([&](int, key64_t key, bool valid) { f(key, valid); });
    }
    // f(i, key, valid) with the register's number
    template <typename F>
    __device__ inline void sweep_numbered(F&& f) const {
        const int lane = fresh_lane();
#pragma unroll
        for (int i0 = 0; i0 < R; i0 += kBlock) {
            if (!SKIP || 64 * i0 < n) {
#pragma unroll
                for (int i = i0; i < i0 + kBlock && i < R; ++i) f(i, kb[i], lane < n - 64 * i);
            }
        }
    }
};

struct StreamKeys {
    const key64_t* buf;
    int n;
    template <typename F>
    __device__ inline void sweep(F&& f) const {
        const int lane = threadIdx.x & 63;
        // several keys per lane in flight at a time: latency is what matters
        for (int base = 0; base < n; base += 64 * kKeysInFlight) {
            key64_t kb[kKeysInFlight];
#pragma unroll
            for (int i = 0; i < kKeysInFlight; ++i) {
                const int j = base + 64 * i + lane;
                kb[i] = j < n ? buf[j] : 0ull;
            }
#pragma unroll
            for (int i = 0; i < kKeysInFlight; ++i) f(kb[i], base + 64 * i + lane < n);
        }
    }
};

// Threshold key `thr` and count `kept` such that exactly `kept` of the row's n distinct keys
// are >= thr, with k <= kept <= max(k, limit).  MSB-first radix descent, up to 8 bits per pass; it
// stops as soon as the bin holding the k-th largest key is small enough for `kept` to respect
// the limit (limit == k: exact selection).  Requires n > k.  Wave-uniform arguments.
//
// The descent starts at the highest bit in which two score words of the row differ (one OR / AND
// scan of the keys): the candidates of a row are the upper tail of its score distribution, so their
// sign and exponent bits agree, and a first pass over those bits would put every key into one or
// two bins -- no information, and 64 lanes adding to the same LDS word serialise.  Windows never
// straddle the boundary between the score word and the index word, so each pass works on one
// 32-bit half of the keys.
template <typename Keys>
__device__ inline key64_t wave_radix_kth(const Keys& keys, int k, int limit, int* hist, int* kept) {
    const int lane = threadIdx.x & 63;
    uint32_t any_hi = 0u, all_hi = 0xFFFFFFFFu;
    keys.sweep([&](key64_t key, bool valid) {
        const uint32_t hi = static_cast<uint32_t>(key >> 32);
        any_hi |= valid ? hi : 0u;
        all_hi &= valid ? hi : 0xFFFFFFFFu;
    });
    any_hi = wave_or(any_hi);
    all_hi = wave_and(all_hi);
    const uint32_t diff_hi = any_hi ^ all_hi;
    // highest undecided bit of the 64-bit key; equal scores everywhere: the index word decides
    int top = diff_hi != 0u ? 63 - __builtin_clz(diff_hi) : 31;
    key64_t prefix = top >= 32
        ? static_cast<key64_t>(all_hi & ~((2u << (top - 32)) - 1u)) << 32
        : static_cast<key64_t>(all_hi) << 32;
    int need = k;
    int bin = 0;
    for (;;) {
        const int shift = max(top - 7, top >= 32 ? 32 : 0);  // this pass decides bits [shift, top]
        const int nbits = top - shift + 1;
        const uint32_t dmask = (1u << nbits) - 1u;
#pragma unroll
        for (int i = 0; i < 4; ++i) hist[lane + 64 * i] = 0;
        __builtin_amdgcn_wave_barrier();
        if (shift >= 32) {
            // digits of the score word: 32-bit arithmetic on the high half of the key
            const int sh = shift - 32;
            const bool whole = top == 63;  // nothing above the window
            const uint32_t want = whole ? 0u : static_cast<uint32_t>(prefix >> 32) >> (top - 31);
            keys.sweep([&](key64_t key, bool valid) {
                const uint32_t hi = static_cast<uint32_t>(key >> 32);
                const bool in_prefix = whole || ((hi >> (top - 31)) == want);
                if (valid && in_prefix) atomicAdd(&hist[(hi >> sh) & dmask], 1);
            });
        } else {
            // equal scores: digits of the index word
            const key64_t want = prefix >> (top + 1);
            keys.sweep([&](key64_t key, bool valid) {
                const bool in_prefix = (key >> (top + 1)) == want;
                if (valid && in_prefix) atomicAdd(&hist[static_cast<uint32_t>(key >> shift) & dmask], 1);
            });
        }
        __builtin_amdgcn_wave_barrier();
        // Lane l owns bins 255-4l .. 252-4l (walking down from the top bin).
        int h[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) h[j] = hist[255 - 4 * lane - j];
        __builtin_amdgcn_wave_barrier();
        const int local = h[0] + h[1] + h[2] + h[3];
        const int incl = wave_prefix_sum(local);
        int cum = incl - local;  // keys in bins above this lane's
        const bool crossing = cum < need && need <= incl;  // true in exactly one lane
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
        bin = lane_value(new_bin, src);
        prefix |= static_cast<key64_t>(digit) << shift;
        // keys >= prefix: the (k - need) in higher bins plus this whole bin
        if (k - need + bin <= limit || shift == 0) break;
        top = shift - 1;
    }
    *kept = k - need + bin;
    return prefix;
}

struct IdentitySlot {
    __device__ inline int operator()(int i) const { return i; }
};
__device__ __forceinline__ void put_key(key64_t* dst, key64_t key) { *dst = key; }
__device__ __forceinline__ void put_key(rank_t* dst, key64_t key) { *dst = rank_of(key); }

// Writes the row's keys >= thr to dst[slot(0)], dst[slot(1)], ... in key order (dst may be the
// row buffer itself when slot is the identity: a block of keys is always read before anything
// at or behind it is written).  `cap` bounds the logical positions written.  Returns how many
// keys qualified.
template <typename Keys, typename Out, typename Slot = IdentitySlot>
__device__ inline int wave_keep(const Keys& keys, key64_t thr, Out* dst, int cap, Slot slot = Slot()) {
    int pos = 0;
    keys.sweep([&](key64_t key, bool valid) {
        const bool keep = valid && key >= thr;
        const unsigned long long mask = __ballot(keep);
        const int below = __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask >> 32),
                          __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask), 0u));
        if (keep && pos + below < cap) put_key(dst + slot(pos + below), key);
        pos += __popcll(mask);
    });
    return pos;
}

// ---- wave-level sort ------------------------------------------------------------------------
// Bitonic network over P keys (a power of two >= 16) in one wave's slice of LDS, best (largest)
// key first.  A compare-exchange at stride 2^j only pairs keys whose positions differ in bit j,
// so a lane that holds the 2^NB keys spanning bits [b, b+NB) of the position can run NB
// consecutive strides of the network in registers: one LDS round trip per group of up to four
// strides instead of one per stride (15 instead of 55 for P = 1024).
// Sixteen keys (128 B) are followed by two slots of padding, so that lanes reading their own
// 16-key block with 128-bit loads start in different banks.
struct SortSlot {
    __device__ inline int operator()(int i) const { return i + ((i >> 4) << 1); }
};
__host__ __device__ inline int sort_slots(int P) { return P + P / 8; }

// Strides 2^(b+NB-1) .. 2^b of the merge phase that builds sorted runs of `size` (> 2^(b+NB-1)).
// THREADS = 64: by one wave on its own slice of LDS, without barriers; more: by the whole workgroup.
template <int THREADS>
__device__ __forceinline__ int sort_thread() { return static_cast<int>(THREADS == 64 ? threadIdx.x & 63 : threadIdx.x); }
template <int THREADS>
__device__ __forceinline__ void sort_barrier() {
    if constexpr (THREADS == 64) __builtin_amdgcn_wave_barrier();
    else __syncthreads();
}
template <int NB, int THREADS>
__device__ inline void sort_pass(rank_t* s, int P, int b, int size) {
    constexpr int E = 1 << NB;
    const SortSlot slot;
    for (int u = sort_thread<THREADS>(); u < (P >> NB); u += THREADS) {
        const int base = (u & ((1 << b) - 1)) | ((u >> b) << (b + NB));
        const uint32_t sign = (base & size) == 0 ? 0u : 0x80000000u;
        rank_t v[E];
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = flip(s[slot(base | (j << b))], sign);
#pragma unroll
        for (int d = E >> 1; d > 0; d >>= 1)
#pragma unroll
            for (int i = 0; i < (E >> 1); ++i) {
                const int lo = 2 * i - (i & (d - 1));
                exchange(v[lo], v[lo + d]);
            }
#pragma unroll
        for (int j = 0; j < E; ++j) s[slot(base | (j << b))] = flip(v[j], sign);
    }
    sort_barrier<THREADS>();
}

// The LG lowest strides (2^(LG-1) .. 1) on a lane's own block of E = 2^LG consecutive keys (LG = 3
// or 4, so that a block never straddles a padding gap); with FIRST, the whole network up to runs
// of E (sizes 2 .. E) instead.
template <int LG, bool FIRST, int THREADS>
__device__ inline void sort_block(rank_t* s, int P, int size) {
    constexpr int E = 1 << LG;
    typedef rank_t rankx2 __attribute__((ext_vector_type(2)));
    const SortSlot slot;
    for (int base = E * sort_thread<THREADS>(); base < P; base += E * THREADS) {
        rankx2* blk = reinterpret_cast<rankx2*>(s + slot(base));  // 16-byte aligned
        const uint32_t sign = (base & (FIRST ? E : size)) == 0 ? 0u : 0x80000000u;
        rank_t v[E];
#pragma unroll
        for (int j = 0; j < E / 2; ++j) {
            const rankx2 t = blk[j];
            v[2 * j] = flip(t.x, sign);
            v[2 * j + 1] = flip(t.y, sign);
        }
#pragma unroll
        for (int sz = FIRST ? 2 : E; sz <= E; sz <<= 1)
#pragma unroll
            for (int d = sz >> 1; d > 0; d >>= 1)
#pragma unroll
                for (int i = 0; i < E / 2; ++i) {
                    const int lo = 2 * i - (i & (d - 1));
                    if (sz == E || (lo & sz) == 0) exchange(v[lo], v[lo + d]);
                    else exchange(v[lo + d], v[lo]);
                }
#pragma unroll
        for (int j = 0; j < E / 2; ++j) {
            rankx2 t;
            t.x = flip(v[2 * j], sign);
            t.y = flip(v[2 * j + 1], sign);
            blk[j] = t;
        }
    }
    sort_barrier<THREADS>();
}

// LG = keys per lane and pass (as a power of two): 4 keeps all 64 lanes busy from P = 1024 on,
// 3 does so for P = 512.
template <int LG, int THREADS>
__device__ inline void sort_descending_by(rank_t* s, int P) {
    sort_block<LG, true, THREADS>(s, P, 0);
    for (int lg = LG + 1; (1 << lg) <= P; ++lg) {
        const int size = 1 << lg;
        for (int top = lg; top > LG;) {  // stride bits [LG, lg), up to LG at a time from the top
            const int nb = min(LG, top - LG);
            const int b = top - nb;
            if (nb == 4) sort_pass<4, THREADS>(s, P, b, size);
            else if (nb == 3) sort_pass<3, THREADS>(s, P, b, size);
            else if (nb == 2) sort_pass<2, THREADS>(s, P, b, size);
            else sort_pass<1, THREADS>(s, P, b, size);
            top = b;
        }
        sort_block<LG, false, THREADS>(s, P, size);
    }
}

// Whether the first c keys are in order already (equal scores in the order they were met): one round of reads on
// a list that is not.  What it saves in the single pass (us): one head, negative weight, so that the best are all 0, 16384
// queries, k = 2048 1940 -> 1681, 32768, k = 1024 1854 -> 1640; distinct scores unchanged.
__device__ inline bool wave_sorted(const rank_t* s, int c) {
    const SortSlot slot;
    for (int base = 1; base < c; base += 64) {
        const int i = min(base + static_cast<int>(threadIdx.x & 63), c - 1);
        if (__ballot(s[slot(i - 1)] < s[slot(i)]) != 0ull) return false;
    }
    return true;
}

// s: sort_slots(P) keys of LDS owned by this wave, key i at s[SortSlot()(i)]; P a power of two >= 16.
__device__ inline void wave_sort_descending(rank_t* s, int P) {
    if (P <= 512) sort_descending_by<3, 64>(s, P);
    else sort_descending_by<4, 64>(s, P);
}

// ---- wave-level selection and sort in one: bins of equal score width -----------------------------
// The best min(k, n) of a row's keys, best first, to s[SortSlot()(0)], [SortSlot()(1)], ...: the keys are
// counted into kWaveRankBins bins of equal score width, those of the bins that can hold the best k are
// laid out in bin order, the bin across the k-th place is cut by comparing its keys, and what is then
// out of order only by positions inside a bin is put right by sorting blocks of 16 keys in a lane's
// registers, aligned and shifted by 8 in turn, until the block borders agree (two passes while no key is 8
// or more places off).  Bins only group keys; every decision compares whole keys, so the result is exact.
// As in group_rank_sort, far outliers share the first bin instead of squeezing the rest.
// About 40 vector instructions per 64 keys and 800 for the blocks, where the exact radix cut and the
// bitonic network take three passes over the keys and 440 exchanges per lane at k = 1024.  In the single pass
// (us, before -> after): 32768 queries, k = 1024 2394 -> 2199; 2 x 8191, k = 300 317 -> 280; 65536, k = 512
// 7565 -> 7451; 262144, k = 1024 109170 -> 107046.
// s: sort_slots(k rounded up to 16, + kWaveRankMaxBin) keys; bins: kWaveRankBins / 2 words, 16-byte aligned.  An empty row: nothing.
// Returns false with nothing decided (equal or infinite scores, a bin of more than kWaveRankMaxBin
// keys): the caller takes the radix cut and the network.
constexpr int kWaveRankBins = 2048;
constexpr int kWaveRankMaxBin = 64;

// Batcher's odd-even merge sort of 16 keys, largest first.
__device__ inline void sort_16(rank_t (&v)[16]) {
#pragma unroll
    for (int p = 1; p < 16; p <<= 1)
#pragma unroll
        for (int d = p; d > 0; d >>= 1)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                // i is the upper partner of a comparison at distance d inside a merge of runs of p
                const bool first = i >= d % p && ((i - d % p) / d) % 2 == 0;
                if (first && i + d < 16 && i / (2 * p) == (i + d) / (2 * p)) exchange(v[i], v[i + d]);
            }
}

// Keys [base, base + 16) of a list, base a multiple of 8: each half block is 16-byte aligned and without a gap.
__device__ inline void sort_16_at(rank_t* s, int base) {
    typedef rank_t rankx2 __attribute__((ext_vector_type(2)));
    const SortSlot slot;
    rankx2* first = reinterpret_cast<rankx2*>(s + slot(base));
    rankx2* second = reinterpret_cast<rankx2*>(s + slot(base + 8));
    rank_t v[16];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const rankx2 t = first[j], u = second[j];
        v[2 * j] = t.x;
        v[2 * j + 1] = t.y;
        v[8 + 2 * j] = u.x;
        v[8 + 2 * j + 1] = u.y;
    }
    sort_16(v);
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        rankx2 t, u;
        t.x = v[2 * j];
        t.y = v[2 * j + 1];
        u.x = v[8 + 2 * j];
        u.y = v[8 + 2 * j + 1];
        first[j] = t;
        second[j] = u;
    }
}

// Bin 0 holds the best scores; what is out of range goes to the nearest end.
template <int BINS>
__device__ __forceinline__ uint32_t rank_bin(float score, float from, float scale) {
    const float at = (from - score) * scale;
#if defined(__HIP_DEVICE_COMPILE__)
    return static_cast<uint32_t>(__builtin_amdgcn_fmed3f(at, 0.0f, static_cast<float>(BINS - 1)));
#else
    return static_cast<uint32_t>(at);
#endif
}
typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
struct RankCut {
    int bin, begin, end;  // the bin across the last place wanted, and the places it covers
    int most;             // this thread's fullest bin
    bool full;            // it, or a better one of the same thread, holds more than kWaveRankMaxBin keys
};
// A thread's bins are the halves of MINE consecutive words, low half first; no two counts add up to 2^16.  Their sum.
template <int MINE>
__device__ __forceinline__ int rank_count(const uintx4* mine, int* most) {
    typedef unsigned short ushortx2 __attribute__((ext_vector_type(2)));
    uint32_t both = 0u;
    ushortx2 top = {0, 0};
#pragma unroll
    for (int i = 0; i < MINE / 4; ++i) {
        const uintx4 t = mine[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            both += t[j];
            top = __builtin_elementwise_max(top, __builtin_bit_cast(ushortx2, static_cast<uint32_t>(t[j])));
        }
    }
    *most = max(static_cast<int>(top.x), static_cast<int>(top.y));
    return static_cast<int>((both & 0xFFFFu) + (both >> 16));
}
// The bin, among those of the wave's lane `src` (whose first place is `place`), that holds place want - 1: one bin per lane.
template <int MINE>
__device__ __forceinline__ void rank_find_cut(const uint32_t* wave_bins, int src, int place, int want, RankCut* cut) {
    static_assert(2 * MINE <= 64, "a lane for each of a thread's bins");
    const int lane = threadIdx.x & 63;
    const uint32_t word = wave_bins[src * MINE + min(lane >> 1, MINE - 1)];
    const int count = lane < 2 * MINE ? static_cast<int>((lane & 1) != 0 ? word >> 16 : word & 0xFFFFu) : 0;
    const int end = place + wave_prefix_sum(count);
    const int at = __builtin_ctzll(__ballot(end >= want));
    cut->bin = 2 * MINE * src + at;
    cut->end = lane_value(end, at);
    cut->begin = cut->end - lane_value(count, at);
    cut->full = __ballot(lane <= at && count > kWaveRankMaxBin) != 0ull;
}
// The thread's counts become the first places of its bins, the first of which starts at `place`.  Places past 2^16 - 1 do not exist.
template <int MINE>
__device__ __forceinline__ void rank_places(uintx4* mine, int place) {
    uint32_t at = static_cast<uint32_t>(place) * 0x10001u;
#pragma unroll
    for (int i = 0; i < MINE / 4; ++i) {
        const uintx4 t = mine[i];
        uintx4 p;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint32_t c = t[j];
            p[j] = at + (c << 16);
            at += c + ((c >> 16) | (c << 16));  // both halves: the sum of the two counts
        }
        mine[i] = p;
    }
}
// One wave: of the bin across the last place only the best want - begin keys stay, in order (it holds at most kWaveRankMaxBin);
// the places up to `padded` are emptied.
__device__ __forceinline__ void rank_trim(rank_t* s, const RankCut& cut, int want, int padded) {
    const int lane = threadIdx.x & 63;
    const SortSlot slot;
    if (cut.end > want) {
        const int size = cut.end - cut.begin;
        const rank_t key = lane < size ? s[slot(cut.begin + lane)] : no_rank();
        int better = 0;
        for (int j = 0; j < size; ++j) {
            const rank_t other = rank_from_words(__builtin_amdgcn_readlane(static_cast<int>(rank_high(key)), j),
                                                 __builtin_amdgcn_readlane(static_cast<int>(rank_low(key)), j));
            better += other > key ? 1 : 0;
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < size && cut.begin + better < want) s[slot(cut.begin + better)] = key;
    }
    __builtin_amdgcn_wave_barrier();
    if (lane < padded - want) s[slot(want + lane)] = no_rank();
}

template <int R>
__device__ inline bool wave_rank_select(const RegKeys<R>& keys, int k, rank_t* s, uint32_t* bins) {
    constexpr int kWords = kWaveRankBins / 2;  // two 16-bit counts per word (a row has fewer than 2^16 keys)
    constexpr int kMine = kWords / 64;         // words of a lane
    static_assert(64 * R < 65536 && kMine % 4 == 0, "counts and places are 16 bits wide");
    const int lane = threadIdx.x & 63;
    const float inf = __builtin_huge_valf();
    const SortSlot slot;
    const int n = keys.n;
    if (n == 0) return true;
    // (key 0 of the row is lane 0's first register)
    const float some = lane_value(key_score(keys.kb[0]), 0);
    float lo = inf, hi = -inf, sum = 0.0f;
    keys.sweep([&](key64_t key, bool valid) {
        const float v = key_score(key);
        lo = fminf(lo, valid ? v : inf);
        hi = fmaxf(hi, valid ? v : -inf);
        sum += valid ? v - some : 0.0f;
    });
    lo = wave_min(lo);
    hi = wave_max(hi);
    sum = wave_sum(sum);
    const float span = fminf(hi - lo, 8.0f * (sum / static_cast<float>(n) + (some - lo)));
    const float scale = static_cast<float>(kWaveRankBins - 1) / span;
    if (!(span > 0.0f && scale < inf && scale > 0.0f)) return false;
    const float from = lo + span;

    uintx4* const mine = reinterpret_cast<uintx4*>(bins + lane * kMine);  // words [lane * kMine, + kMine)
#pragma unroll
    for (int i = 0; i < kMine / 4; ++i) mine[i] = uintx4{0u, 0u, 0u, 0u};
    __builtin_amdgcn_wave_barrier();
    uint32_t bin[R];
    keys.sweep_numbered([&](int i, key64_t key, bool valid) {
        bin[i] = rank_bin<kWaveRankBins>(key_score(key), from, scale);
        if (valid) atomicAdd(&bins[bin[i] >> 1], 1u << (16 * (bin[i] & 1)));
    });
    __builtin_amdgcn_wave_barrier();
    // counts -> first places, and the bin across place k (the last one in use if there are at most k keys)
    const int want = min(k, n);
    RankCut cut;
    const int local = rank_count<kMine>(mine, &cut.most);
    const int place = wave_prefix_sum(local) - local;
    const int src = __builtin_ctzll(__ballot(place < want && want <= place + local));
    rank_find_cut<kMine>(bins, src, lane_value(place, src), want, &cut);
    if (cut.full || __ballot(place + local < want && cut.most > kWaveRankMaxBin) != 0ull) return false;
    rank_places<kMine>(mine, place);
    __builtin_amdgcn_wave_barrier();
    keys.sweep_numbered([&](int i, key64_t key, bool valid) {
        if (valid && static_cast<int>(bin[i]) <= cut.bin) {
            const int sh = 16 * (bin[i] & 1);
            const int at = static_cast<int>((atomicAdd(&bins[bin[i] >> 1], 1u << sh) >> sh) & 0xFFFFu);
            s[slot(at)] = rank_of(key);
        }
    });
    __builtin_amdgcn_wave_barrier();
    const int padded = (want + 15) / 16 * 16;
    rank_trim(s, cut, want, padded);
    __builtin_amdgcn_wave_barrier();
    for (int shift = 0, pass = 0;; shift ^= 8, ++pass) {
        for (int base = 16 * lane + shift; base + 16 <= padded; base += 16 * 64) sort_16_at(s, base);
        __builtin_amdgcn_wave_barrier();
        if (pass == 0 && padded > 16) continue;
        // sorted if the borders between the blocks just sorted agree
        bool fine = true;
        for (int border = 16 * lane + (shift != 0 ? 8 : 16); border < padded; border += 16 * 64)
            fine = fine && s[slot(border - 1)] >= s[slot(border)];
        if (__ballot(!fine) == 0ull) break;
    }
    return true;
}

}  // namespace si
