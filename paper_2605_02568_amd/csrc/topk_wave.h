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
    __device__ inline void load(const key64_t* buf, int n_) {
        n = min(n_, 64 * R);
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int j = lane + 64 * i;
            kb[i] = j < n ? buf[j] : 0ull;
        }
    }
    // f(key, valid, first_lane_index): called for successive blocks of 64 keys, in key order
    template <typename F>
    __device__ inline void sweep(F&& f) const {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i0 = 0; i0 < R; i0 += kBlock) {
            if (!SKIP || 64 * i0 < n) {
#pragma unroll
                for (int i = i0; i < i0 + kBlock && i < R; ++i) f(kb[i], lane + 64 * i < n);
            }
        }
    }
    // f(i, key, valid) with the register's number
    template <typename F>
    __device__ inline void sweep_numbered(F&& f) const {
        const int lane = threadIdx.x & 63;
#pragma unroll
        for (int i0 = 0; i0 < R; i0 += kBlock) {
            if (!SKIP || 64 * i0 < n) {
#pragma unroll
                for (int i = i0; i < i0 + kBlock && i < R; ++i) f(i, kb[i], lane + 64 * i < n);
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

// Writes the row's keys >= thr to dst[slot(0)], dst[slot(1)], ... in key order (dst may be the
// row buffer itself when slot is the identity: a block of keys is always read before anything
// at or behind it is written).  `cap` bounds the logical positions written.  Returns how many
// keys qualified.
template <typename Keys, typename Slot = IdentitySlot>
__device__ inline int wave_keep(const Keys& keys, key64_t thr, key64_t* dst, int cap, Slot slot = Slot()) {
    int pos = 0;
    keys.sweep([&](key64_t key, bool valid) {
        const bool keep = valid && key >= thr;
        const unsigned long long mask = __ballot(keep);
        const int below = __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(mask >> 32),
                          __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(mask), 0u));
        if (keep && pos + below < cap) dst[slot(pos + below)] = key;
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

__device__ inline void compare_exchange(key64_t& x, key64_t& y, bool descending) {
    const bool swap = (x < y) == descending;
    const key64_t a = swap ? y : x;
    const key64_t b = swap ? x : y;
    x = a;
    y = b;
}

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
__device__ inline void sort_pass(key64_t* s, int P, int b, int size) {
    constexpr int E = 1 << NB;
    const SortSlot slot;
    for (int u = sort_thread<THREADS>(); u < (P >> NB); u += THREADS) {
        const int base = (u & ((1 << b) - 1)) | ((u >> b) << (b + NB));
        const bool descending = (base & size) == 0;
        key64_t v[E];
#pragma unroll
        for (int j = 0; j < E; ++j) v[j] = s[slot(base | (j << b))];
#pragma unroll
        for (int d = E >> 1; d > 0; d >>= 1)
#pragma unroll
            for (int i = 0; i < (E >> 1); ++i) {
                const int lo = 2 * i - (i & (d - 1));
                compare_exchange(v[lo], v[lo + d], descending);
            }
#pragma unroll
        for (int j = 0; j < E; ++j) s[slot(base | (j << b))] = v[j];
    }
    sort_barrier<THREADS>();
}

// The LG lowest strides (2^(LG-1) .. 1) on a lane's own block of E = 2^LG consecutive keys (LG = 3
// or 4, so that a block never straddles a padding gap); with FIRST, the whole network up to runs
// of E (sizes 2 .. E) instead.
template <int LG, bool FIRST, int THREADS>
__device__ inline void sort_block(key64_t* s, int P, int size) {
    constexpr int E = 1 << LG;
    typedef key64_t key64x2 __attribute__((ext_vector_type(2)));
    const SortSlot slot;
    for (int base = E * sort_thread<THREADS>(); base < P; base += E * THREADS) {
        key64x2* blk = reinterpret_cast<key64x2*>(s + slot(base));  // 16-byte aligned
        key64_t v[E];
#pragma unroll
        for (int j = 0; j < E / 2; ++j) {
            const key64x2 t = blk[j];
            v[2 * j] = t.x;
            v[2 * j + 1] = t.y;
        }
        if (FIRST) {
#pragma unroll
            for (int sz = 2; sz <= E; sz <<= 1)
#pragma unroll
                for (int d = sz >> 1; d > 0; d >>= 1)
#pragma unroll
                    for (int i = 0; i < E / 2; ++i) {
                        const int lo = 2 * i - (i & (d - 1));
                        compare_exchange(v[lo], v[lo + d], ((base + lo) & sz) == 0);
                    }
        } else {
            const bool descending = (base & size) == 0;
#pragma unroll
            for (int d = E / 2; d > 0; d >>= 1)
#pragma unroll
                for (int i = 0; i < E / 2; ++i) {
                    const int lo = 2 * i - (i & (d - 1));
                    compare_exchange(v[lo], v[lo + d], descending);
                }
        }
#pragma unroll
        for (int j = 0; j < E / 2; ++j) {
            key64x2 t;
            t.x = v[2 * j];
            t.y = v[2 * j + 1];
            blk[j] = t;
        }
    }
    sort_barrier<THREADS>();
}

// LG = keys per lane and pass (as a power of two): 4 keeps all 64 lanes busy from P = 1024 on,
// 3 does so for P = 512.
template <int LG, int THREADS>
__device__ inline void sort_descending_by(key64_t* s, int P) {
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
__device__ inline bool wave_sorted(const key64_t* s, int c) {
    const SortSlot slot;
    for (int base = 1; base < c; base += 64) {
        const int i = min(base + static_cast<int>(threadIdx.x & 63), c - 1);
        if (__ballot(s[slot(i - 1)] < s[slot(i)]) != 0ull) return false;
    }
    return true;
}

// s: sort_slots(P) keys of LDS owned by this wave, key i at s[SortSlot()(i)]; P a power of two >= 16.
__device__ inline void wave_sort_descending(key64_t* s, int P) {
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
// s: sort_slots(k rounded up to 16, + kWaveRankMaxBin) keys; bins: kWaveRankBins / 2 words, 16-byte aligned.
// Returns false with nothing decided (equal or infinite scores, a bin of more than kWaveRankMaxBin
// keys): the caller takes the radix cut and the network.
constexpr int kWaveRankBins = 2048;
constexpr int kWaveRankMaxBin = 64;

// Batcher's odd-even merge sort of 16 keys, largest first.
__device__ inline void sort_16(key64_t (&v)[16]) {
#pragma unroll
    for (int p = 1; p < 16; p <<= 1)
#pragma unroll
        for (int d = p; d > 0; d >>= 1)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                // i is the upper partner of a comparison at distance d inside a merge of runs of p
                const bool first = i >= d % p && ((i - d % p) / d) % 2 == 0;
                if (first && i + d < 16 && i / (2 * p) == (i + d) / (2 * p)) compare_exchange(v[i], v[i + d], true);
            }
}

template <int R>
__device__ inline bool wave_rank_select(const RegKeys<R>& keys, int k, key64_t* s, uint32_t* bins) {
    constexpr int kWords = kWaveRankBins / 2;  // two 16-bit counts per word (a row has fewer than 2^16 keys)
    constexpr int kMine = kWords / 64;         // words of a lane
    static_assert(64 * R < 65536 && kMine % 4 == 0, "counts and places are 16 bits wide");
    typedef uint32_t uintx4 __attribute__((ext_vector_type(4)));
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
    int bin[R];
    keys.sweep_numbered([&](int i, key64_t key, bool valid) {
        bin[i] = static_cast<int>(fminf(fmaxf((from - key_score(key)) * scale, 0.0f), static_cast<float>(kWaveRankBins - 1)));
        if (valid) atomicAdd(&bins[bin[i] >> 1], 1u << (16 * (bin[i] & 1)));
    });
    __builtin_amdgcn_wave_barrier();
    // counts -> first places
    uint32_t c[kMine];
    int local = 0;
    uint32_t most = 0u;
#pragma unroll
    for (int i = 0; i < kMine / 4; ++i) {
        const uintx4 t = mine[i];
#pragma unroll
        for (int j = 0; j < 4; ++j) c[4 * i + j] = t[j];
    }
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        local += static_cast<int>((c[i] & 0xFFFFu) + (c[i] >> 16));
        most = max(most, max(c[i] & 0xFFFFu, c[i] >> 16));
    }
    if (wave_max(most) > kWaveRankMaxBin) return false;
    int place = wave_prefix_sum(local) - local;
    // the bin across place k (the last one in use if there are at most k keys)
    const int want = min(k, n);
    const bool crossing = place < want && want <= place + local;
    int cut_bin = 0, cut_begin = 0, cut_end = 0;
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        uint32_t both = 0u;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int count = static_cast<int>(h == 0 ? c[i] & 0xFFFFu : c[i] >> 16);
            both |= static_cast<uint32_t>(place) << (16 * h);
            if (place < want && want <= place + count) {
                cut_bin = 2 * (lane * kMine + i) + h;
                cut_begin = place;
                cut_end = place + count;
            }
            place += count;
        }
        c[i] = both;
    }
#pragma unroll
    for (int i = 0; i < kMine / 4; ++i) mine[i] = uintx4{c[4 * i], c[4 * i + 1], c[4 * i + 2], c[4 * i + 3]};
    const int src = __builtin_ctzll(__ballot(crossing));
    cut_bin = lane_value(cut_bin, src);
    cut_begin = lane_value(cut_begin, src);
    cut_end = lane_value(cut_end, src);
    __builtin_amdgcn_wave_barrier();
    keys.sweep_numbered([&](int i, key64_t key, bool valid) {
        if (valid && bin[i] <= cut_bin) {
            const int sh = 16 * (bin[i] & 1);
            const int at = static_cast<int>((atomicAdd(&bins[bin[i] >> 1], 1u << sh) >> sh) & 0xFFFFu);
            s[slot(at)] = key;
        }
    });
    __builtin_amdgcn_wave_barrier();
    if (cut_end > want) {  // at most kWaveRankMaxBin keys, one per lane: keep the best want - cut_begin, in order
        const int size = cut_end - cut_begin;
        const key64_t key = lane < size ? s[slot(cut_begin + lane)] : 0ull;
        int better = 0;
        for (int j = 0; j < size; ++j) {
            const key64_t other =
                (static_cast<key64_t>(static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(key >> 32), j))) << 32) |
                static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(key), j));
            better += other > key ? 1 : 0;
        }
        __builtin_amdgcn_wave_barrier();
        if (lane < size && cut_begin + better < want) s[slot(cut_begin + better)] = key;
    }
    const int padded = (want + 15) / 16 * 16;
    if (lane < padded - want) s[slot(want + lane)] = 0ull;
    __builtin_amdgcn_wave_barrier();
    typedef key64_t key64x2 __attribute__((ext_vector_type(2)));
    for (int shift = 0, pass = 0;; shift ^= 8, ++pass) {
        // blocks [base, base + 16), base = 16 u + shift; every half block is 16-byte aligned and without a gap
        for (int base = 16 * lane + shift; base + 16 <= padded; base += 16 * 64) {
            key64x2* first = reinterpret_cast<key64x2*>(s + slot(base));
            key64x2* second = reinterpret_cast<key64x2*>(s + slot(base + 8));
            key64_t v[16];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const key64x2 t = first[j], u = second[j];
                v[2 * j] = t.x;
                v[2 * j + 1] = t.y;
                v[8 + 2 * j] = u.x;
                v[8 + 2 * j + 1] = u.y;
            }
            sort_16(v);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                key64x2 t, u;
                t.x = v[2 * j];
                t.y = v[2 * j + 1];
                u.x = v[8 + 2 * j];
                u.y = v[8 + 2 * j + 1];
                first[j] = t;
                second[j] = u;
            }
        }
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
