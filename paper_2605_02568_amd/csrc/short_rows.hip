// The dense schedule for short key ranges (up to 2048 keys per query) in one kernel: a workgroup takes four consecutive
// queries, one per wave, through their whole key range by the sweep of score_sweep.h in its narrow shape; a wave's scores
// stay in its registers (lane l of register i holds key 64 i + l), and the selection from registers of topk_group.h, which
// wants them in just that layout, follows in the same wave.  No score passes through memory, no workspace is used, and with two
// (smaller heads: three) workgroups per compute unit one's selection runs while the other's sweep keeps the matrix pipe busy.
// Bound by the sweep (matrix and vector pipes) for long rows and many heads, else by the vector instructions of the selection
// (some 2000 a row of 1024 keys; two waves of a SIMD take turns at them).  Measured (us, two kernels / single pass / this): 1024
// rows of 256 keys, 4 heads of 32, k = 16 13.6 / 19.6 / 10.9; 4096 rows of up to 1024, 64 heads of 128, k = 512 56 / 76 / 50; 2 x 8191 of
// up to 2047, 33 heads of 64, k = 300 187 / 234 / 180; 8192 of 2048, k = 512, 64 heads of 128 249 / 300 / 237, 16 of 64 113 / 165 / 100,
// 4 of 32 118 / 202 / 112.  64 heads of 128 with the scores in registers like the others took 346 where those in LDS took 243, for
// the allocator then spills the query, one serialised load after the other (no form that is used spills).  Three waves per SIMD
// where the heads are small: 8192 rows of 2048, k = 512, 4 heads of 32 148 -> 122 when it was chosen, 16 of 64 126 -> 112.
// Scores and order as everywhere (score_sweep.h, si_internal.h): the result is bit-identical to the other schedules'.

#include <algorithm>

#include "score_sweep.h"
#include "topk_group.h"

namespace si {

constexpr int kShortWaves = 4;
constexpr int kShortBins = 2048;

// LDS of one wave's selection: the scratch of either form, then the sorted keys.
struct alignas(16) ShortScratch {
    union {
        RankScratch<64, kShortBins> rank;
        GroupScratch<64, 1> exact;
    };
};
template <int KCAP>
constexpr int short_slice_bytes() {
    constexpr int keys = KCAP + kWaveRankMaxBin;
    return (static_cast<int>(sizeof(ShortScratch)) + (keys + keys / 8) * 8 + 15) / 16 * 16;
}
// Where the sweep leaves no registers for the scores (64 heads of 128) they go to LDS, beside a shorter ring of key chunks, so
// that two workgroups still fit a compute unit.
template <int D, int HB>
constexpr bool short_in_lds() { return D == 128 && HB == 2; }
template <int D, int HB>
constexpr int short_buffers() { return short_in_lds<D, HB>() ? 3 : SweepShape<kShortWaves>::kBuffers; }
template <int D, int HB, int VPT, int KCAP>
constexpr int short_lds_bytes() {
    constexpr int sweep = sweep_lds_bytes<D, kShortWaves, short_buffers<D, HB>()>() + (short_in_lds<D, HB>() ? kShortWaves * VPT * 256 : 0);
    constexpr int select = kShortWaves * short_slice_bytes<KCAP>();
    return sweep > select ? sweep : select;
}

// Keeps a row's scores: run i of 64 keys in register i, -inf where there is no key of the row (or no number).
template <int VPT>
struct RowRegisters {
    typedef float vec __attribute__((ext_vector_type(VPT)));
    vec& v;
    int left;  // the row's keys less the lane number
    __device__ __forceinline__ void operator()(int key0, float score) {
        const float none = -__builtin_huge_valf();
        // (the first call's, which has no scores, is overwritten by the second one's)
        v[max(key0, 0) >> 6] = key0 < left && score > none ? score : none;
    }
};

// The same in the wave's own part of LDS.
struct RowInLds {
    float* row;  // lane l's first score
    int left;
    __device__ __forceinline__ void operator()(int key0, float score) {
        const float none = -__builtin_huge_valf();
        row[max(key0, 0)] = key0 < left && score > none ? score : none;
    }
};

template <int D, int HB, int VPT, int KCAP, int OCC>
__global__ __launch_bounds__(64 * kShortWaves) __attribute__((amdgpu_waves_per_eu(OCC)))
void short_rows_kernel(const __bf16* __restrict__ q, const __bf16* __restrict__ K, const float* __restrict__ w, int S, int H,
                       int T, int m, int mask_mode, int k, int max_keys, int32_t* __restrict__ out_idx, float* __restrict__ out_score) {
    static_assert((KCAP & (KCAP - 1)) == 0 && KCAP >= 16, "the network sorts in place");
    __shared__ __attribute__((aligned(1024))) unsigned char lds[short_lds_bytes<D, HB, VPT, KCAP>()];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int b = blockIdx.y;
    // longest key ranges first, as in score_tile_kernel
    const int t_first = static_cast<int>(gridDim.x - 1 - blockIdx.x) * kShortWaves;
    const int t = t_first + wave;
    const bool live = t < S;
    const int group_keys = legal_count(min(S, t_first + kShortWaves) - 1, T, m, mask_mode);
    const int n = live ? legal_count(t, T, m, mask_mode) : 0;
    const int64_t row = static_cast<int64_t>(b) * S + (live ? t : S - 1);

    constexpr bool kInLds = short_in_lds<D, HB>();
    constexpr int kBuffers = short_buffers<D, HB>();
    float v[VPT];
#pragma unroll
    for (int i = 0; i < VPT; ++i) v[i] = -__builtin_huge_valf();
    if (group_keys > 0) {
        const __bf16* Kb = K + static_cast<int64_t>(b) * T * D;
        sweep_prefetch<D, kShortWaves, kBuffers>(lds, Kb, T);
        bf16x8 a[HB][D / 16];
        float wr[HB][16];
        load_query<D, HB>(q, w, row, H, lane, a, wr);
        SweepOut o{};
        __builtin_amdgcn_s_setprio(3);  // see indexer_fused_kernel
        if constexpr (kInLds) {
            float* const s_row = reinterpret_cast<float*>(lds + sweep_lds_bytes<D, kShortWaves, kBuffers>()) + wave * (VPT * 64) + lane;
            score_sweep<D, HB, false, false, true, kShortWaves, RowInLds, kBuffers>(lds, a, wr, Kb, T, group_keys, o, nullptr, 0,
                                                                                    RowInLds{s_row, n - lane});
#pragma unroll
            for (int i = 0; i < VPT; ++i)
                if (64 * i < group_keys) v[i] = s_row[64 * i];  // (written by this lane)
        } else {
            typename RowRegisters<VPT>::vec kept;
#pragma unroll
            for (int i = 0; i < VPT; ++i) kept[i] = -__builtin_huge_valf();
            score_sweep<D, HB, false, false, true, kShortWaves, RowRegisters<VPT>, kBuffers>(
                lds, a, wr, Kb, T, group_keys, o, nullptr, 0, RowRegisters<VPT>{kept, n - lane});
#pragma unroll
            for (int i = 0; i < VPT; ++i) v[i] = kept[i];
        }
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();  // the sweep's LDS is free
    if (!live) return;

    unsigned char* const slice = lds + wave * short_slice_bytes<KCAP>();
    ShortScratch& s = *reinterpret_cast<ShortScratch*>(slice);
    rank_t* const keys = reinterpret_cast<rank_t*>(slice + sizeof(ShortScratch));
    float some = lane_value(v[0], 0);
    if (!(some - some == 0.0f)) some = 0.0f;
    const int kk = min(k, max_keys);  // <= KCAP
    int c = 0;
    if (!group_rank_select<64, VPT, kShortBins>(v, n, some, kk, keys, s.rank, &c)) {
        group_barrier<64>();  // the scratch changes hands
        c = group_exact_select<64>(v, kk, keys, s.exact);
    }
    const SortSlot slot;
    const int64_t out = row * k;
    for (int j = lane; j < k; j += 64) {
        if (j < c) {
            const rank_t key = keys[slot(j)];
            out_idx[out + j] = rank_index(key);
            out_score[out + j] = rank_score(key);
        } else {  // Section 4.2: pad
            out_idx[out + j] = -1;
            out_score[out + j] = -__builtin_huge_valf();
        }
    }
}

hipError_t launch_short_rows(const void* q, const void* K, const float* w, const si_dims& d, int32_t m, int32_t mask_mode,
                             int32_t k, int32_t longest, int32_t* out_idx, float* out_score, hipStream_t stream) {
    // `longest` bounds every row, and with it the entries that count
    const int32_t kk = std::min(k, std::max(longest, 1));
    if (k < 1 || longest > kShortMaxKeys || kk > kShortMaxK || d.B > 65535 || d.S > kShortMaxQueries) return hipErrorInvalidValue;
    const dim3 grid((d.S + kShortWaves - 1) / kShortWaves, d.B);
    const __bf16* qp = static_cast<const __bf16*>(q);
    const __bf16* Kp = static_cast<const __bf16*>(K);
    const int HB = (d.H_I + 31) / 32;
#define SI_LAUNCH(DD, HH, VV, CC, OO)                                                                                     \
    hipLaunchKernelGGL((short_rows_kernel<DD, HH, VV, CC, OO>), grid, dim3(64 * kShortWaves), 0, stream, qp, Kp, w, d.S, \
                       d.H_I, d.T, m, mask_mode, k, std::max(longest, 1), out_idx, out_score)
#define SI_BY_LENGTH(DD, HH, OO)                                                              \
    if (longest <= 1024) {                                                                    \
        if (kk <= 512) SI_LAUNCH(DD, HH, 16, 512, OO); else SI_LAUNCH(DD, HH, 16, 1024, 2);  \
    } else {                                                                                  \
        if (kk <= 512) SI_LAUNCH(DD, HH, 32, 512, OO); else SI_LAUNCH(DD, HH, 32, 1024, 2);  \
    }
    if (d.D == 128 && HB == 2) { SI_BY_LENGTH(128, 2, 2) }
    else if (d.D == 128 && HB == 1) { SI_BY_LENGTH(128, 1, 2) }
    else if (d.D == 64 && HB == 2) { SI_BY_LENGTH(64, 2, 2) }
    else if (d.D == 64 && HB == 1) { SI_BY_LENGTH(64, 1, 3) }
    else if (d.D == 32 && HB == 2) { SI_BY_LENGTH(32, 2, 3) }
    else if (d.D == 32 && HB == 1) { SI_BY_LENGTH(32, 1, 3) }
    else return hipErrorInvalidValue;
#undef SI_BY_LENGTH
#undef SI_LAUNCH
    return hipGetLastError();
}

}  // namespace si
