// The consumer of the index lists (Section 3, step 4): sparse attention of every query over
// U(t) = TopK(t) U Window(t), where the keys and the values are the rows of the compressed cache K_C
// (Section 3, step 1), TopK(t) is the query's index list as si_indexer_topk writes it (pads = -1)
// and Window(t) is the last min(n_win, legal(t)) legal keys (Section 4.2 for legal(t)):
//
//   out[t,h,:] = sum_{s in U(t)} p_s K_C[s,:],   p = softmax_{s in U(t)}( scale * <qa[t,h,:], K_C[s,:]> )
//
// and out = 0 where U(t) is empty.  The paper names this step and gives no formula; the reading is
// spelled out in the public header.
//
// Mapping (gfx950, wave64).  One workgroup = one query; its waves split the heads, 32 per wave, and
// share the gathered key rows.  The rows of U(t) are gathered 32 at a time (a tile) straight from
// global memory into LDS (global_load ... lds, no register round trip), row-major and XOR-swizzled
// like the indexer's key chunks, two tiles in flight.  Per tile and wave:
//   S^T[32 keys x 32 heads] = Ktile . q^T     v_mfma_f32_32x32x16_bf16, keys on the M side: each lane
//                                             then holds 16 keys of ONE head, so the softmax
//                                             statistics of a head are in-lane (+ one lane^32 exchange)
//   p = exp2(x - m_ref)                       running reference maximum per head, raised (and the
//                                             accumulators rescaled) only when a tile exceeds it by
//                                             more than 2^8; fp32
//   O^T[D x 32 heads] += Vtile^T . P^T        P^T is the B operand straight from the S^T registers
//                                             (the contraction order over the tile's keys is permuted
//                                             the same way on both operands); Vtile^T, a column access
//                                             of the row-major tile, comes from the transposing LDS
//                                             read ds_read_b64_tr_b16.  p is split into two bf16
//                                             (high part + remainder) and multiplied twice, so the
//                                             weights carry 16 mantissa bits, not 8.
// The denominator is accumulated in fp32 from the unsplit p and divides O^T at the end.
// Few queries take sparse_attention_few_kernel, which spreads a query over more waves with the same order of every sum.

#include <hip/hip_runtime.h>

#include <algorithm>
#include <atomic>
#include <type_traits>

#include "si_internal.h"
#include "streamindex_attention.h"

namespace si {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

constexpr int kTileKeys = 32;        // keys per gathered tile
constexpr float kRescaleSlack = 8.0f;  // log2 units a tile may exceed the reference maximum

// LDS slot (16-byte unit inside the tile) of piece `piece` (8 elements) of tile row `row`.
// Rows are unpadded (2*D bytes); the pieces of a row are XOR-swizzled with a number made of the row's, so that lanes served
// together hit different bank groups.  D = 128: eight consecutive rows get eight different numbers modulo 8 for the row reads of the
// first product (16 bytes from each of 8 rows), and four consecutive rows four that differ above the lowest bit for the transposing
// reads of the second one (two neighbouring pieces from each of 4 rows).  With the row number itself, where rows 2 i and 2 i + 1 share
// two pieces' banks, 16384 queries, k = 512 + 128, 64 heads had 56.6 M conflict cycles instead of 18.9 M; decoding, whose chain
// the reads are part of, took 2 to 4 % longer.  D = 64, two rows to the 64 banks: half the row number (the other form: 289 -> 308 us).
template <int D>
__device__ __forceinline__ int row_swizzle(int row) {
    return D == 128 ? ((row & 3) << 1) | ((row >> 2) & 1) | (row & 8) : (row >> 1) % (D / 8);
}
template <int D>
__device__ __forceinline__ int tile_slot(int row, int piece) {
    return row * (D / 8) + (piece ^ row_swizzle<D>(row));
}

// The value lane (l ^ 32) holds, by v_permlane32_swap instead of an LDS round trip: of the swap's two
// results one carries the low half-wave's values in both halves, the other the high half-wave's;
// each lane picks the one that is not its own.
__device__ __forceinline__ float other_half(float v) {
    const unsigned bits = __builtin_bit_cast(unsigned, v);
    const auto both = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
    return __builtin_bit_cast(float, (threadIdx.x & 32) ? both[0] : both[1]);
}

// U(t) into s_list: the list's entries outside the window (they are valid and distinct by contract), in list order,
// then the window [w0, legal), padded to whole tiles with key 0; returns their number.  The workgroup's W waves take an
// equal share of the list, up to 512 entries each and round, all requested before the first is used: one trip to
// memory, where one wave taking 64 at a time made k / 64 (16384 queries, k = 512: 495 -> 484 us; without
// the exchange of counts, every wave going through the whole list: 497).  s_kept: W ints.
template <int W>
__device__ __forceinline__ int build_list(const int32_t* __restrict__ row, int k, int w0, int legal, int* s_list, int* s_kept) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    int n = 0;
    constexpr int kPer = 8;
    const int per = min(kPer, (k + 64 * W - 1) / (64 * W));  // runs of 64 entries a wave takes in a round
    const bool one_run = k <= 64;  // every wave counts it by itself, and wave 0 stores it
    for (int j0 = 0; j0 < k; j0 += W * per * 64) {
        const int first = j0 + (one_run ? 0 : wave * (per * 64)) + lane;
        int s[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (i < per) s[i] = row[min(first + 64 * i, k - 1)];
        unsigned long long kept[kPer];
        int mine = 0;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            kept[i] = 0ull;
            if (i < per) kept[i] = __ballot(first + 64 * i < k && s[i] >= 0 && !(s[i] >= w0 && s[i] < legal));
            mine += static_cast<int>(__popcll(kept[i]));
        }
        int pos = n, total = mine;
        if (W > 1 && !one_run) {
            if (j0 > 0) __syncthreads();  // the previous round's counts have been read
            if (lane == 0) s_kept[wave] = mine;
            __syncthreads();
            total = 0;
#pragma unroll
            for (int i = 0; i < W; ++i) {
                const int c = s_kept[i];
                pos += i < wave ? c : 0;
                total += c;
            }
        }
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const int below = __builtin_amdgcn_mbcnt_hi(static_cast<unsigned>(kept[i] >> 32),
                              __builtin_amdgcn_mbcnt_lo(static_cast<unsigned>(kept[i]), 0u));
            if (((kept[i] >> lane) & 1) && (!one_run || wave == 0)) s_list[pos + below] = s[i];
            pos += static_cast<int>(__popcll(kept[i]));
        }
        n += total;
    }
    for (int s = w0 + static_cast<int>(threadIdx.x); s < legal; s += 64 * W) s_list[n + (s - w0)] = s;
    n += legal - w0;
    const int padded = (n + kTileKeys - 1) / kTileKeys * kTileKeys;
    for (int j = n + static_cast<int>(threadIdx.x); j < padded; j += 64 * W) s_list[j] = 0;
    return n;
}

// One workgroup = one query and HW waves of 64 lanes; wave w owns heads [32 w, 32 w + 32) and all waves share each
// gathered tile.
// Dynamic LDS: 2 tiles of 32 x D bf16, then the query's key list (k + n_win ints, padded to a tile).
// Two waves per SIMD are asked for explicitly: with a register budget of 256 the compiler keeps the
// accumulators in ordinary VGPRs; left to a budget of 512 it parks them in AGPRs and copies all 64
// of them out and back around the rescale test of every tile.
template <int D, int HW>
__global__ __launch_bounds__(64 * HW) __attribute__((amdgpu_waves_per_eu(2)))
void sparse_attention_kernel(const __bf16* __restrict__ qa, const __bf16* __restrict__ Kc,
                             const int32_t* __restrict__ idx, int S, int H, int T, int m, int mask_mode,
                             int k, int n_win, float scale_log2e, float* __restrict__ out) {
    constexpr int KS = D / 16;                 // MFMA steps along d in the first product
    constexpr int DB = D / 32;                 // 32-row blocks of O^T
    constexpr int kRowBytes = D * 2;
    constexpr int kPieces = D / 8;             // 16-byte pieces per key row
    constexpr int kTileBytes = kTileKeys * kRowBytes;
    constexpr int kLoadsPerWave = kTileBytes / 1024 / HW;  // wave-wide 1 KiB gathers per wave and tile
    static_assert(kTileBytes % (1024 * HW) == 0 && kLoadsPerWave >= 1, "a tile must split over the waves");
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    int* const s_list = reinterpret_cast<int*>(lds + 2 * kTileBytes);
    __shared__ int s_kept[HW];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int col = lane & 31;
    const int half = lane >> 5;
    const int64_t row_q = blockIdx.x;          // b * S + t
    const int b = static_cast<int>(row_q / S);
    const int t = static_cast<int>(row_q % S);
    const int legal = legal_count(t, T, m, mask_mode);
    const int w0 = max(0, legal - n_win);      // Window(t) = [w0, legal)
    const int n = build_list<HW>(idx + row_q * k, k, w0, legal, s_list, s_kept);
    __syncthreads();
    const int n_u = __builtin_amdgcn_readfirstlane(n);
    const int64_t out_base = (row_q * H) * D;
    if (n_u == 0) {  // empty set: zeros (uniform over the workgroup)
        for (int i = threadIdx.x; i < H * D; i += 64 * HW) out[out_base + i] = 0.0f;
        return;
    }
    const int n_tiles = (n_u + kTileKeys - 1) / kTileKeys;
    const __bf16* Kb = Kc + static_cast<int64_t>(b) * T * D;

    // ---- gather of one tile: wave w brings rows [rows_per_wave * w, ...) of the tile
    typedef __attribute__((address_space(3))) void lds_void;
    typedef __attribute__((address_space(1))) const void gbl_void;
    auto gather = [&](int tile, int buf) {
        int key[kLoadsPerWave];  // all of this lane's list entries first: one LDS round trip, not one per load
#pragma unroll
        for (int i = 0; i < kLoadsPerWave; ++i) {
            const int unit = (wave * kLoadsPerWave + i) * 64 + lane;  // 16-byte LDS slot this lane fills
            key[i] = s_list[tile * kTileKeys + unit / kPieces];
        }
#pragma unroll
        for (int i = 0; i < kLoadsPerWave; ++i) {
            const int blk = wave * kLoadsPerWave + i;         // 1 KiB block of the tile
            const int unit = blk * 64 + lane;
            const int r = unit / kPieces;                      // tile row
            const int slot = unit % kPieces;
            const int piece = slot ^ row_swizzle<D>(r);
            const char* src = reinterpret_cast<const char*>(Kb) + static_cast<int64_t>(key[i]) * kRowBytes + piece * 16;
            __builtin_amdgcn_global_load_lds((gbl_void*)src, (lds_void*)(lds + buf * kTileBytes + blk * 1024), 16, 0, 0);
        }
    };
    gather(0, 0);

    // ---- this wave's query operand: head = 32*wave + col, 8 consecutive d at 16*ks + 8*half
    bf16x8 qf[KS];
    {
        const int h = min(32 * wave + col, H - 1);
        const __bf16* src = qa + (row_q * H + h) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(src + ks * 16);
    }

    // A negative scale goes into the query operand: flipping the sign bit of a bf16 is exact, every
    // product and partial sum changes sign and nothing else, so the scores are those of (-q, -scale).
    if (scale_log2e < 0.0f) {
        typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
            qf[ks] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(uintx4, qf[ks]) ^ 0x80008000u);
        scale_log2e = -scale_log2e;
    }
    // LDS byte offsets that do not depend on the tile: first product, row = col, piece 2 ks + half
    int ka[KS];
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ka[ks] = tile_slot<D>(col, 2 * ks + half) * 16;
    // second product: this lane is source lane s = lane % 16 of its 16-lane group G = lane / 16 for the
    // transposing read; the group serves d rows [32 db + 16 (G % 2), +16) and the keys of half G / 2.
    // Source lane s points at 4 consecutive d (8 bytes) of key row 4 (G / 2) + s / 4 (+ 8 for the
    // second read, + 16 u), at d = 32 db + 16 (G % 2) + 4 (s % 4).
    int va[DB][2];
    {
        const int G = lane >> 4, s = lane & 15;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int r = 8 * w + 4 * (G >> 1) + (s >> 2);
                const int d = 32 * db + 16 * (G & 1) + 4 * (s & 3);
                va[db][w] = tile_slot<D>(r, d / 8) * 16 + ((d % 8) / 4) * 8;
            }
    }

    floatx16 acc[DB];
    const floatx16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = zero16;
    float m_ref = -__builtin_huge_valf();  // reference maximum of this lane's head (log2 domain)
    float l_sum = 0.0f;                    // sum of p over this half-wave's keys

    // One tile; the buffer index is a compile-time constant so that every LDS address of the tile is
    // a loop-invariant register plus an immediate offset.
    auto step = [&](int tile, auto buf_tag) {
        constexpr int buf = decltype(buf_tag)::value;
        // tile `tile` has landed for every wave; everyone is done with tile - 1, whose buffer the next
        // gather overwrites
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
        __syncthreads();
        if (tile + 1 < n_tiles) gather(tile + 1, buf ^ 1);
        const unsigned char* tb = lds + buf * kTileBytes;

        // S^T = Ktile . q^T : register j of a lane = key row 8 (j / 4) + 4 half + j % 4, head = col
        floatx16 sacc = zero16;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            const bf16x8 kf = *reinterpret_cast<const bf16x8*>(tb + ka[ks]);
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sacc, 0, 0, 0);
        }
        // The scale is >= 0 here (a negative one was moved into the query operand), so the largest scaled
        // score is the largest raw one times the scale, and scale and reference go into one fma per key.
        const bool ragged = tile == n_tiles - 1 && n_u < n_tiles * kTileKeys;  // rows past the end of U(t): rare
        if (ragged) {
            float low = -3.0e38f;
            asm volatile("" : "+v"(low));  // keeps this block a branch instead of 16 selects per tile
            const int live = n_u - tile * kTileKeys;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (8 * (j >> 2) + 4 * half + (j & 3) >= live) sacc[j] = low;  // out of the maximum; weight zeroed below
        }
        float smax = sacc[0];
#pragma unroll
        for (int j = 1; j < 16; ++j) smax = fmaxf(smax, sacc[j]);
        float tmax = smax * scale_log2e;
        tmax = fmaxf(tmax, other_half(tmax));  // the tile's maximum for this head (finite: row 0 of a tile is live)
        const bool raise = tmax > m_ref + kRescaleSlack;
        if (__ballot(raise) != 0ull) {  // rare after the first tiles
            const float m_new = raise ? tmax : m_ref;
            const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new);  // 1 where nothing changes, 0 on the first tile
#pragma unroll
            for (int db = 0; db < DB; ++db)
#pragma unroll
                for (int j = 0; j < 16; ++j) acc[db][j] *= alpha;
            l_sum *= alpha;
            m_ref = m_new;
        }
        float p[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) p[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[j], scale_log2e, -m_ref));
        if (ragged) {
            float none = 0.0f;
            asm volatile("" : "+v"(none));
            const int live = n_u - tile * kTileKeys;
#pragma unroll
            for (int j = 0; j < 16; ++j)
                if (8 * (j >> 2) + 4 * half + (j & 3) >= live) p[j] = none;
        }
        // weights as two bf16 parts, two keys per conversion: hi = bf16(p), lo = bf16(p - hi)
        typedef float floatx2 __attribute__((ext_vector_type(2)));
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
        uintx4 hi_bits[2], lo_bits[2];
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            const float p0 = p[2 * jj], p1 = p[2 * jj + 1];
            l_sum += p0 + p1;
            const unsigned hb = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{p0, p1}, bf16x2));
            const float r0 = p0 - __builtin_bit_cast(float, hb << 16);
            const float r1 = p1 - __builtin_bit_cast(float, hb & 0xFFFF0000u);
            hi_bits[jj >> 2][jj & 3] = hb;
            lo_bits[jj >> 2][jj & 3] = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{r0, r1}, bf16x2));
        }
        bf16x8 p_hi[2], p_lo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            p_hi[u] = __builtin_bit_cast(bf16x8, hi_bits[u]);
            p_lo[u] = __builtin_bit_cast(bf16x8, lo_bits[u]);
        }
        // O^T += Vtile^T . P^T : contraction index e of step u <-> tile row 16 u + 8 (e / 4) + 4 half + e % 4
        // on both operands
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int db = 0; db < DB; ++db) {
                typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
                const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    (lds_bf16x4*)(tb + va[db][0] + u * 16 * kRowBytes));
                const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16(
                    (lds_bf16x4*)(tb + va[db][1] + u * 16 * kRowBytes));
                const bf16x8 vf = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p_hi[u], acc[db], 0, 0, 0);
                acc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, p_lo[u], acc[db], 0, 0, 0);
            }
    };
    for (int tile = 0; tile < n_tiles; tile += 2) {
        step(tile, std::integral_constant<int, 0>{});
        if (tile + 1 < n_tiles) step(tile + 1, std::integral_constant<int, 1>{});
    }

    // ---- out[t, head, d] = O^T[d, head] / l : register j of block db = d row 32 db + 8 (j / 4) + 4 half + j % 4
    const float l_all = l_sum + other_half(l_sum);
    const float inv = 1.0f / l_all;
    const int h = 32 * wave + col;
    if (h < H) {
        float* o = out + out_base + static_cast<int64_t>(h) * D;
#pragma unroll
        for (int db = 0; db < DB; ++db)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const floatx4 v = {acc[db][4 * a] * inv, acc[db][4 * a + 1] * inv, acc[db][4 * a + 2] * inv,
                                   acc[db][4 * a + 3] * inv};
                *reinterpret_cast<floatx4*>(o + 32 * db + 8 * a + 4 * half) = v;
            }
    }
}

// Few queries, which would leave most of the chip idle and walk their 20 to 40 tiles one after the other: a workgroup
// takes one query and one block of 32 heads (grid: queries x head blocks) and spreads the work of a tile over its
// waves without changing the order of any sum, so that a query's result does not depend on how many queries
// share the call (the bits are those of sparse_attention_kernel):
//   4 score waves    one tile each of a group of four: gather, S^T, the tile's maxima; then, with the maxima of the
//                    whole group, the reference maximum each tile meets, its weights to LDS as matrix operands, and the
//                    sums of weight pairs
//   D / 32 value waves  one block of 32 d each: all tiles in list order, rescaling, denominator and second product.
// The value waves work on the group before the score waves', with two barriers per group.  Bound by the score waves' chain of
// dependent steps, about 3000 cycles a group: two groups of gathers on their way, value rows read ahead, and half
// the value waves with two blocks each (a third less LDS traffic) all changed nothing.
// Dynamic LDS: 3 groups of tiles (one multiplied, one scored, one on its way), the operands and pair sums of a group, two
// groups' maxima, the key list.
constexpr int kGroupTiles = 4;
template <int D>
constexpr int few_lds_bytes() { return 3 * kGroupTiles * kTileKeys * D * 2 + kGroupTiles * (4096 + 2048) + 2 * kGroupTiles * 32 * 4; }
template <int D>
__global__ __launch_bounds__(64 * (kGroupTiles + D / 32)) __attribute__((amdgpu_waves_per_eu(2)))
void sparse_attention_few_kernel(const __bf16* __restrict__ qa, const __bf16* __restrict__ Kc,
                                 const int32_t* __restrict__ idx, int S, int H, int T, int m, int mask_mode,
                                 int k, int n_win, int head_blocks, float scale_log2e, float* __restrict__ out) {
    constexpr int G = kGroupTiles;
    constexpr int W = G + D / 32;
    constexpr int KS = D / 16;
    constexpr int kRowBytes = D * 2;
    constexpr int kPieces = D / 8;
    constexpr int kTileBytes = kTileKeys * kRowBytes;
    constexpr int kLoads = kTileBytes / 1024;
    typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
    extern __shared__ __attribute__((aligned(1024))) unsigned char lds[];
    unsigned char* const s_weights = lds + 3 * G * kTileBytes;                // [G][hi 0, hi 1, lo 0, lo 1][64 lanes] 16 bytes
    unsigned char* const s_pairs = s_weights + G * 4096;                      // [G][2][64 lanes] 16 bytes
    float* const s_max = reinterpret_cast<float*>(s_pairs + G * 2048);        // [2][G][32 heads]
    int* const s_list = reinterpret_cast<int*>(lds + few_lds_bytes<D>());
    __shared__ int s_kept[W];

    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int col = lane & 31;
    const int half = lane >> 5;
    const int64_t row_q = blockIdx.x / head_blocks;  // b * S + t
    const int h0 = 32 * static_cast<int>(blockIdx.x % head_blocks);
    const int b = static_cast<int>(row_q / S);
    const int t = static_cast<int>(row_q % S);
    const int legal = legal_count(t, T, m, mask_mode);
    const int w0 = max(0, legal - n_win);
    const int n = build_list<W>(idx + row_q * k, k, w0, legal, s_list, s_kept);
    __syncthreads();
    const int n_u = __builtin_amdgcn_readfirstlane(n);
    const int64_t out_base = (row_q * H) * D;
    if (n_u == 0) {
        for (int i = h0 * D + static_cast<int>(threadIdx.x); i < min(H, h0 + 32) * D; i += 64 * W) out[out_base + i] = 0.0f;
        return;
    }
    const int n_tiles = (n_u + kTileKeys - 1) / kTileKeys;
    const int n_groups = (n_tiles + G - 1) / G;
    const floatx16 zero16 = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    float m_ref = -__builtin_huge_valf();  // reference maximum of this lane's head (log2 domain)

    // A barrier that leaves the gathers in flight (they are waited for by the wave that issued them, before it
    // scores the tile, a barrier ahead of anybody else's use); LDS accesses are done on both sides.
#define SI_GROUP_BARRIER()                       \
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); \
    __builtin_amdgcn_s_barrier();                \
    asm volatile("" ::: "memory");
    // The next tile's maximum TMAX against the reference: SCALE(alpha) runs where some head of the block is raised.
#define SI_RAISE(TMAX, SCALE)                                                       \
    {                                                                               \
        const float tmax_ = (TMAX);                                                 \
        const bool raise_ = tmax_ > m_ref + kRescaleSlack;                          \
        if (__ballot(raise_) != 0ull) {                                             \
            const float m_new_ = raise_ ? tmax_ : m_ref;                            \
            const float alpha = __builtin_amdgcn_exp2f(m_ref - m_new_);             \
            SCALE                                                                   \
            m_ref = m_new_;                                                         \
        }                                                                           \
    }
    if (wave < G) {
        const __bf16* Kb = Kc + static_cast<int64_t>(b) * T * D;
        typedef __attribute__((address_space(3))) void lds_void;
        typedef __attribute__((address_space(1))) const void gbl_void;
        auto gather = [&](int tile, unsigned char* dst) {
            int key[kLoads];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) key[i] = s_list[tile * kTileKeys + (i * 64 + lane) / kPieces];
#pragma unroll
            for (int i = 0; i < kLoads; ++i) {
                const int unit = i * 64 + lane;
                const int r = unit / kPieces;
                const int piece = (unit % kPieces) ^ row_swizzle<D>(r);
                const char* src = reinterpret_cast<const char*>(Kb) + (static_cast<int64_t>(key[i]) * kRowBytes + piece * 16);
                __builtin_amdgcn_global_load_lds((gbl_void*)src, (lds_void*)(dst + i * 1024), 16, 0, 0);
            }
        };
        if (wave < n_tiles) gather(wave, lds + wave * kTileBytes);
        bf16x8 qf[KS];
        const __bf16* src = qa + (row_q * H + min(h0 + col, H - 1)) * D + half * 8;
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) qf[ks] = *reinterpret_cast<const bf16x8*>(src + ks * 16);
        if (scale_log2e < 0.0f) {  // exact: see sparse_attention_kernel
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                qf[ks] = __builtin_bit_cast(bf16x8, __builtin_bit_cast(uintx4, qf[ks]) ^ 0x80008000u);
            scale_log2e = -scale_log2e;
        }
        int ka[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ka[ks] = tile_slot<D>(col, 2 * ks + half) * 16;

        int buf = 0;  // group g is in buffer g % 3
        for (int g = 0; g < n_groups; ++g) {
            const int tile = g * G + wave;
            const bool mine = tile < n_tiles;
            const unsigned char* tb = lds + (buf * G + wave) * kTileBytes;
            buf = buf == 2 ? 0 : buf + 1;
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // this wave's tile has landed
            // (the value waves left the buffer of group g - 2 at the last barrier)
            if (tile + G < n_tiles) gather(tile + G, lds + (buf * G + wave) * kTileBytes);
            floatx16 sacc = zero16;
            const bool ragged = tile == n_tiles - 1 && n_u < n_tiles * kTileKeys;
            const int live = n_u - tile * kTileKeys;
            if (mine) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    const bf16x8 kf = *reinterpret_cast<const bf16x8*>(tb + ka[ks]);
                    sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[ks], sacc, 0, 0, 0);
                }
                if (ragged) {
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (8 * (j >> 2) + 4 * half + (j & 3) >= live) sacc[j] = -3.0e38f;
                }
                float smax = sacc[0];
#pragma unroll
                for (int j = 1; j < 16; ++j) smax = fmaxf(smax, sacc[j]);
                float tmax = smax * scale_log2e;
                tmax = fmaxf(tmax, other_half(tmax));
                if (half == 0) s_max[((g & 1) * G + wave) * 32 + col] = tmax;
            }
            SI_GROUP_BARRIER()
            float m_tile = m_ref;
#pragma unroll
            for (int i = 0; i < G; ++i)
                if (g * G + i < n_tiles) {
                    SI_RAISE(s_max[((g & 1) * G + i) * 32 + col], (void)alpha;)
                    if (i == wave) m_tile = m_ref;
                }
            if (mine) {
                float p[16];
#pragma unroll
                for (int j = 0; j < 16; ++j) p[j] = __builtin_amdgcn_exp2f(__builtin_fmaf(sacc[j], scale_log2e, -m_tile));
                if (ragged) {
#pragma unroll
                    for (int j = 0; j < 16; ++j)
                        if (8 * (j >> 2) + 4 * half + (j & 3) >= live) p[j] = 0.0f;
                }
                typedef float floatx2 __attribute__((ext_vector_type(2)));
                typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
                uintx4 hi_bits[2], lo_bits[2];
                floatx4 pairs[2];
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) {
                    const float p0 = p[2 * jj], p1 = p[2 * jj + 1];
                    pairs[jj >> 2][jj & 3] = p0 + p1;
                    const unsigned hb = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{p0, p1}, bf16x2));
                    const float r0 = p0 - __builtin_bit_cast(float, hb << 16);
                    const float r1 = p1 - __builtin_bit_cast(float, hb & 0xFFFF0000u);
                    hi_bits[jj >> 2][jj & 3] = hb;
                    lo_bits[jj >> 2][jj & 3] = __builtin_bit_cast(unsigned, __builtin_convertvector(floatx2{r0, r1}, bf16x2));
                }
                uintx4* wt = reinterpret_cast<uintx4*>(s_weights + wave * 4096) + lane;
                wt[0] = hi_bits[0];
                wt[64] = hi_bits[1];
                wt[128] = lo_bits[0];
                wt[192] = lo_bits[1];
                floatx4* pr = reinterpret_cast<floatx4*>(s_pairs + wave * 2048) + lane;
                pr[0] = pairs[0];
                pr[64] = pairs[1];
            }
            SI_GROUP_BARRIER()
        }
        SI_GROUP_BARRIER()  // the value waves' last group has two barriers as well
        SI_GROUP_BARRIER()
    } else {
        const int db = wave - G;
        int va[2];  // see sparse_attention_kernel
        {
            const int Gr = lane >> 4, s = lane & 15;
#pragma unroll
            for (int w = 0; w < 2; ++w) {
                const int r = 8 * w + 4 * (Gr >> 1) + (s >> 2);
                const int d = 32 * db + 16 * (Gr & 1) + 4 * (s & 3);
                va[w] = tile_slot<D>(r, d / 8) * 16 + ((d % 8) / 4) * 8;
            }
        }
        floatx16 acc = zero16;
        float l_sum = 0.0f;
        SI_GROUP_BARRIER()  // the score waves' first group
        SI_GROUP_BARRIER()
        int buf = 0;
        for (int g = 0; g < n_groups; ++g) {
            const unsigned char* group = lds + buf * G * kTileBytes;
            buf = buf == 2 ? 0 : buf + 1;
            // the group's operands, sums and maxima to registers: the score waves overwrite the first two after the barrier
            uintx4 wt[G][4];
            floatx4 pairs[G][2];
            float tmax[G];
#pragma unroll
            for (int i = 0; i < G; ++i) {
#pragma unroll
                for (int j = 0; j < 4; ++j) wt[i][j] = reinterpret_cast<const uintx4*>(s_weights + i * 4096)[64 * j + lane];
#pragma unroll
                for (int j = 0; j < 2; ++j) pairs[i][j] = reinterpret_cast<const floatx4*>(s_pairs + i * 2048)[64 * j + lane];
                tmax[i] = s_max[((g & 1) * G + i) * 32 + col];
            }
#pragma unroll
            for (int i = 0; i < G; ++i) {
                if (i == G / 2) { SI_GROUP_BARRIER() }
                if (g * G + i >= n_tiles) continue;  // uniform
                SI_RAISE(tmax[i], {
                    _Pragma("unroll") for (int j = 0; j < 16; ++j) acc[j] *= alpha;
                    l_sum *= alpha;
                })
#pragma unroll
                for (int jj = 0; jj < 8; ++jj) l_sum += pairs[i][jj >> 2][jj & 3];
                const unsigned char* tb = group + i * kTileBytes;
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
                    const bf16x4 v0 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(tb + va[0] + u * 16 * kRowBytes));
                    const bf16x4 v1 = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4*)(tb + va[1] + u * 16 * kRowBytes));
                    const bf16x8 vf = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, wt[i][u]), acc, 0, 0, 0);
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf, __builtin_bit_cast(bf16x8, wt[i][2 + u]), acc, 0, 0, 0);
                }
            }
            SI_GROUP_BARRIER()
        }
        const float l_all = l_sum + other_half(l_sum);
        const float inv = 1.0f / l_all;
        const int h = h0 + col;
        if (h < H) {
            float* o = out + out_base + static_cast<int64_t>(h) * D + 32 * db;
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const floatx4 v = {acc[4 * a] * inv, acc[4 * a + 1] * inv, acc[4 * a + 2] * inv, acc[4 * a + 3] * inv};
                *reinterpret_cast<floatx4*>(o + 8 * a + 4 * half) = v;
            }
        }
    }
#undef SI_RAISE
#undef SI_GROUP_BARRIER
}

size_t list_bytes(int k, int n_win) {
    return static_cast<size_t>((k + n_win + kTileKeys - 1) / kTileKeys * kTileKeys) * sizeof(int);
}

// Raises the dynamic LDS limit of a kernel once per device and size (as in the write-out kernel).
template <typename Kernel>
hipError_t allow_lds(Kernel kernel, size_t bytes, std::atomic<size_t>* allowed) {
    if (bytes <= 48 * 1024) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool tracked = dev >= 0 && dev < 64;
    if (tracked && allowed[dev].load(std::memory_order_acquire) >= bytes) return hipSuccess;
    e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                            static_cast<int>(bytes));
    if (e == hipSuccess && tracked) {
        size_t seen = allowed[dev].load(std::memory_order_relaxed);
        while (seen < bytes && !allowed[dev].compare_exchange_weak(seen, bytes, std::memory_order_release)) {}
    }
    return e;
}

template <int D, int HW>
hipError_t launch(const __bf16* qa, const __bf16* Kc, const int32_t* idx, const si_dims& d, int32_t m,
                  int32_t mask_mode, int32_t k, int32_t n_win, float scale, float* out, hipStream_t stream) {
    static std::atomic<size_t> allowed[64];
    const size_t lds = 2 * static_cast<size_t>(kTileKeys) * D * 2 + list_bytes(k, n_win);
    hipError_t e = allow_lds(sparse_attention_kernel<D, HW>, lds, allowed);
    if (e != hipSuccess) return e;
    const int64_t rows = static_cast<int64_t>(d.B) * d.S;
    hipLaunchKernelGGL((sparse_attention_kernel<D, HW>), dim3(static_cast<unsigned>(rows)), dim3(64 * HW), lds,
                       stream, qa, Kc, idx, d.S, d.H_I, d.T, m, mask_mode, k, n_win,
                       scale * 1.4426950408889634f, out);
    return hipGetLastError();
}

template <int D>
hipError_t launch_few(const __bf16* qa, const __bf16* Kc, const int32_t* idx, const si_dims& d, int32_t m,
                      int32_t mask_mode, int32_t k, int32_t n_win, float scale, float* out, hipStream_t stream) {
    static std::atomic<size_t> allowed[64];
    const size_t lds = few_lds_bytes<D>() + list_bytes(k, n_win);
    static_assert(few_lds_bytes<D>() + 2 * kMaxK * 4 <= 159 * 1024, "the longest list fits as well");
    hipError_t e = allow_lds(sparse_attention_few_kernel<D>, lds, allowed);
    if (e != hipSuccess) return e;
    const int head_blocks = (d.H_I + 31) / 32;
    const int64_t grid = static_cast<int64_t>(d.B) * d.S * head_blocks;
    hipLaunchKernelGGL((sparse_attention_few_kernel<D>), dim3(static_cast<unsigned>(grid)),
                       dim3(64 * (kGroupTiles + D / 32)), lds, stream, qa, Kc, idx, d.S, d.H_I, d.T, m, mask_mode, k,
                       n_win, head_blocks, scale * 1.4426950408889634f, out);
    return hipGetLastError();
}

// One round of the chip's compute units, or two with long lists of wide rows.  Measured (us, sparse_attention_kernel -> this;
// the launch and an empty list take 9): k + n_win = 1152, 64 heads of 128, 1 / 32 / 128 / 256 / 384 queries 38 -> 17, 39 -> 18,
// 43 -> 22, 45 -> 41, 54 -> 58; 32 heads of 128, 256 / 512 queries 39 -> 21, 42 -> 40; 64 heads of 64, 128 / 256 queries 28 -> 17,
// 31 -> 31; k + n_win = 640, 64 heads of 128, 128 / 192 queries 25 -> 15, 26 -> 27; 256 keys 12 -> 9.5, 13 -> 17; 32 keys 10 -> 9.2,
// 10 -> 11; 4224 keys, 16 queries 133 -> 50.
bool few_queries(const si_dims& d, int k, int n_win) {
    const int64_t workgroups = static_cast<int64_t>(d.B) * d.S * ((d.H_I + 31) / 32);
    return workgroups <= 256 || (workgroups <= 512 && d.D == 128 && k + n_win >= 1024);
}

}  // namespace

}  // namespace si

using namespace si;

extern "C" {

si_status si_sparse_attention(const void* qa, const void* Kc, const int32_t* idx, const si_dims* dims,
                              int32_t m, int32_t k, si_mask_mode mask_mode, int32_t n_win, float scale,
                              float* out, void* stream) {
    if (!dims || !qa || !Kc || !idx || !out) return SI_ERR_INVALID_ARG;
    const si_dims d = *dims;
    if (d.B < 1 || d.S < 1 || d.H_I < 1 || d.D < 1 || d.T < 1 || m < 1 || k < 1 || n_win < 0) return SI_ERR_INVALID_ARG;
    if (mask_mode != SI_MASK_NONE && mask_mode != SI_MASK_CAUSAL_BLOCK) return SI_ERR_INVALID_ARG;
    if (!(scale == scale) || scale - scale != 0.0f) return SI_ERR_INVALID_ARG;  // NaN or infinite
    if (d.D != 64 && d.D != 128) return SI_ERR_UNSUPPORTED_SHAPE;
    if (d.H_I > kMaxHeads || k > kMaxK || n_win > kMaxK) return SI_ERR_UNSUPPORTED_SHAPE;
    if (static_cast<int64_t>(d.B) * d.S >= (int64_t{1} << 31)) return SI_ERR_UNSUPPORTED_SHAPE;
    const __bf16* q = static_cast<const __bf16*>(qa);
    const __bf16* K = static_cast<const __bf16*>(Kc);
    hipStream_t hs = static_cast<hipStream_t>(stream);
    const bool two = d.H_I > 32;
    hipError_t e;
#define SI_LAUNCH(DD)                                                                                \
    e = few_queries(d, k, n_win) ? launch_few<DD>(q, K, idx, d, m, mask_mode, k, n_win, scale, out, hs) \
        : two ? launch<DD, 2>(q, K, idx, d, m, mask_mode, k, n_win, scale, out, hs)                   \
              : launch<DD, 1>(q, K, idx, d, m, mask_mode, k, n_win, scale, out, hs)
    if (d.D == 128) SI_LAUNCH(128);
    else SI_LAUNCH(64);
#undef SI_LAUNCH
    return e == hipSuccess ? SI_OK : SI_ERR_HIP;
}

}  // extern "C"
