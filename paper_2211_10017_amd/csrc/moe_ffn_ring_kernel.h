// Grouped GEMM with fused dequantisation for launches with few rows per expert or few row tiles (Sec. 3.3,
// Sec. 3.4): the packed weights, the group scales and the activation rows all go from memory straight
// into a ring of two to five LDS stages, up to four K steps ahead.
//
// Such a launch is bound by how many bytes it keeps in flight (few rows per expert: it streams weights), or, with
// about one tile per compute unit, by the latency of what a lone wavefront per SIMD waits for.  Loads into
// registers can be one or two steps ahead at most (moe_ffn_tiled_kernel.h); loads into LDS need no registers,
// are counted by hand, and NST - 1 stages of them stay in flight: three with 16-row blocks (two with 8-bit weights and group scales), two
// with taller ones, one with 64-row blocks of 8-bit weights, whose stage is 32 KB of the 80 KB that two blocks per compute unit
// leave each (three or four in the long kernel, where a block has the compute unit to itself, see ring_long).  The K range is split over the two pairs of wavefronts of the block, whose partial tiles meet in LDS at the end, added
// in the order of K: twice the blocks, each with half the chain of K steps.
//
// Block: 2 x 2 wavefronts; wavefront (wc, kp) computes BM rows x 64 channels over the kp-th half of K.  A stage
// holds, per K part, the rows' 64 K values (unpadded 128-byte rows, 16-byte chunks at position
// chunk ^ ((row >> 1) & 7): conflict-free fragment reads), and per wavefront its two tiles' fragment
// blocks and, for group scales, the 64 channels' scales of the step's group.
//
// Measured (64 tokens, 32 experts of 2048 x 8192, 4-bit, per step): 1 x 4 column wavefronts without a split 128 us, 2 x 4 (one
// block per compute unit) 147, 2 x 2 with two blocks per compute unit 124, with three 115; weights loaded temporal instead of
// non-temporal 154 (8-bit, two blocks: 190, temporal 237).  Rates: 64 tokens on 16 experts of 4096 x 16384, 8-bit, 2.1 GB in a step of
// 351 us, 6.1 TB/s; in register-fed tiles 459 us.
#pragma once
#include <type_traits>

#include "moe_ffn_epilogue.h"

namespace moe {

template <int BITS, int SMODE, int BM>
struct RingShape {
    static constexpr int WC = 2, WK = 2;                            // wavefronts along the channels and along K
    static constexpr int NW = BITS == 4 ? 1 : 2;                    // fragment blocks per tile and 64-deep K step
    static constexpr int TM = BM < 32 ? 1 : BM / 32;                // 32-row matrix tiles (of a 16-row block the upper half repeats the lower)
    static constexpr int kWaves = WC * WK;
    static constexpr bool GROUPED = !channel_scales(SMODE);
    static constexpr int kPartA = BM * 128;                         // bytes of one K part's rows in a stage
    static constexpr int kWaveB = 2 * NW * kFragBytes + (GROUPED ? 256 : 0);
    static constexpr int kStage = WK * kPartA + kWaves * kWaveB;
    static constexpr int kReduce = kWaves * TM * 2 * 16 * 64 * 4;
    // at the end the stages' space holds the partial tiles, then the patches of the tile end, and the row entries behind either
    static constexpr int kRows = kReduce > kWaves * kPatchBytes<16 / WK> ? kReduce : kWaves * kPatchBytes<16 / WK>;
    static constexpr int kEnd = kRows + (int)sizeof(TileRows<32 * TM>);
    // LDS of a compute unit (160 KB): three blocks where a block's share still holds three stages, else two
    static constexpr int kLimit = (BM > 32 || BITS == 8 ? 80 : 53) * 1024;
    static constexpr int NST = kLimit / kStage;                     // stages
    static constexpr int kLds(int stages) { return stages * kStage > kEnd ? stages * kStage : kEnd; }
    static_assert(NST >= 2 && NST <= 4 && kLds(NST) <= kLimit, "a stage in use and one to three in flight (the chain of waits)");
    // 64-row blocks of 8-bit weights, with one stage in flight, may take all of a compute unit's LDS instead (grouped_gemm_ring_long_kernel)
    static constexpr bool kLong = BITS == 8 && BM > 32;
    static constexpr int kMost = kLong ? 160 * 1024 / kStage : NST;
    static_assert(!kLong || (NST == 2 && kMost >= 4 && kMost <= 5 && kLds(kMost) <= 160 * 1024), "up to four in flight (the chain of waits)");
};

template <int BITS, int SMODE, int BM, int NST>
__device__ __forceinline__ void ring_gemm(const GemmArgs &p)
{
    using S = RingShape<BITS, SMODE, BM>;
    constexpr int TM = S::TM, NW = S::NW, WC = S::WC, WK = S::WK;
    constexpr bool GROUPED = S::GROUPED, ACC = SMODE == SCALE_GROUP_ACC, BF = SMODE == SCALE_CHANNEL_BF16;
    constexpr int D = NST - 1;                          // stages in flight, of NST
    constexpr int NA = BM / 8 > WC ? BM / 8 / WC : 1;   // row loads per wavefront and stage (8 rows each)
    constexpr int L = NA + 2 * NW + (GROUPED ? 1 : 0);  // loads per wavefront and stage
    static_assert((D - 1) * L < 64, "the load counter has six bits");
    extern __shared__ __align__(16) uint8_t lds[];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wc = wave % WC, kp = wave / WC;
    const int K = p.K, N = p.N;
    int e, col, row0, rows;
    constexpr int UNIT = BM < 32 ? BM : 32;
    // (scratch of the index: the last stage, which is filled behind the first barrier)
    static_assert(S::kStage >= (int)sizeof(IndexScratch), "the index's scratch fits");
    IndexScratch &index = *reinterpret_cast<IndexScratch *>(lds + (NST - 1) * S::kStage);
    const int ncol = (N + 64 * WC - 1) / (64 * WC);
    if (!(p.gate_idx ? find_unsorted_item<UNIT>(p, BM, ncol, index, &e, &col, &row0, &rows)
                     : find_item<UNIT>(p.offsets, p.E, p.R, BM, ncol, blockIdx.x, &e, &col, &row0, &rows))) return;
    e = __builtin_amdgcn_readfirstlane(e), col = __builtin_amdgcn_readfirstlane(col);
    row0 = __builtin_amdgcn_readfirstlane(row0), rows = __builtin_amdgcn_readfirstlane(rows);

    RowEntry<32 * TM> entry;                                 // what the rows need at the end is requested now
    entry.load(p, index, row0, rows);
    // this wavefront's two 32-channel tiles (N is a multiple of 64: both exist or neither does)
    const int tile_ok = (col * WC + wc) * 64 < N;
    const int ntile0 = tile_ok ? (col * WC + wc) * 2 : 0;
    float cs_lane = 1.0f, bias_lane = 0.0f;             // channel factors: lane l brings channel l of the wavefront's 64
    if (!GROUPED) cs_lane = __half2float(p.scales[(size_t)e * N + ntile0 * 32 + lane]);
    if (p.bias) bias_lane = __half2float(p.bias[(size_t)e * N + ntile0 * 32 + lane]);
    // this wavefront's part of the K steps
    const int nk = K / 64, per = (nk + WK - 1) / WK;
    const int first = kp * per, mine = tile_ok ? min(max(nk - first, 0), per) : 0;

    // ---- global addresses.  A load fills eight LDS rows; lane l brings chunk position l & 7 of row l >> 3,
    // which holds K chunk (l & 7) ^ ((row >> 1) & 7).
    const uint16_t *a_ptr[NA];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int row = 8 * ((i * WC + wc) % (BM / 8)) + (lane >> 3);
        a_ptr[i] = p.a + (size_t)source_row(p, index, row0, min(row, rows - 1)) * K + ((lane & 7) ^ ((row >> 1) & 7)) * 8;      // clamped: always a valid row
    }
    const uint8_t *b_ptr[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
        b_ptr[t] = p.wq + (size_t)e * packed_bytes_per_expert(K, N, BITS) + (size_t)(ntile0 + t) * (K / frag_k(BITS)) * kFragBytes + lane * 16;
    const __half *s_ptr = p.scales + (size_t)e * (K / p.g) * N + ntile0 * 32 + (lane & 31) * 2;

    // all loads of stage `slot`, for K step first + s of this part (past the end: the last step again)
    auto issue = [&](int s, int slot) {
        const int kb = min(first + s, nk - 1);
        uint8_t *st = lds + slot * S::kStage;
        uint8_t *sb = st + WK * S::kPartA + wave * S::kWaveB;
#pragma unroll
        for (int i = 0; i < NA; ++i)
            load_to_lds16(a_ptr[i] + kb * 64, reinterpret_cast<uint16_t *>(st + kp * S::kPartA + (i * WC + wc) % (BM / 8) * 1024));
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int w = 0; w < NW; ++w)
                load_to_lds16<TM == 1>(b_ptr[t] + (size_t)(kb * NW + w) * kFragBytes, reinterpret_cast<uint16_t *>(sb + (t * NW + w) * kFragBytes));
        // (weights of blocks that hold an expert's rows in one tile, mostly, are read once: non-temporal)
        if constexpr (GROUPED) load_to_lds4(s_ptr + (size_t)((kb * 64) / p.g) * N, sb + 2 * NW * kFragBytes);
    };

    float16_t acc[TM][2];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[m][t][i] = 0.0f;

    float16_t part[ACC ? TM : 1][2];                    // sums of the current group
    if constexpr (ACC)
#pragma unroll
        for (int m = 0; m < TM; ++m)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int i = 0; i < 16; ++i) part[m][t][i] = 0.0f;

    auto compute = [&](int slot, bool last_of_group, auto live_c) {
        constexpr int LIVE = decltype(live_c)::value;               // row tiles of this block that hold rows
        const uint8_t *st = lds + slot * S::kStage;
        const uint16_t *sa = reinterpret_cast<const uint16_t *>(st + kp * S::kPartA);
        const uint8_t *sb = st + WK * S::kPartA + wave * S::kWaveB;
        uint32_t raw[2][NW * 4];
        _Float16 sc[2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                const uint4 v = *reinterpret_cast<const uint4 *>(sb + (t * NW + w) * kFragBytes + lane * 16);
                raw[t][4 * w + 0] = v.x; raw[t][4 * w + 1] = v.y; raw[t][4 * w + 2] = v.z; raw[t][4 * w + 3] = v.w;
            }
            if constexpr (GROUPED)
                sc[t] = *reinterpret_cast<const _Float16 *>(sb + 2 * NW * kFragBytes + (t * 32 + (lane & 31)) * 2);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            half8_t a[TM];
#pragma unroll
            for (int m = 0; m < TM; ++m)
                if (m < LIVE) a[m] = *reinterpret_cast<const half8_t *>(sa + (32 * m + (lane & (BM < 32 ? BM - 1 : 31))) * 64 + 8 * ((2 * j + (lane >> 5)) ^ ((lane >> 1) & 7)));
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                uint32_t bw[4];
                if constexpr (BF) codes_to_bf16<BITS>(raw[t] + j * NW, bw);
                else if (BITS == 4) dequant4(raw[t][j], bw);
                else dequant8(raw[t][2 * j], raw[t][2 * j + 1], bw);
                if constexpr (SMODE == SCALE_GROUP) {
                    const half2_t s2 = {sc[t], sc[t]};
#pragma unroll
                    for (int q = 0; q < 4; ++q) bw[q] = h2_bits(bits_h2(bw[q]) * s2);
                }
#pragma unroll
                for (int m = 0; m < TM; ++m) {
                    if (m >= LIVE) continue;
                    if constexpr (ACC) {
                        part[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[m], frag_from(bw), part[m][t], 0, 0, 0);
                    } else {
                        acc[m][t] = tile_product<BF>(a[m], frag_from(bw), acc[m][t]);
                    }
                }
            }
        }
        if constexpr (ACC) {        // exact codes went in: at the end of a group (or of this part of K) its sums are folded with the scale in fp32
            if (last_of_group) {
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const float sf = (float)sc[t];
#pragma unroll
                    for (int m = 0; m < TM; ++m)
                        if (m < LIVE)
#pragma unroll
                            for (int i = 0; i < 16; ++i) {
                                acc[m][t][i] = fmaf(part[m][t][i], sf, acc[m][t][i]);
                                part[m][t][i] = 0.0f;
                            }
                }
            }
        }
    };

    // Stages issued and not yet used stay in flight; at the top of a step the wavefront waits for its own
    // share of the step's stage (the loads of the `rem` stages after it may be outstanding: the counter is
    // in order), and the barrier makes everyone's share visible and tells that everyone has left the
    // stage before it, which is then refilled.
#pragma unroll
    for (int s = 0; s < D; ++s)
        if (s < per) issue(s, s);
    auto k_loop = [&](auto live_c) {
        int slot = 0;
        for (int s = 0; s < per; ++s) {
            const int rem = min(per - 1 - s, D - 1);
            if (rem == D - 1) wait_loads<(D - 1) * L>();
            else if (D > 3 && rem == 2) wait_loads<(D > 3) * 2 * L>();
            else if (D > 2 && rem == 1) wait_loads<(D > 2) * L>();
            else wait_loads<0>();
            __syncthreads();
            if (s + D < per) issue(s + D, slot == 0 ? NST - 1 : slot - 1);
            if (s < mine) compute(slot, s + 1 == mine || (first + s + 1) * 64 % p.g == 0, live_c);
            slot = slot + 1 == NST ? 0 : slot + 1;
        }
    };
    if (TM == 1 || rows > 32) k_loop(std::integral_constant<int, TM>{});
    else k_loop(std::integral_constant<int, 1>{});

    // ---- the K parts meet: every wavefront leaves its partial tiles in LDS and finishes registers
    // [QN kp, QN kp + QN) of each tile of its channels
    constexpr int QN = 16 / WK;
    float cs[2], bias[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        cs[t] = __shfl(cs_lane, 32 * t + (lane & 31)) * (BF ? kBf16CodeUnit : 1.0f);      // (bf16 codes go in as q / kBf16CodeUnit)
        bias[t] = __shfl(bias_lane, 32 * t + (lane & 31));
    }
    __syncthreads();                                    // every wavefront is done with the ring
    TileRows<32 * TM> &tile_rows = *reinterpret_cast<TileRows<32 * TM> *>(lds + S::kRows);
    entry.put(tile_rows);
    float *red = reinterpret_cast<float *>(lds);    // [wave][m][t][16][64]
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) red[((wave * TM + m) * 2 + t) * 1024 + i * 64 + lane] = acc[m][t][i];
    __syncthreads();
    float v[TM][2][QN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < 2; ++t)
#pragma unroll
            for (int q = 0; q < QN; ++q) {
                const float *src = red + ((wc * TM + m) * 2 + t) * 1024 + (kp * QN + q) * 64 + lane;
                float sum = src[0];
#pragma unroll
                for (int w = 1; w < WK; ++w) sum += src[(size_t)w * WC * TM * 2 * 1024];
                v[m][t][q] = sum;
            }
    __syncthreads();                                // the partial tiles have been read
    if (tile_ok) finish_tile<TM, QN, 32 * TM>(p, v, tile_rows, cs, bias, rows, 8 * (QN / 4) * kp, ntile0 * 32, lds + wave * kPatchBytes<QN>);
}

// So are the rows' type and the codes': with a loop for bf16 beside the one for FP16 in a kernel a launch of 40 rows of 8-bit experts, whose code no block
// has run before, took longer (a step of 40 tokens, one of 32 of 1024 x 4096, 47.6 us in one, 47.2 apart; 997 bf16 tokens of 768 x 3072 62.6 and 62.1).
// The number of stages is a constant of the kernel: as an argument of one kernel for both it cost the shorter ring with group scales 1 to 3 %
// (590 tokens, two of 5 experts of 1600 x 11456, 175 us a step and 169).
template <int BITS, int SMODE, int BM>
__global__ __launch_bounds__(256, 2) void grouped_gemm_ring_kernel(GemmArgs p)
{
    ring_gemm<BITS, SMODE, BM, RingShape<BITS, SMODE, BM>::NST>(p);
}

template <int BITS, int SMODE, int BM>
__global__ __launch_bounds__(256, 2) void grouped_gemm_ring_long_kernel(GemmArgs p)
{
    ring_gemm<BITS, SMODE, BM, RingShape<BITS, SMODE, BM>::kMost>(p);
}

template <int BITS, int SMODE, int BM>
static void launch_ring_shape(const GemmArgs &p, dim3 grid, hipStream_t s)
{
    using S = RingShape<BITS, SMODE, BM>;
    if constexpr (S::kLong) {
        if (p.ring_long) {
            static std::atomic<uint64_t> raised;
            raise_lds_limit(reinterpret_cast<const void *>(&grouped_gemm_ring_long_kernel<BITS, SMODE, BM>), S::kLds(S::kMost), raised);
            hipLaunchKernelGGL((grouped_gemm_ring_long_kernel<BITS, SMODE, BM>), grid, dim3(256), S::kLds(S::kMost), s, p);
            return;
        }
    }
    static std::atomic<uint64_t> raised;
    raise_lds_limit(reinterpret_cast<const void *>(&grouped_gemm_ring_kernel<BITS, SMODE, BM>), S::kLds(S::NST), raised);
    hipLaunchKernelGGL((grouped_gemm_ring_kernel<BITS, SMODE, BM>), grid, dim3(256), S::kLds(S::NST), s, p);
}

template <int BITS, int SMODE>
static void launch_ring_variants(const GemmArgs &p, int bm, dim3 grid, hipStream_t s)
{
    if (bm == 16) launch_ring_shape<BITS, SMODE, 16>(p, grid, s);
    else if (bm == 32) launch_ring_shape<BITS, SMODE, 32>(p, grid, s);
    else launch_ring_shape<BITS, SMODE, 64>(p, grid, s);
}

}  // namespace moe
