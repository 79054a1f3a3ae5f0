// LDS-tiled grouped GEMM with fused dequantisation, for experts with many rows
// (Sec. 3.3 grouped GEMM, Sec. 3.4 fused dequantisation).
//
// Tokens are the MFMA A operand (rows), weights the B operand (columns).  A wavefront fetches
// its weight fragments straight from HBM into registers (one 16-byte load per lane per 1 KB
// fragment block, see moe_common.h), converts the codes to FP16 with the 0x6400 trick and
// feeds v_mfma_f32_32x32x16_f16; only the activations go through LDS (FP16 rows straight from
// global memory; bf16 rows converted to scaled FP16 beforehand, or as they are to bf16 codes), shared by the four wavefronts of a block, each
// of which owns its own 64 output channels.
#pragma once
#include <type_traits>

#include "moe_ffn_epilogue.h"

namespace moe {

constexpr int kLdsRow = 64;              // halfs per LDS row: one K step, no padding; the 16-byte chunks of a row are
                                         // stored at position (k chunk) ^ ((row >> 1) & 7), which makes the b128
                                         // fragment reads conflict-free and keeps a wavefront's 64 chunks contiguous
constexpr int kTN = 2;                   // 32-channel tiles per wavefront

// (bf16 rows that meet bf16 codes are a scale mode, not a branch: both loops in one kernel take 194 registers for 64-row tiles of 8-bit weights, two wavefronts per
// SIMD, each by itself 162 to 164, three; 4096 tokens, two of 128 experts of 2048 x 8192, skewed, a step 1145 us in one, 1116 apart)
template <int BITS, int SMODE, int TM>
__global__ __launch_bounds__(256, TM == 1 && !(SMODE == SCALE_GROUP_ACC || SMODE == SCALE_GROUP_SPLIT) ? 4 : 2) void grouped_gemm_kernel(GemmArgs p)
{
    constexpr bool BF = SMODE == SCALE_CHANNEL_BF16;
    constexpr int BM = 32 * TM;
    constexpr int NW = BITS == 4 ? 1 : 2;             // 16-byte loads per tile per 64-deep K step
    // two stages of rows; at the end the patches through which the wavefronts' results leave
    constexpr int kStageBytes = 2 * BM * kLdsRow * 2, kPatches = 4 * kPatchBytes<16>;
    __shared__ __align__(16) uint8_t lds_raw[kStageBytes > kPatches ? kStageBytes : kPatches];
    uint16_t (*lds_a)[BM * kLdsRow] = reinterpret_cast<uint16_t (*)[BM * kLdsRow]>(lds_raw);
    __shared__ TileRows<BM> tile_rows;

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: tile addresses stay scalar
    const int K = p.K, N = p.N;
    int e, col, row0, rows;
    // (scratch of the index: behind the first stage, which is filled while other wavefronts still read their rows' assignments)
    static_assert(sizeof(lds_raw) >= kStageBytes / 2 + sizeof(IndexScratch), "the index's scratch fits");
    IndexScratch &index = *reinterpret_cast<IndexScratch *>(lds_raw + kStageBytes / 2);
    // 64-row tiles of group sums, the largest layers' loop, never sort (with the code for it 8192 tokens, two of 64 experts of 4096 x 16384, 4533 us a step, without 4506)
    if constexpr (SMODE == SCALE_GROUP_ACC && TM == 2) p.gate_idx = nullptr;
    if (!(p.gate_idx ? find_unsorted_item(p, 32 * p.tile_units, (N + 255) / 256, index, &e, &col, &row0, &rows)
                     : find_item(p.offsets, p.E, p.R, 32 * p.tile_units, (N + 255) / 256, blockIdx.x, &e, &col, &row0, &rows))) return;
    e = __builtin_amdgcn_readfirstlane(e), col = __builtin_amdgcn_readfirstlane(col);      // the same in every lane: kept in scalar registers
    row0 = __builtin_amdgcn_readfirstlane(row0), rows = __builtin_amdgcn_readfirstlane(rows);

    // what the rows need at the end is requested now; the tallest tile has no registers to carry it through the K loop
    RowEntry<BM> entry;
    entry.load(p, index, row0, rows);
    if constexpr (TM == 4) entry.put(tile_rows);
    const int nk = K / 64;
    const int ntile0 = (col * 4 + wave) * kTN;         // first 32-channel tile of this wavefront
    const bool tile_ok = ntile0 * 32 < N;              // N is a multiple of 64: both tiles exist or neither does
    const int tile_c = tile_ok ? ntile0 : 0;
    float cs_lane = 1.0f, bias_lane = 0.0f;            // channel factors: lane l brings channel l of the wavefront's 64
    auto load_channels = [&]() {
        const size_t n = (size_t)e * N + tile_c * 32 + lane;
        if (channel_scales(SMODE)) cs_lane = __half2float(p.scales[n]);
        if (p.bias) bias_lane = __half2float(p.bias[n]);
    };
    if constexpr (TM < 4) load_channels();

    // ---- global addresses
    // A: thread loads 16 bytes = 8 K values of row (tid/8 + 32*pass)
    // thread t fills chunk position t & 7 of LDS row t >> 3 (+ 32 per pass); the K chunk that belongs
    // there is (t & 7) ^ ((row >> 1) & 7), the same for every pass
    const int a_row = threadIdx.x >> 3, a_pos = (threadIdx.x & 7) * 8;
    const int a_seg = ((threadIdx.x & 7) ^ ((threadIdx.x >> 4) & 7)) * 8;
    const uint16_t *a_ptr[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        a_ptr[m] = p.a + (size_t)source_row(p, index, row0, min(a_row + 32 * m, rows - 1)) * K + a_seg;      // clamped: always a valid row
    }
    // B: fragment blocks of tile t are contiguous along K
    const uint8_t *w_e = p.wq + (size_t)e * packed_bytes_per_expert(K, N, BITS);
    const uint4 *b_ptr[kTN];
#pragma unroll
    for (int t = 0; t < kTN; ++t) {
        b_ptr[t] = reinterpret_cast<const uint4 *>(w_e + (size_t)(tile_c + t) * (K / frag_k(BITS)) * kFragBytes);   // wave-uniform
    }
    const int G = K / p.g;
    const __half *s_ptr[kTN];
#pragma unroll
    for (int t = 0; t < kTN; ++t) {
        s_ptr[t] = p.scales + (size_t)e * G * N + (tile_c + t) * 32;              // wave-uniform
    }

    float16_t acc[TM][kTN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int t = 0; t < kTN; ++t)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc[m][t][i] = 0.0f;

    // SCALE_GROUP_ACC (groups of 128 = the two K steps of one loop trip): the codes enter the MFMAs
    // unscaled (exact), a group's products are summed in accg and folded into acc with the group's
    // scale in fp32.  Exact like the two-term form, at half its MFMA count; needs the registers of a
    // second accumulator set, so it is built for row tiles of at most 64 rows.
    constexpr bool ACC = SMODE == SCALE_GROUP_ACC;
    // 4-bit codes that go in unscaled are taken the same way, as q 2^-9 (2^24 itself is no FP16 number), which the factor at the end makes up for:
    // two-operand masks instead of v_and_or_b32 with three registers.  4096 FP16 tokens, two of 16 experts of 2048 x 8192, a step 501 -> 498 us, 16384, one of 64 of
    // 1024 x 4096 326.3 -> 325.3; 8192 bf16 tokens, two of 64 of 4096 x 16384, which are converted, 3859 and 3859, with groups of 128 4563 -> 4534.
    constexpr bool EXACT4 = BITS == 4 && (SMODE == SCALE_CHANNEL || ACC);
    static_assert(!ACC || TM <= 2, "two accumulator sets fit for TM <= 2 only");
    float16_t accg[ACC ? TM : 1][kTN];

    // Activations are fetched one K step ahead (they come from L2); packed weights and group
    // scales PF = 2 steps ahead, into two register sets used alternately (they come from HBM, and
    // one step of MFMA work is shorter than that latency).  The tallest 8-bit tile has registers
    // for one set only and fetches one step ahead.
    constexpr int PF = (BITS == 8 && TM == 4) ? 1 : 2;
    // The rows (16 bits each; group-scaled layers get bf16 rows converted, see rows_to_f16_kernel) go from global memory straight into
    // the LDS stage: no staging registers, no LDS write instructions.
    constexpr int LB = kTN * NW + (channel_scales(SMODE) ? 0 : kTN);   // loads of one load_b()
    auto dma_a = [&](int kb, uint16_t *stage, int m) {
        load_to_lds16(a_ptr[m] + kb * 64, stage + (32 * m + 8 * wave) * kLdsRow);
    };
    uint4 gb[PF][kTN][NW];
    _Float16 gs[PF][kTN];
    auto load_b = [&](int kb, auto slot_c) {
        constexpr int WS = decltype(slot_c)::value;
#pragma unroll
        for (int t = 0; t < kTN; ++t) {
#pragma unroll
            for (int w = 0; w < NW; ++w) gb[WS][t][w] = (b_ptr[t] + (size_t)(kb * NW + w) * 64)[lane];
            if (!channel_scales(SMODE))
                gs[WS][t] = __builtin_bit_cast(_Float16, (s_ptr[t] + (size_t)((kb * 64) / p.g) * N)[lane & 31]);
        }
    };

    const int live = (rows + 31) / 32;
#pragma unroll
    for (int m = 0; m < TM; ++m)
        if (m < live) dma_a(0, lds_a[0], m);
    load_b(0, std::integral_constant<int, 0>{});
    if constexpr (PF == 2) load_b(min(1, nk - 1), std::integral_constant<int, 1>{});
    // Private copies of the steps being computed.  They are taken (and the loads of the next
    // steps issued) once per pair of K steps, at the top of the loop body (PF = 1: at the top of
    // each step): at the loop edge every weight load is then at least a full step old, so the
    // drain of the load counter that the compiler places at a loop head does not wait for fresh loads.
    uint32_t raw2[PF][kTN][NW * 4];
    _Float16 sc2[PF][kTN];
    auto take = [&](auto slot_c) {
        constexpr int WS = decltype(slot_c)::value;
#pragma unroll
        for (int t = 0; t < kTN; ++t) {
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                // real register moves (opaque to the compiler): if it merged these copies with
                // the load registers, the refills would land elsewhere and have to be moved
                // back at the loop edge, i.e. waited for right after being issued
                raw2[WS][t][4 * w + 0] = opaque_copy(gb[WS][t][w].x); raw2[WS][t][4 * w + 1] = opaque_copy(gb[WS][t][w].y);
                raw2[WS][t][4 * w + 2] = opaque_copy(gb[WS][t][w].z); raw2[WS][t][4 * w + 3] = opaque_copy(gb[WS][t][w].w);
            }
            sc2[WS][t] = __builtin_bit_cast(_Float16, (uint16_t)opaque_copy((uint32_t)__builtin_bit_cast(uint16_t, gs[WS][t])));
        }
    };
    // One barrier per step, at its top: it publishes this step's stage (written during the
    // previous step) and tells that every wavefront has left the other stage, which is then
    // refilled at the end of the step, when its rows have had time to arrive; the arrival of
    // the rows is not waited for in front of a barrier.
    auto k_step = [&](int kb, auto slot_c, auto live_c, auto window_c) {
        constexpr int SL = decltype(slot_c)::value;      // = kb & 1: LDS stage and weight register set
        constexpr bool WINDOW = decltype(window_c)::value;
        constexpr int LIVE = decltype(live_c)::value;    // row tiles of this block that hold rows
        uint16_t *stage = lds_a[SL];
        // this wavefront's share of the stage has landed once only the weight refills issued after
        // it (in the previous step) are still in flight
        wait_loads<PF == 2 ? (SL == 1 ? 2 * LB : 0) : LB>();
        __syncthreads();
        uint32_t (&raw)[kTN][NW * 4] = raw2[PF == 2 ? SL : 0];
        _Float16 (&sc)[kTN] = sc2[PF == 2 ? SL : 0];
        // The step's loads are dealt over its four MFMA sub-steps, so that the memory pipeline
        // takes a few at a time between matrix instructions: the next step's activation rows in
        // the first two, the weight refills after them (the load counter is in order, so the wait
        // for the rows leaves the younger weight loads in flight).  No branches around the loads:
        // past the end they re-read the last step, which keeps the loop body free of joins and
        // the load counter exact.
        auto issue = [&](int j) {
            const int kn = min(kb + 1, nk - 1);
            if (j < 2) {
#pragma unroll
                for (int m = 0; m < TM; ++m)       // (row tiles past the expert's last row are neither loaded nor written)
                    if (m < LIVE && (TM == 1 ? j == 0 : (m < TM / 2) == (j == 0))) {
                        dma_a(kn, lds_a[1 - SL], m);          // the other stage: every wavefront has left it
                    }
            } else if constexpr (PF == 2) {
                if constexpr (SL == 0) {
                    if (j == 2) load_b(min(kb + 2, nk - 1), std::integral_constant<int, 0>{});
                    else load_b(min(kb + 3, nk - 1), std::integral_constant<int, 1>{});
                }
            } else if (j == 2) {
                load_b(min(kb + 1, nk - 1), std::integral_constant<int, 0>{});
            }
        };

        // unpack + convert one 16-deep step of weight fragments in registers
        ScaledCodes factors[kTN];
        if constexpr (WINDOW || EXACT4)
#pragma unroll
            for (int t = 0; t < kTN; ++t) factors[t] = ScaledCodes(EXACT4 ? (_Float16)32768.0f : sc[t]);
        auto dequant_step = [&](int j, uint32_t (&bw)[kTN][4], uint32_t (&bl)[kTN][4]) {
#pragma unroll
            for (int t = 0; t < kTN; ++t) {
                if constexpr (BF) {
                    codes_to_bf16<BITS>(raw[t] + j * NW, bw[t]);
                    continue;
                }
                if constexpr (WINDOW || EXACT4) {
                    factors[t].convert(raw[t][j], bw[t]);
                    continue;
                }
                if (BITS == 4) dequant4(raw[t][j], bw[t]);
                else dequant8(raw[t][2 * j], raw[t][2 * j + 1], bw[t]);
                if (SMODE == SCALE_GROUP) {
                    const half2_t s2 = {sc[t], sc[t]};
#pragma unroll
                    for (int q = 0; q < 4; ++q) bw[t][q] = h2_bits(bits_h2(bw[t][q]) * s2);
                } else if (SMODE == SCALE_GROUP_SPLIT) {
                    // exact two-term weight: hi = fl(q*s'), lo = q*s' - hi, with s' = 256*s so
                    // that lo stays a normal FP16 number; the epilogue divides by 256
                    const _Float16 s8 = sc[t] * (_Float16)256.0f;
                    const half2_t s2 = {s8, s8};
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const half2_t qv = bits_h2(bw[t][q]);
                        const half2_t hi = qv * s2;
                        half2_t lo;
                        lo[0] = __builtin_fmaf16(qv[0], s2[0], -hi[0]);
                        lo[1] = __builtin_fmaf16(qv[1], s2[1], -hi[1]);
                        bw[t][q] = h2_bits(hi);
                        bl[t][q] = h2_bits(lo);
                    }
                }
            }
        };
        // ---- MFMA over the four 16-deep steps of this K slab; the fragments of step j+1 are
        // converted while the MFMAs of step j run (VALU work hides under the matrix pipe)
        // Where the registers allow (PIPE), the A fragments of step j+1 are read from LDS before the
        // MFMAs of step j are issued, so that the LDS latency passes under a full step of matrix
        // work; otherwise each fragment is read just before its MFMAs and the other wavefront of
        // the SIMD covers the wait.
        constexpr bool PIPE = TM < 4 || !(SMODE == SCALE_GROUP_SPLIT || false);
        uint32_t bw[2][kTN][4], bl[2][kTN][4];
        half8_t af[PIPE ? 2 : 1][TM];
        auto read_a = [&](int j, int m) {
            return *reinterpret_cast<const half8_t *>(stage + (32 * m + (lane & 31)) * kLdsRow + 8 * ((2 * j + (lane >> 5)) ^ ((lane >> 1) & 7)));
        };
        auto read_step = [&](int j, half8_t (&dst)[TM]) {
#pragma unroll
            for (int m = 0; m < TM; ++m)
                if (m < LIVE) dst[m] = read_a(j, m);    // row tiles past the expert's last row are skipped
        };
        if (PIPE) read_step(0, af[0]);
        dequant_step(0, bw[0], bl[0]);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            issue(j);
            if (PIPE && j + 1 < 4) read_step(j + 1, af[PIPE ? (j + 1) & 1 : 0]);
            __builtin_amdgcn_sched_barrier(0);          // loads and LDS reads stay ahead of this sub-step's MFMAs
            if (j + 1 < 4) dequant_step(j + 1, bw[(j + 1) & 1], bl[(j + 1) & 1]);
#pragma unroll
            for (int m = 0; m < TM; ++m) {
                if (m < LIVE) {
                    const half8_t a = PIPE ? af[PIPE ? j & 1 : 0][m] : read_a(j, m);
#pragma unroll
                    for (int t = 0; t < kTN; ++t) {
                        if constexpr (ACC) {
                            float16_t c = accg[m][t];
                            if (SL == 0 && j == 0)          // first products of a group: start from zero
#pragma unroll
                                for (int i = 0; i < 16; ++i) c[i] = 0.0f;
                            accg[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, frag_from(bw[j & 1][t]), c, 0, 0, 0);
                        } else {
                            acc[m][t] = tile_product<BF>(a, frag_from(bw[j & 1][t]), acc[m][t]);
                            if (SMODE == SCALE_GROUP_SPLIT)
                                acc[m][t] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a, frag_from(bl[j & 1][t]), acc[m][t], 0, 0, 0);
                        }
                    }
                }
            }
        }
        if constexpr (ACC && SL == 1) {                 // end of the group: acc += scale * accg
#pragma unroll
            for (int t = 0; t < kTN; ++t) {
                const float sf = (float)sc[t] * (EXACT4 ? 512.0f : 1.0f);
#pragma unroll
                for (int m = 0; m < TM; ++m)
                    if (m < LIVE)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[m][t][i] = fmaf(accg[m][t][i], sf, acc[m][t][i]);
            }
        }
    };
    // Group scales with the multiply and the subtraction of the code's offset in one instruction (ScaledCodes): an accumulator
    // column, which is a lane's channel, is kept in units of a power of two that brings the channel's first scale to the middle
    // of what that conversion takes, and a wavefront that meets a scale outside of it goes on in the general loop.
    // (4-bit codes only: for 8-bit ones, which save as many instructions, it takes the 32-row tile's fourth wavefront per SIMD, 140 registers for 128,
    // and gains nothing.  us a step with / without, groups of 128: 4000 tokens, one of 128 experts of 1024 x 4096 262.7 / 262.6, 8000 350.4 / 350.4, 3000, one of 64 of
    // 2048 x 8192 511.9 / 510.9.)
    constexpr bool WINDOWED = SMODE == SCALE_GROUP && BITS == 4;
    int unit[kTN] = {};
    // The K loop exists once per number of live row tiles (the last tile of an expert usually
    // holds few rows): a run-time test inside the loop would cut the MFMA stream into pieces.
    // Returns the K step that it stopped at.
    auto k_loop = [&](int kb, auto live_c, auto window_c) {
        for (; kb < nk; kb += 2) {
            take(std::integral_constant<int, 0>{});
            if constexpr (PF == 2) take(std::integral_constant<int, PF - 1>{});
            if constexpr (decltype(window_c)::value) {
                bool in = true;
#pragma unroll
                for (int s = 0; s < PF; ++s)
#pragma unroll
                    for (int t = 0; t < kTN; ++t) {
                        sc2[s][t] = __builtin_amdgcn_ldexph(sc2[s][t], unit[t]);
                        in &= scale_in_window(sc2[s][t]);
                    }
                if (!__all(in)) break;
            }
            k_step(kb, std::integral_constant<int, 0>{}, live_c, window_c);
            if (kb + 1 < nk) {
                if constexpr (PF == 1) take(std::integral_constant<int, 0>{});
                k_step(kb + 1, std::integral_constant<int, 1>{}, live_c, window_c);
            }
        }
        return kb;
    };
    // Both loops exist per number of live row tiles.  (With the general one for full tiles only, layers whose scales leave the window, which wide-spread weights do
    // at once, paid for tiles that hold no rows.  us a step with 1 % of the groups 16 times as large, all live / by number / general loop from the start: 2048 tokens, two of 16
    // experts of 2048 x 8192 384 / 342 / 341, 8192, two of 64 of 4096 x 16384 4834 / 4391 / 4382; all groups alike, no window to be left, 332, and 341 without windows.)
    auto whole_k = [&](auto live_c) {
        if constexpr (WINDOWED) {
#pragma unroll
            for (int t = 0; t < kTN; ++t) unit[t] = window_unit(gs[0][t]);
            const int kb = k_loop(0, live_c, std::true_type{});
            if (kb == nk) return;
#pragma unroll
            for (int t = 0; t < kTN; ++t) {
                const float back = __builtin_ldexpf(1.0f, kWindowShift - unit[t]);
#pragma unroll
                for (int m = 0; m < TM; ++m)
                    if (m < decltype(live_c)::value)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[m][t][i] *= back;
                unit[t] = kWindowShift;
            }
            k_loop(kb, live_c, std::false_type{});
        } else {
            k_loop(0, live_c, std::false_type{});
        }
    };
    if (TM == 1 || live == TM) whole_k(std::integral_constant<int, TM>{});
    else if (TM >= 4 && live == 3) whole_k(std::integral_constant<int, 3>{});
    else if (TM >= 2 && live == 2) whole_k(std::integral_constant<int, 2>{});
    else whole_k(std::integral_constant<int, 1>{});
    wait_loads<0>();      // the last step's (unused) refill of the other stage must land before the block's LDS is given up

    // ---- epilogue: acc[m][t][i] is row 32*m + 8*(i/4) + 4*(lane/32) + i%4 of the tile, channel lane%32 of tile t
    if constexpr (TM < 4) entry.put(tile_rows);
    __syncthreads();                                   // every wavefront has left the stages
    if (!tile_ok) return;
    float cs[kTN], bias[kTN];
    const float unit_cs = EXACT4 ? 512.0f : BF ? kBf16CodeUnit : 1.0f;      // unscaled codes went in as q / unit_cs
    if constexpr (TM == 4) load_channels();
#pragma unroll
    for (int t = 0; t < kTN; ++t) {
        cs[t] = channel_scales(SMODE) ? __shfl(cs_lane, 32 * t + (lane & 31)) * unit_cs : SMODE == SCALE_GROUP_SPLIT ? 1.0f / 256.0f
              : WINDOWED ? __builtin_ldexpf(1.0f, kWindowShift - unit[t]) : 1.0f;
        bias[t] = __shfl(bias_lane, 32 * t + (lane & 31));
    }
    finish_tile<TM, 16, BM>(p, acc, tile_rows, cs, bias, rows, 0, ntile0 * 32, lds_raw + wave * kPatchBytes<16>);
}

template <int BITS, int SMODE>
static void launch_tm(const GemmArgs &p, int tm, dim3 grid, hipStream_t s)
{
    if (tm == 1) hipLaunchKernelGGL((grouped_gemm_kernel<BITS, SMODE, 1>), grid, dim3(256), 0, s, p);
    else if (tm == 2) hipLaunchKernelGGL((grouped_gemm_kernel<BITS, SMODE, 2>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((grouped_gemm_kernel<BITS, SMODE, 4>), grid, dim3(256), 0, s, p);
}

// All kernels of one weight width and one kind of scale mode (one translation unit each, so that they
// compile side by side): EXACT = the two forms that keep the group scales out of the FP16 weights.
template <int BITS, bool EXACT>
static void launch_tiled_variants(const GemmArgs &p, int smode, int tm, dim3 grid, hipStream_t s)
{
    if constexpr (!EXACT) {
        if (smode == SCALE_CHANNEL_BF16) launch_tm<BITS, SCALE_CHANNEL_BF16>(p, tm, grid, s);
        else if (smode == SCALE_CHANNEL) launch_tm<BITS, SCALE_CHANNEL>(p, tm, grid, s);
        else launch_tm<BITS, SCALE_GROUP>(p, tm, grid, s);
    } else if (smode == SCALE_GROUP_ACC) {                 // row tiles of at most 64 rows
        if (tm == 1) hipLaunchKernelGGL((grouped_gemm_kernel<BITS, SCALE_GROUP_ACC, 1>), grid, dim3(256), 0, s, p);
        else hipLaunchKernelGGL((grouped_gemm_kernel<BITS, SCALE_GROUP_ACC, 2>), grid, dim3(256), 0, s, p);
    } else {
        launch_tm<BITS, SCALE_GROUP_SPLIT>(p, tm, grid, s);
    }
}

}  // namespace moe
