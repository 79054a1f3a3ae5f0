// End of a grouped GEMM tile: scale, bias, activation and store, shared by the kernels with row tiles.
//
// An element costs two to four vector instructions and one 2- or 4-byte LDS write: the choices that are the
// same for the whole launch (row factors, activation, gate scales, output type) are made once per pass over
// the registers, not once per element, and rows leave through a patch of LDS of the wavefront's own, 16 bytes per
// lane and whole 128-byte lines.  With a branch per element and per choice, the row factors read from memory
// between the stores, and a neighbour exchange for 4-byte stores, this was 16-20 vector instructions per element: as
// much as sixteen K steps of a 64-row tile.  Measured per layer step: 997 tokens of 768 x 3072 (bf16, GELU, 16 experts) 118 -> 97 us,
// 16384 tokens of 1024 x 4096 (64 experts) 380 -> 333 us, 8192 bf16 tokens of 4096 x 16384 5200 -> 4900 us; same bits.
#pragma once
#include <type_traits>

#include "moe_ffn_common.h"

namespace moe {

constexpr int kPatchRow = 144;                                       // bytes: 128 of data, rows start 4 banks apart
template <int NQ> constexpr int kPatchBytes = 2 * NQ * kPatchRow;    // per wavefront

// What the rows of a tile need at the end, one entry per row, in LDS.
template <int BM>
struct __align__(16) TileRows {
    float pow[BM];          // power of two the row went in scaled down by (bf16 rows)
    float scale[BM];        // gate scale of the fused un-permute
    int32_t dst[BM];        // output row
};

// Thread i < BM brings row i's entries (rows past the last one repeat it): loaded early, put into LDS when the caller likes.
template <int BM>
struct RowEntry {
    float pow = 1.0f, scale = 1.0f;
    int32_t dst = 0;
    __device__ inline void load(const GemmArgs &p, const IndexScratch &s, int row0, int rows)
    {
        if ((int)threadIdx.x < BM) {
            const int i = min((int)threadIdx.x, rows - 1), r = row0 + i;
            if (p.row_pow) pow = p.row_pow[source_row(p, s, row0, i)].y;     // (a row of A's: factors go with what was converted)
            dst = r;
            if (p.out_dst) {
                dst = p.out_dst[r];
                scale = p.out_scale[dst];
            }
        }
    }
    __device__ inline void put(TileRows<BM> &t) const
    {
        if ((int)threadIdx.x < BM) {
            t.pow[threadIdx.x] = pow;
            t.scale[threadIdx.x] = scale;
            t.dst[threadIdx.x] = dst;
        }
    }
};

// acc[m][t][q], m < TM, t < 2, q < NQ: the wavefront's part of the tile.  Register q is row
// 32 m + rq + 8 (q / 4) + 4 (lane / 32) + q % 4, channel chan0 + 32 t + lane % 32.  cs, bias: the lane's channel
// factors.  patch: kPatchBytes<NQ> of LDS that no other wavefront uses.
template <int TM, int NQ, int BM, class Acc>
__device__ inline void finish_tile(const GemmArgs &p, Acc &acc, const TileRows<BM> &tr, const float (&cs)[2], const float (&bias)[2],
                                   int rows, int rq, int chan0, uint8_t *patch)
{
    const int lane = threadIdx.x & 63, ch = lane & 31, r4 = 4 * (lane >> 5);
#pragma unroll
    for (int m = 0; m < TM; ++m) {
        if (32 * m >= rows) break;
        float v[2][NQ];
        auto each = [&](auto f) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < NQ; ++q) f(t, q);
        };
        // a row factor per element: four consecutive rows per read
        auto with_rows = [&](const float *rowv, auto f) {
#pragma unroll
            for (int g = 0; g < NQ / 4; ++g) {
                const float4 w = *reinterpret_cast<const float4 *>(rowv + 32 * m + rq + 8 * g + r4);
                const float fr[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int i = 0; i < 4; ++i) f(t, 4 * g + i, fr[i]);
            }
        };
        if (p.row_pow) with_rows(tr.pow, [&](int t, int q, float w) { v[t][q] = fmaf(acc[m][t][q] * cs[t], w, bias[t]); });
        else each([&](int t, int q) { v[t][q] = fmaf(acc[m][t][q], cs[t], bias[t]); });
        if (p.act == MOE_ACT_RELU) each([&](int t, int q) { v[t][q] = activate(v[t][q], MOE_ACT_RELU); });
        else if (p.act == MOE_ACT_GELU) each([&](int t, int q) { v[t][q] = activate(v[t][q], MOE_ACT_GELU); });
        if (p.out_dst) with_rows(tr.scale, [&](int t, int q, float w) { v[t][q] *= w; });

        auto store = [&](auto out_tag) {
            using OT = decltype(out_tag);                            // float | _Float16 | __bf16
            constexpr bool WIDE = sizeof(OT) == 4;                   // a patch row holds 32 fp32 channels or 64 16-bit channels
            OT *out = reinterpret_cast<OT *>(p.out);
#pragma unroll
            for (int h = 0; h < (WIDE ? 2 : 1); ++h) {
                OT *w = reinterpret_cast<OT *>(patch + r4 * kPatchRow) + ch;
#pragma unroll
                for (int q = 0; q < NQ; ++q)
#pragma unroll
                    for (int t = WIDE ? h : 0; t < (WIDE ? h + 1 : 2); ++t)
                        w[(8 * (q >> 2) + (q & 3)) * (kPatchRow / sizeof(OT)) + (WIDE ? 0 : 32 * t)] = (OT)v[t][q];
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");       // other lanes' writes, same wavefront
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int it = 0; it < NQ / 4; ++it) {
                    const int lr = 8 * it + (lane >> 3), row = 32 * m + rq + lr;
                    const uint4 d = *reinterpret_cast<const uint4 *>(patch + lr * kPatchRow + (lane & 7) * 16);
                    if (row < rows)
                        *reinterpret_cast<uint4 *>(reinterpret_cast<uint8_t *>(out + (size_t)tr.dst[row] * p.N + chan0 + (WIDE ? 32 * h : 0)) + (lane & 7) * 16) = d;
                }
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            }
        };
        if (p.out_dtype == MOE_F32) store(float{});
        else if (p.out_dtype == MOE_BF16) store(__bf16{});
        else store(_Float16{});
    }
}

}  // namespace moe
