// moe_quantize_experts: symmetric range-based weight quantisation (Sec. 3.4) producing the
// interchange codes, the fp16 scales and the pre-shuffled offset-binary layout (Sec. 3.4.1)
// that the grouped FFN kernels stream.
#include <type_traits>

#include "moe_common.h"

namespace moe {

// A unit is one scale group (g rows of K; the whole K range for per-channel scales) of one 32-channel slab.  WU wavefronts
// share a unit; a wavefront owns whole fragment blocks (64 rows with 4-bit, 32 rows with 8-bit codes), lane l the rows and
// the channel whose codes are lane l's 16 bytes of the packed block: it reads 128-byte row segments (two rows per
// instruction) and stores 1 KB per block.  What bounds it is reading the fp32 masters, so they are read once: 128 rows per
// wavefront stay in registers between the search for the largest magnitude and the conversion, and only rows
// beyond WU x 128 are read a second time.  A compute unit has room for two blocks, so what a block takes to convert is time in which
// little is being read: the codes are put together by fp32 multiply-adds, and masters that no cache holds and that are read once
// (NT) are loaded non-temporal.  (32 experts of 1024 x 4096, 4-bit: 332 us with two reads in strips, 143 with shifts and plain loads, 129 with
// multiply-adds, 122 with both, 5.0 TB/s; 8-bit 147 -> 134; groups of 128 124 -> 108; 4096 x 1024, which is read twice: 174 -> 171.)
//
// CH: channels of a unit.  Long units (per-channel scales of more than 2048 rows) of a few slabs leave compute units idle and are read twice: there a
// slab is cut into units of sixteen or eight channels, PARTS of them, and a wavefront takes that many blocks of rows side by side, so the same registers hold
// two or four times the rows.  A row segment is then 64 or 32 bytes, which is slower per byte: only where it fills the chip (see quantize_channels).
template <int BITS, int WU, bool CANON, bool NT, int CH>
__global__ __launch_bounds__(WU == 16 ? 1024 : 512) void quantize_kernel(const float *__restrict__ w, int K, int N, int g,
                                                                         long units, int8_t *__restrict__ q_canon,
                                                                         __half *__restrict__ scales,
                                                                         uint8_t *__restrict__ q_packed)
{
    constexpr int QMAX = BITS == 8 ? 127 : 7;
    constexpr int FK = BITS == 4 ? 64 : 32;             // rows of a fragment block
    constexpr int J = FK / 16;                          // octets of rows per lane and block
    constexpr int FB = 128 / FK;                        // blocks a wavefront keeps
    constexpr int UPB = (WU == 16 ? 16 : 8) / WU;       // units per workgroup
    constexpr int PARTS = 32 / CH;                      // units of a slab, and blocks of rows side by side in a wavefront
    __shared__ float s_amax[UPB][WU][CH];
    __shared__ __align__(16) uint8_t s_canon[CANON ? UPB * WU : 1][CANON ? FK * 32 * BITS / 8 : 16];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = wave / WU, wu = wave % WU;
    const int nl = lane % CH, half = lane / CH & 1, side = lane / (2 * CH);
    const int nslab = N / 32, G = K / g;
    // [expert][group][slab]: neighbouring workgroups read neighbouring columns; the parts of a slab, which share its lines, run side by
    // side on one XCD
    const long unit = PARTS == 1 ? (long)blockIdx.x * UPB + sub : (long)(blockIdx.x / (8 * PARTS)) * 8 + blockIdx.x % 8;
    const int part = PARTS == 1 ? 0 : blockIdx.x / 8 % PARTS;
    const bool live = unit < units;
    const long u = live ? unit : units - 1;
    const int nb = (int)(u % nslab), gi = (int)(u / nslab % G);
    const long e = u / nslab / G;
    const int n = nb * 32 + part * CH + nl;
    const int nblk = g / FK;                            // fragment blocks of the unit
    const int nrun = (nblk + PARTS - 1) / PARTS;        // runs of PARTS blocks, of which a lane has one
    auto block_of = [&](int r) { return PARTS == 1 ? r : min(r * PARTS + side, nblk - 1); };      // (past the last one: that one again)
    const float *base = w + ((size_t)e * K + (size_t)gi * g) * N + n;

    // rows FK b + 16 j + 8 half + i of the unit, b the lane's block of run r
    auto fetch = [&](int r, float (&v)[J][8]) __attribute__((always_inline)) {
        const float *p = base + (size_t)(block_of(r) * FK + 8 * half) * N;
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) v[j][i] = NT ? __builtin_nontemporal_load(p + (size_t)(16 * j + i) * N) : p[(size_t)(16 * j + i) * N];
    };
    auto largest = [&](const float (&v)[J][8], float m) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) m = fmaxf(m, fabsf(v[j][i]));
        return m;
    };
    float keep[FB][J][8];
    float amax = 0.0f;
#pragma unroll
    for (int f = 0; f < FB; ++f)
        if (f * WU + wu < nrun) fetch(f * WU + wu, keep[f]);
#pragma unroll
    for (int f = 0; f < FB; ++f)
        if (f * WU + wu < nrun) amax = largest(keep[f], amax);
    for (int r = FB * WU + wu; r < nrun; r += WU) {
        float v[J][8];
        fetch(r, v);
        amax = largest(v, amax);
    }
#pragma unroll
    for (int off = CH; off < 64; off *= 2) amax = fmaxf(amax, __shfl_xor(amax, off));
    if (WU > 1) {
        if (lane < CH) s_amax[sub][wu][nl] = amax;
        __syncthreads();
        amax = s_amax[sub][0][nl];
#pragma unroll
        for (int q = 1; q < WU; ++q) amax = fmaxf(amax, s_amax[sub][q][nl]);
    }
    if (!live) return;                                  // (no barrier follows)
    // Every load so far has been used, which the compiler loses sight of behind the branches above: a conversion would wait for them again, and with them for the stores
    // of the one before (32 experts of 1024 x 4096: 4-bit 119.3 -> 116.5 us, with canonical codes 163.8 -> 157.2, 8-bit 133.6 -> 125.9).
    __builtin_amdgcn_s_waitcnt(0x0f70);                 // (vmcnt 0)
    const __half sh = __float2half_rn(amax / (float)QMAX);   // IEEE divide, round to nearest even
    const float s = __half2float(sh);
    if (wu == 0 && lane < CH) scales[((size_t)e * G + gi) * N + n] = sh;

    // w / s, correctly rounded: with y = 1/s rounded to nearest and a quotient within one unit in the last place, one
    // residual step gives the correctly rounded quotient (Markstein); the first step makes it that accurate.  A scale of zero
    // has codes of zero, an infinite one as well, but for the infinite weights that it may come from (inf / inf: the lowest code).
    const bool finite = s <= 65504.0f;
    const float y = s != 0.0f && finite ? 1.0f / s : 0.0f, sd = finite ? s : 0.0f, lim = s != 0.0f ? (float)QMAX : 0.0f;
    auto code_of = [&](float x) __attribute__((always_inline)) -> float {
        float q = x * y;
        q = fmaf(fmaf(-q, sd, x), y, q);
        q = fmaf(fmaf(-q, sd, x), y, q);
        return __builtin_amdgcn_fmed3f(rintf(q), -lim, lim);
    };
    auto convert = [&](int r, const float (&v)[J][8]) __attribute__((always_inline)) {
        uint32_t word[4];
        float fc[J][8];
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int i = 0; i < 8; ++i) fc[j][i] = code_of(v[j][i]);
        // codes are put together as sums of fp32 numbers below 2^24, which are exact: fewer steps than shifts of each
        if (BITS == 4) {
#pragma unroll
            for (int j = 0; j < J; ++j) {       // nibble positions 0,4,1,5,2,6,3,7: even codes in the lower half, odd ones in the upper
                float h[2];
#pragma unroll
                for (int o = 0; o < 2; ++o) h[o] = fmaf(fc[j][6 + o], 4096.0f, fmaf(fc[j][4 + o], 256.0f, fmaf(fc[j][2 + o], 16.0f, fc[j][o] + 34952.0f)));
                word[j] = (uint32_t)h[0] | (uint32_t)h[1] << 16;
            }
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                float h[2];
#pragma unroll
                for (int o = 0; o < 2; ++o) h[o] = fmaf(fc[q >> 1][4 * (q & 1) + 2 * o + 1], 256.0f, fc[q >> 1][4 * (q & 1) + 2 * o] + 32896.0f);
                word[q] = (uint32_t)h[0] | (uint32_t)h[1] << 16;
            }
        }
        int code[CANON ? J : 1][8];
        if constexpr (CANON)
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int i = 0; i < 8; ++i) code[j][i] = (int)fc[j][i];
        const int kb = gi * nblk + block_of(r);
        if (q_packed && (PARTS == 1 || r * PARTS + side < nblk))
            *reinterpret_cast<uint4 *>(q_packed + (size_t)e * packed_bytes_per_expert(K, N, BITS) + ((size_t)nb * (K / FK) + kb) * kFragBytes +
                                       (half * 32 + part * CH + nl) * 16) = make_uint4(word[0], word[1], word[2], word[3]);
        if constexpr (CANON) {
            // the block's rows meet in the wavefront's own piece of LDS (served in order: no barrier) and leave 16 bytes per lane
            constexpr int ROW = CH * BITS / 8;          // bytes of a row
            uint8_t *tile = s_canon[sub * WU + wu];
#pragma unroll
            for (int j = 0; j < J; ++j)
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int row = side * FK + 16 * j + 8 * half + i;
                    if (BITS == 8) {
                        tile[row * ROW + nl] = (uint8_t)code[j][i];
                    } else {
                        const int other = __builtin_amdgcn_update_dpp(0, code[j][i], 0xB1, 0xf, 0xf, false);     // the neighbouring channel's code
                        if (!(lane & 1)) tile[row * ROW + (nl >> 1)] = (uint8_t)((code[j][i] & 0xf) | ((other & 0xf) << 4));
                    }
                }
            __builtin_amdgcn_wave_barrier();
            if constexpr (ROW >= 16 && PARTS == 1) {
                constexpr int VPR = ROW / 16;           // 16-byte vectors per row
                const uint4 v = *reinterpret_cast<const uint4 *>(tile + lane * 16);
                *reinterpret_cast<uint4 *>(reinterpret_cast<uint8_t *>(q_canon) + (((size_t)e * K + (size_t)kb * FK + lane / VPR) * N + nb * 32) * BITS / 8 + (lane % VPR) * 16) = v;
            } else {
                auto leave = [&](auto vec, int at) __attribute__((always_inline)) {      // the tile's bytes from `at` on, a piece of one row
                    const int row = at / ROW;
                    if (r * PARTS * FK + row >= g) return;                               // (the rows of a last block that is there again)
                    *reinterpret_cast<decltype(vec) *>(reinterpret_cast<uint8_t *>(q_canon) +
                                                       (((size_t)e * K + (size_t)gi * g + (size_t)r * PARTS * FK + row) * N + nb * 32 + part * CH) * BITS / 8 + at % ROW) =
                        *reinterpret_cast<const decltype(vec) *>(tile + at);
                };
                if constexpr (ROW >= 16) leave(uint4{}, lane * 16);
                else if constexpr (ROW == 8) leave(uint2{}, lane * 8), leave(uint2{}, 512 + lane * 8);
                else
#pragma unroll
                    for (int i = 0; i < 4; ++i) leave(uint32_t{}, 256 * i + lane * 4);
            }
            __builtin_amdgcn_wave_barrier();
        }
    };
#pragma unroll
    for (int f = 0; f < FB; ++f)
        if (f * WU + wu < nrun) convert(f * WU + wu, keep[f]);
    for (int r = FB * WU + wu; r < nrun; r += WU) {
        float v[J][8];
        fetch(r, v);
        convert(r, v);
    }
}

template <int BITS, int WU, int CH = 32>
static void launch_quantize(const float *w, int E, int K, int N, int g, void *q_canon, void *scales, void *q_packed, hipStream_t s)
{
    constexpr int UPB = (WU == 16 ? 16 : 8) / WU;
    const long units = (long)E * (K / g) * (N / 32);
    static_assert(CH == 32 || UPB == 1, "parts of a slab are workgroups");
    const dim3 grid((unsigned)(CH == 32 ? (units + UPB - 1) / UPB : (units + 7) / 8 * 8 * (32 / CH))), block(WU == 16 ? 1024 : 512);
    // masters larger than the L2s together, units that the registers hold (a second read finds part of its rows in the last-level cache: 4096 x
    // 1024 171 us plain, 184 non-temporal; one expert of 1024 x 4096 just written 7.8 and 8.5)
    const bool nt = CH == 32 && (size_t)E * K * N >= (size_t)16 << 20 && g <= WU * 128;      // (parts share lines)
    auto launch = [&](auto canon, auto once) {
        hipLaunchKernelGGL((quantize_kernel<BITS, WU, decltype(canon)::value, decltype(once)::value, CH>), grid, block, 0, s, w, K, N, g, units, (int8_t *)q_canon,
                           (__half *)scales, (uint8_t *)q_packed);
    };
    if (q_canon) nt ? launch(std::true_type{}, std::true_type{}) : launch(std::true_type{}, std::false_type{});
    else nt ? launch(std::false_type{}, std::true_type{}) : launch(std::false_type{}, std::false_type{});
}

// Channels of a unit of more than 2048 rows: all of a slab while the slabs fill half of the compute units or more, else as few as leave a compute unit to
// each block.  us, units of 32 / 16 / 8 channels: one expert of 4096 x 1024, 4-bit (32 slabs) 17.9 / 12.8 / 11.0, 8-bit 18.3 / 13.4 / 10.9, of 8192 x 2048 (64)
// 37.5 / 29.0 / 22.0, of 16384 x 4096 (128) 125 / 103 / 149; four of 4096 x 1024 (128) 23.3 / 18.6 / 22.2, two of 8192 x 2048 (128) 57 / 48 / 66; eight of 3072 x 768
// (192) 21.8 / 23.3 / 26.7, 32 of 4096 x 1024 (1024) 174 / 183 / 257.
static int quantize_channels(long slabs) { return slabs <= 64 ? 8 : slabs <= 128 ? 16 : 32; }

// Wavefronts per unit: the fewest whose registers hold the unit (128 rows each), sixteen for the longest.
template <int BITS>
static void launch_quantize_bits(const float *w, int E, int K, int N, int g, void *q_canon, void *scales, void *q_packed, hipStream_t s)
{
    if (g <= 128) launch_quantize<BITS, 1>(w, E, K, N, g, q_canon, scales, q_packed, s);
    else if (g <= 512) launch_quantize<BITS, 4>(w, E, K, N, g, q_canon, scales, q_packed, s);
    else if (g <= 1024) launch_quantize<BITS, 8>(w, E, K, N, g, q_canon, scales, q_packed, s);
    else {
        const int ch = g <= 2048 ? 32 : quantize_channels((long)E * (K / g) * (N / 32));
        if (ch == 32) launch_quantize<BITS, 16>(w, E, K, N, g, q_canon, scales, q_packed, s);
        else if (ch == 16) launch_quantize<BITS, 16, 16>(w, E, K, N, g, q_canon, scales, q_packed, s);
        else launch_quantize<BITS, 16, 8>(w, E, K, N, g, q_canon, scales, q_packed, s);
    }
}

// Unquantised fp16 weights in the fragment layout (one MFMA step, 16 K values, per 1 KB block):
// lane l of block (nb, kb) holds w[16 kb + 8 (l >> 5) + 0..7][32 nb + (l & 31)].
__global__ __launch_bounds__(256) void pack_f16_kernel(const float *__restrict__ w, int K, int N,
                                                       uint16_t *__restrict__ packed)
{
    const int e = blockIdx.z, kb = blockIdx.y;
    const int nb = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (nb >= N / 32) return;
    const int n = nb * 32 + (lane & 31), k0 = kb * 16 + 8 * (lane >> 5);
    uint16_t v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const __half h = __float2half_rn(w[((size_t)e * K + k0 + i) * N + n]);
        v[i] = *reinterpret_cast<const uint16_t *>(&h);
    }
    uint16_t *dst = packed + (size_t)e * K * N + (((size_t)nb * (K / 16) + kb) * 64 + lane) * 8;
    *reinterpret_cast<uint4 *>(dst) = make_uint4(v[0] | (uint32_t)v[1] << 16, v[2] | (uint32_t)v[3] << 16,
                                                 v[4] | (uint32_t)v[5] << 16, v[6] | (uint32_t)v[7] << 16);
}

}  // namespace moe

extern "C" int moe_pack_fp16_experts(const float *w, int E, int K, int N, void *w_packed, void *stream)
{
    using namespace moe;
    if (!w || !w_packed) return fail(MOE_ERR_INVALID_ARG, "moe_pack_fp16_experts: NULL pointer");
    if (E <= 0 || K <= 0 || N <= 0) return fail(MOE_ERR_INVALID_ARG, "moe_pack_fp16_experts: E, K, N must be positive");
    if (N % 32 || K % 16) return fail(MOE_ERR_INVALID_ARG, "moe_pack_fp16_experts: need N %% 32 == 0 and K %% 16 == 0 (K=%d N=%d)", K, N);
    if (E > 65535 || K / 16 > 65535) return fail(MOE_ERR_UNSUPPORTED, "moe_pack_fp16_experts: too many experts or K blocks for one launch");
    if (!aligned16(w) || !aligned16(w_packed)) return fail(MOE_ERR_INVALID_ARG, "moe_pack_fp16_experts: buffers must be 16-byte aligned");
    dim3 grid((N / 32 + 3) / 4, K / 16, E);
    hipLaunchKernelGGL(pack_f16_kernel, grid, dim3(256), 0, as_stream(stream), w, K, N, (uint16_t *)w_packed);
    return check_launch("moe_pack_fp16_experts");
}

extern "C" int moe_quantize_experts(const float *w, int E, int K, int N, int bits, int group_size,
                                    void *q_canon, void *scales, void *q_packed, void *stream)
{
    using namespace moe;
    if (!w || !scales) return fail(MOE_ERR_INVALID_ARG, "moe_quantize_experts: w and scales must not be NULL");
    if (E <= 0 || K <= 0 || N <= 0) return fail(MOE_ERR_INVALID_ARG, "moe_quantize_experts: E, K, N must be positive");
    if (bits != 4 && bits != 8) return fail(MOE_ERR_UNSUPPORTED, "moe_quantize_experts: bits must be 4 or 8 (got %d)", bits);
    if (N % 32 || K % 64) return fail(MOE_ERR_INVALID_ARG, "moe_quantize_experts: need N %% 32 == 0 and K %% 64 == 0 (K=%d N=%d)", K, N);
    const int g = (group_size == 0 || group_size == K) ? K : group_size;
    if (g < 0 || g % 64 || K % g) return fail(MOE_ERR_INVALID_ARG, "moe_quantize_experts: group_size %d must be a multiple of 64 dividing K=%d", group_size, K);
    if (E > 65535 || K / g > 65535) return fail(MOE_ERR_UNSUPPORTED, "moe_quantize_experts: too many experts or groups for one launch");
    if (!aligned16(w) || !aligned16(scales) || !aligned16(q_canon) || !aligned16(q_packed))
        return fail(MOE_ERR_INVALID_ARG, "moe_quantize_experts: buffers must be 16-byte aligned");
    if ((long)E * (K / g) * (N / 32) > 0x7fffffffL) return fail(MOE_ERR_UNSUPPORTED, "moe_quantize_experts: too many slabs for one launch");
    if (bits == 8) launch_quantize_bits<8>(w, E, K, N, g, q_canon, scales, q_packed, as_stream(stream));
    else launch_quantize_bits<4>(w, E, K, N, g, q_canon, scales, q_packed, as_stream(stream));
    return check_launch("moe_quantize_experts");
}
