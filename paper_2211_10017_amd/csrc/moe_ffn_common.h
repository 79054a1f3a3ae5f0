// Device helpers shared by the grouped-GEMM kernels: argument block, the magic-number
// integer-to-FP16 conversions (Sec. 3.4.1-3.4.3) and the tile lookup.
#pragma once

#include "moe_common.h"

namespace moe {

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));

// SCALE_CHANNEL_BF16: the rows are bf16 and meet the codes, exact in bf16, in bf16 matrix instructions.
enum { SCALE_CHANNEL = 0, SCALE_GROUP = 1, SCALE_GROUP_SPLIT = 2, SCALE_GROUP_ACC = 3, SCALE_CHANNEL_BF16 = 4 };
constexpr bool channel_scales(int smode) { return smode == SCALE_CHANNEL || smode == SCALE_CHANNEL_BF16; }

struct GemmArgs {
    const uint16_t *a;        // [R, K] fp16 bit patterns (rows that were bf16 come converted, scaled by 2^-p per row, or, SCALE_CHANNEL_BF16, as they are)
    const float2 *row_pow;    // null, or per row (2^-p, 2^p): the tiled kernel multiplies its output rows by 2^p
    const int32_t *offsets;   // [E+1]
    const uint8_t *wq;        // packed codes, [E] x packed_bytes_per_expert
    const __half *scales;     // [E, K/g, N]
    const __half *bias;       // [E, N] or null
    void *out;                // [R, N]
    int E, R, K, N, g;
    int out_dtype;
    int act;                  // MOE_ACT_NONE (plain GEMM) | MOE_ACT_RELU | MOE_ACT_GELU applied after the bias
    int tile_units;           // tiled kernel: row tiles of at most 32 * tile_units rows (set by the launcher)
    int indexed;              // of a call whose rows come through the routing index: both its GEMMs run in row tiles
    int ring_long;            // ring kernel: whether a block may have its compute unit's LDS to itself (set by the launcher)
    // tiled kernel only: rows fetched / stored through the routing index instead of a permuted copy
    const int32_t *a_src;     // [R] or null: row r of A is a[a_src[r] / a_div]
    int a_div;
    const int32_t *out_dst;   // [R] or null: row r of the result goes to out[out_dst[r]], times out_scale[out_dst[r]]
    const float *out_scale;
    // straight-line streaming kernel (decode-sized batches) and row tiles: the permutation is rebuilt from the
    // gate's output inside the launch.  gate_idx[a] is the expert of assignment a (E = pruned row),
    // row a / gate_k of `a` is its token; the first block of every expert (or row tile) writes the index arrays.
    const int32_t *gate_idx;  // [n_assign] or null
    int n_assign, gate_k;
    int32_t *perm_src_out, *inv_perm_out, *offsets_out;
    float *zero_out;          // or null: fp32 buffer the launch clears (zero_count floats, a multiple of 4) for the
    long zero_count;          // launch after it, which adds rows into it
    // straight-line streaming kernel, fused un-permute for k <= 2: with out_add set, row r of the result,
    // times out_scale[a], a = out_dst[r], is ADDED to row a / out_div of the fp32 buffer `out` (cleared
    // before).  A token's at most two terms arrive in either order; fp32 addition of two terms onto
    // zero is commutative, so the sum does not depend on it.
    int out_add, out_div;
};

// FFN of a decode-sized batch: one streaming launch plus a small reduction (moe_ffn_decode.hip).
struct DecodeArgs {
    const uint16_t *x;          // [T, d] un-permuted, fp16 or bf16
    const int32_t *gate_idx;    // [n_assign] expert of assignment a (E = pruned row)
    const float *gate_scale;    // [n_assign] gate scale of assignment a
    int n_assign, gate_k;
    int E, d, F, act;
    int g;                      // group size of the scales, 0 = per channel
    uint32_t group_inv;         // 2^32 / (g / 64), rounded up, 0 for groups of 64 (set by the launcher)
    int cw;                     // channels of d_ff per slice, in 64s: 1, 2, 4 or 8
    int row_tiles;              // sixteens of rows per item: 1 or 2 (set by the launcher)
    const uint8_t *w1, *w2;     // packed codes
    const __half *s1, *s2;      // scales [E, d / g, F] / [E, F / g, d], one row per expert for channel scales
    const __half *b1, *b2;      // biases or null
    float *partial;             // [F / (64 cw), n_assign, d] fp32: y of every assignment summed over one slice of d_ff
    void *out;                  // [T, d] layer output
    int out_dtype;
    int32_t *perm_src_out, *inv_perm_out, *offsets_out;
};
constexpr int kDecMaxExperts = 4096;
constexpr int kDecMaxAssign = 512;
bool decode_ffn_supports(int n_assign, int k, int E, int d, int F, int bits, int group_size);
size_t decode_ffn_partial_bytes(int n_assign, int d, int F, int cw);
int decode_slice_width(int n_assign, int E, int F);
double decode_active_experts(int n_assign, int E);
int launch_decode_ffn(const DecodeArgs &p, int bits, bool bf, hipStream_t s);

constexpr int kGatedMaxAssign = 256;    // assignments the fused permutation takes: one per thread of a block
constexpr int kUnsortedMaxAssign = 4096, kUnsortedMaxExperts = 1024;    // of row tiles that sort for themselves: sixteen keys per thread

int launch_tiled_gemm(const GemmArgs &p, int bits, int smode, hipStream_t s);
double row_tile_blocks(const GemmArgs &p, int bits, int smode);
double expected_row_tiles(long R, long E, int bm);
bool bf16_codes_pay(int R, int tokens, int E, int d, int F, int bits, bool indexed);
void launch_tiled_4(const GemmArgs &p, int smode, int tm, dim3 grid, hipStream_t s);
void launch_tiled_4_exact(const GemmArgs &p, int smode, int tm, dim3 grid, hipStream_t s);
void launch_tiled_8(const GemmArgs &p, int smode, int tm, dim3 grid, hipStream_t s);
void launch_tiled_8_exact(const GemmArgs &p, int smode, int tm, dim3 grid, hipStream_t s);
void launch_ring_4(const GemmArgs &p, int smode, int bm, dim3 grid, hipStream_t s);
void launch_ring_8(const GemmArgs &p, int smode, int bm, dim3 grid, hipStream_t s);
int launch_stream_gemm(const GemmArgs &p, int bits, int smode, int max_rows, hipStream_t s);
bool stream_gemm_supports(int K, int bits, int smode);
int stream_gemm_fit_rows(int K);
bool stream_unrolled_supports(int K, int bits, int smode);
int stream_unrolled_fit(int K, int max_rows);
bool stream_unrolled_takes_gate(int K, int bits);
int launch_stream_unrolled(const GemmArgs &p, int bits, int max_rows, hipStream_t s);
int launch_stream_unrolled_variant(const GemmArgs &p, int bits, bool native, int max_rows, hipStream_t s);

enum { MOE_ACT_NONE = -1 };

// GELU in its exact form v * Phi(v) = max(v, 0) - |v| Phi(-|v|), without a branch: with b = |v| / 2, log2(2 Phi(-2 b)) is b times a
// polynomial of degree nine (a weighted minimax fit on [0, 3]; beyond, it falls without end, so that the second term vanishes; b stops
// at 16, which keeps infinities out of the product).  Against 64 bits, normally distributed v of standard deviation 0.02 to 3:
// error 0.7 to 0.85 times, largest error 0.5 to 0.95 times that of 0.5 v (1 + erff(v / sqrt 2)).  What bounds the end of a tile is its vector
// instructions, and erff runs both of its branches on nearly every wavefront.  16384 tokens of
// 1024 x 4096, 64 experts, 4-bit: a step with GELU 385 -> 359 us (ReLU 334); 997 bf16 tokens of 768 x 3072 71 -> 66.5 (64).
__device__ inline float gelu(float v)
{
    const float a = 0.5f * fabsf(v), b = fminf(a, 16.0f);
    float q = -4.015279e-05f;
    q = __builtin_fmaf(q, b, 0.0005579601f);
    q = __builtin_fmaf(q, b, -0.0033400627f);
    q = __builtin_fmaf(q, b, 0.011037564f);
    q = __builtin_fmaf(q, b, -0.019550677f);
    q = __builtin_fmaf(q, b, 0.0012326466f);
    q = __builtin_fmaf(q, b, 0.110654876f);
    q = __builtin_fmaf(q, b, -0.41943568f);
    q = __builtin_fmaf(q, b, -1.8368893f);
    q = __builtin_fmaf(q, b, -2.3022084f);
    return __builtin_fmaf(-b, __builtin_amdgcn_exp2f(q * b), __builtin_fmaf(0.5f, v, a));
}

// The activation between the two GEMMs.
__device__ inline float activate(float v, int act)
{
    if (act == MOE_ACT_RELU) return fmaxf(v, 0.0f);
    if (act == MOE_ACT_GELU) return gelu(v);
    return v;
}

__device__ inline uint32_t h2_bits(half2_t v) { return __builtin_bit_cast(uint32_t, v); }
__device__ inline half2_t bits_h2(uint32_t v) { return __builtin_bit_cast(half2_t, v); }

// Sec. 3.4.1: OR-ing an unsigned code Y < 1024 into the mantissa of FP16 1024.0 (0x6400) gives
// the FP16 number 1024 + Y; an FP16 subtraction of 1024 + offset returns the signed integer,
// exactly.  Two codes are converted per 32-bit register.
//
// 4-bit (Sec. 3.4.3): the eight codes of a dword sit in nibble positions 0,4,1,5,2,6,3,7, so
// (x & 0x000f000f) | 0x64006400 is the pair (i0, i1) + 1024 and (x & 0x00f000f0) | 0x64006400 is
// 16 * (i2, i3) + 1024; the latter is brought back with one fma: v/16 - (64 + 8).
// A register-to-register move that the compiler cannot fold away.
__device__ inline uint32_t opaque_copy(uint32_t x)
{
    uint32_t r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

// (x & mask) | magic in one VALU instruction.  The compiler prefers two VOP2 instructions with
// literal operands here (VOP3 cannot encode literals on this target), so the instruction is
// spelled out, with mask and magic held in registers.
__device__ inline uint32_t and_or(uint32_t x, uint32_t mask, uint32_t magic)
{
    uint32_t r;
    asm("v_and_or_b32 %0, %1, %2, %3" : "=v"(r) : "v"(x), "v"(mask), "v"(magic));
    return r;
}

__device__ inline void dequant4(uint32_t x, uint32_t out[4])
{
    const uint32_t magic = 0x64006400u, mlo = 0x000f000fu, mhi = 0x00f000f0u;
    const half2_t sub = {(_Float16)1032.0f, (_Float16)1032.0f};
    const half2_t sixteenth = {(_Float16)0.0625f, (_Float16)0.0625f};
    const half2_t sub16 = {(_Float16)72.0f, (_Float16)72.0f};
    const uint32_t lo0 = and_or(x, mlo, magic);
    const uint32_t hi0 = and_or(x, mhi, magic);
    x >>= 8;
    const uint32_t lo1 = and_or(x, mlo, magic);
    const uint32_t hi1 = and_or(x, mhi, magic);
    out[0] = h2_bits(bits_h2(lo0) - sub);
    out[1] = h2_bits(bits_h2(hi0) * sixteenth - sub16);
    out[2] = h2_bits(bits_h2(lo1) - sub);
    out[3] = h2_bits(bits_h2(hi1) * sixteenth - sub16);
}

// 8-bit (Sec. 3.4.2): four codes (+128) per dword; a byte permute builds 0x64xx64yy for two of
// them at a time, and an FP16 subtraction of 1152 = 1024 + 128 returns the signed integers.
__device__ inline void dequant8(uint32_t w0, uint32_t w1, uint32_t out[4])
{
    const half2_t sub = {(_Float16)1152.0f, (_Float16)1152.0f};
    const uint32_t magic = 0x64646464u;
    out[0] = h2_bits(bits_h2(__builtin_amdgcn_perm(magic, w0, 0x04010400u)) - sub);
    out[1] = h2_bits(bits_h2(__builtin_amdgcn_perm(magic, w0, 0x04030402u)) - sub);
    out[2] = h2_bits(bits_h2(__builtin_amdgcn_perm(magic, w1, 0x04010400u)) - sub);
    out[3] = h2_bits(bits_h2(__builtin_amdgcn_perm(magic, w1, 0x04030402u)) - sub);
}

// 4-bit codes times their group's scale in one instruction after the unpacking.  FP16 numbers below 2^-13 are whole multiples of 2^-24, bits and
// value in proportion, so a code Y that stands in the low bits of a half by itself is the number Y 2^-24 (2^-20 four bits up), and
// Y 2^-24 * (2^24 s) - 8 s is (Y - 8) s with one rounding, as code times scale is: 8 s is exact, where 1032 s, what the
// 0x6400 form would take off, is not.  9 instructions per eight codes instead of 13.
// 2^24 s has to be an FP16 number and s itself a normal one: the caller scales s by a power of two per channel, 2^unit = 2^24 / 2^t,
// which the accumulator column is then in units of, and takes only what `scale_in_window` accepts.
// What bounds a tile of many rows is the power of matrix and conversion work together.  A step of 8192 tokens, two of 64 experts of
// 4096 x 16384, groups of 128: 4375 -> 4268 us, bf16 (fc2 only) 4642 -> 4601; 2048 tokens, two of 16 experts of 2048 x 8192, 337 -> 328; same bits.
constexpr int kWindowShift = 24;
__device__ inline bool scale_in_window(_Float16 m)        // 2^10 <= m < infinity (and not negative, not a NaN)
{
    return (uint16_t)(__builtin_bit_cast(uint16_t, m) - 0x6400u) < 0x1800u;
}

// Brings s to [2^13, 2^14): room for a factor of 4 up and of 8 down.
__device__ inline int window_unit(_Float16 s) { return 14 - __builtin_amdgcn_frexp_exph(s); }

struct ScaledCodes {
    half2_t lo, hi, off;
    ScaledCodes() = default;
    __device__ inline explicit ScaledCodes(_Float16 m)     // m = 2^24 s
    {
        lo = half2_t{m, m};
        hi = lo * half2_t{(_Float16)0.0625f, (_Float16)0.0625f};
        off = lo * half2_t{(_Float16)-0x1p-21f, (_Float16)-0x1p-21f};
    }
    __device__ inline void convert(uint32_t x, uint32_t out[4]) const
    {
        auto fma2 = [&](uint32_t y, half2_t f) { return h2_bits(__builtin_elementwise_fma(bits_h2(y), f, off)); };
        const uint32_t x8 = x >> 8;
        out[0] = fma2(x & 0x000f000fu, lo);
        out[1] = fma2(x & 0x00f000f0u, hi);
        out[2] = fma2(x8 & 0x000f000fu, lo);
        out[3] = fma2(x8 & 0x00f000f0u, hi);
    }
};

// Eight codes as exact bf16 numbers q 2^-16, for rows that come as bf16.  A code that stands in a half by itself is Y 2^-24 (see ScaledCodes), or Y 2^-20,
// and one mixed multiply-add makes (Y - 2^(B-1)) 2^-16 of it in FP32; there is no packed bf16 arithmetic, so every code is converted on its own,
// 16 or 17 instructions for eight instead of 8 or 9.  What that saves is a pass over the rows of x and of h to bring them to scaled FP16, a launch and a
// read and write each.
// 2^-16: products of bf16 numbers, whole multiples of 2^-133, with the codes are whole multiples of 2^-149, FP32's smallest number, so the sums of rows of any size
// are as exact as those of rows around one, and they overflow from 2^144 on in units of the code: with scales of 2^-16 and more, only where the result does.
constexpr float kBf16CodeUnit = 65536.0f;
template <int BITS>
__device__ inline void codes_to_bf16(const uint32_t *w, uint32_t out[4])
{
    constexpr float LO = 0x1p24f / kBf16CodeUnit, HI = 0x1p20f / kBf16CodeUnit, OFF = (BITS == 4 ? -8.0f : -128.0f) / kBf16CodeUnit;
    auto pair = [&](uint32_t y, float unit) {
        const half2_t v = bits_h2(y);
        const float lo = __builtin_fmaf((float)v[0], unit, OFF), hi = __builtin_fmaf((float)v[1], unit, OFF);
        return __builtin_amdgcn_perm(__float_as_uint(hi), __float_as_uint(lo), 0x07060302u);
    };
    if constexpr (BITS == 4) {
        const uint32_t x = w[0], x8 = x >> 8;
        out[0] = pair(x & 0x000f000fu, LO);
        out[1] = pair(x & 0x00f000f0u, HI);
        out[2] = pair(x8 & 0x000f000fu, LO);
        out[3] = pair(x8 & 0x00f000f0u, HI);
    } else {
#pragma unroll
        for (int q = 0; q < 4; ++q) out[q] = pair(__builtin_amdgcn_perm(0u, w[q >> 1], q & 1 ? 0x0c030c02u : 0x0c010c00u), LO);
    }
}

// The same conversions with the chip's integer-to-float instructions instead of the magic
// number (the variant Sec. 3.4.1 measured as too slow on its hardware): extract the code, convert
// to fp32, remove the offset, round to FP16.  Exact, like the magic-number route.
__device__ inline void dequant4_native(uint32_t x, uint32_t out[4])
{
    // codes of MFMA index i sit in nibble position {0,4,1,5,2,6,3,7}[i]
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float lo = (float)((x >> (4 * q)) & 15u) - 8.0f;        // index 2q
        const float hi = (float)((x >> (4 * q + 16)) & 15u) - 8.0f;   // index 2q + 1
        const half2_t h = {(_Float16)lo, (_Float16)hi};
        out[q] = h2_bits(h);
    }
}

__device__ inline void dequant8_native(uint32_t w0, uint32_t w1, uint32_t out[4])
{
    const uint32_t w[2] = {w0, w1};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float lo = (float)((w[q >> 1] >> (16 * (q & 1))) & 255u) - 128.0f;
        const float hi = (float)((w[q >> 1] >> (16 * (q & 1) + 8)) & 255u) - 128.0f;
        const half2_t h = {(_Float16)lo, (_Float16)hi};
        out[q] = h2_bits(h);
    }
}

__device__ inline half8_t frag_from(const uint32_t w[4])
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    u4 v = {w[0], w[1], w[2], w[3]};
    return __builtin_bit_cast(half8_t, v);
}

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));

// 32 rows x 32 channels x 16 K values of FP16 or bf16 operands
template <bool BF16>
__device__ inline float16_t tile_product(half8_t a, half8_t b, float16_t c)
{
    if constexpr (BF16) return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c, 0, 0, 0);
    else return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

__device__ inline uint16_t to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ inline void store_out(void *out, int dtype, size_t o, float v)
{
    if (dtype == MOE_F32) reinterpret_cast<float *>(out)[o] = v;
    else if (dtype == MOE_BF16) reinterpret_cast<uint16_t *>(out)[o] = to_bf16_rne(v);
    else reinterpret_cast<_Float16 *>(out)[o] = (_Float16)v;
}

// 16 bytes per lane from global memory straight into LDS: lane l's bytes land at dst + 16 l, dst
// the same for the whole wavefront.  Written as assembly so that the compiler's load counter
// does not see it (it would take loads of two kinds to be in flight and wait for all of them at
// the first use of any).  The caller waits for it by hand with wait_loads<N>(), N = the loads
// issued after it that may stay in flight: the counter retires loads in order, and the waits the
// compiler places for its own loads can only be stricter for the ones it does not see.
template <bool NT = false>
__device__ inline void load_to_lds16(const void *src, uint16_t *dst)
{
    const uint32_t l = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst;
    // (NT: non-temporal, for data that is read once)
    if constexpr (NT) asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off nt" ::"v"(src), "s"(l) : "memory", "m0");
    else asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(src), "s"(l) : "memory", "m0");
}

// The same with 4 bytes per lane: lane l's bytes land at dst + 4 l.
__device__ inline void load_to_lds4(const void *src, void *dst)
{
    const uint32_t l = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void *)dst;
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(src), "s"(l) : "memory", "m0");
}

// s_waitcnt vmcnt(N) alone (the other counters' fields say "no wait").
// Built with MOE_WAIT_ALL_LOADS every such wait is for ALL outstanding loads: slower, but free of any
// assumption about how many loads the compiler issues after a direct-to-LDS load.  The library is built
// a second time that way (libmoe_wq_waitall.so) and a GPU test compares the two builds bit for bit, so a
// compiler that merges, splits or reorders one of the counted loads shows up as a failing test, not as
// silently stale rows in LDS.
template <int N>
__device__ inline void wait_loads()
{
    static_assert(N >= 0 && N < 64, "vmcnt has six bits");
#ifdef MOE_WAIT_ALL_LOADS
    __builtin_amdgcn_s_waitcnt(0x0f70);
#else
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0f70);
#endif
}

// Inclusive prefix sum over the 64 lanes in the VALU's data-parallel primitives: shifts by 1, 2, 4
// and 8 inside each row of 16 lanes (zero shifted in), then the last lane of rows 0 and 2 added to rows
// 1 and 3, then lane 31 added to rows 2 and 3.  All lanes must be active.
__device__ inline int wave_inclusive_sum(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);     // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);     // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);     // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);     // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);    // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);    // row_bcast:31 into rows 2 and 3
    return v;
}

// Work distribution of the tiled kernel.  A work item is (expert, column block, row tile); the
// items are ordered expert-major, then by column block, row tile fastest, so that neighbours in
// the order share a weight column block (row tiles of one expert) or an activation row tile
// (column blocks of one expert).  The chip's workgroups go round-robin to its 8 XCDs, each with
// an L2 of its own: workgroup id w runs on XCD w % 8, so XCD x is given the x-th contiguous
// eighth of the order, walked in order by its workgroups w / 8.  What runs together on one XCD
// then streams the same few row tiles and weight blocks through that XCD's L2.
// Every wavefront computes the same answer; returns false when this workgroup has no item.
constexpr int kXcds = 8;

// Expert e's row range, forced into [0, R] and non-negative length: offsets that are not a
// monotone partition of the R rows then give wrong results but no access outside the buffers.
__device__ inline void expert_range(const int32_t *offsets, int e, int R, int *lo, int *hi)
{
    const int l = min(max(offsets[e], 0), R);
    *lo = l;
    *hi = min(max(offsets[e + 1], l), R);
}

template <int UNIT = 32>
__device__ inline bool find_item(const int32_t *offsets, int E, int R, int BM, int ncol, int wg,
                                 int *e_out, int *col, int *row0, int *rows)
{
    const int lane = threadIdx.x & 63;
    // row tiles of the experts of one 64-lane chunk, with their inclusive prefix sum over the chunk
    auto chunk_tiles = [&](int e0, int &lo, int &hi, int &tiles, int &incl) {
        const int e = e0 + lane;
        lo = 0, hi = 0;
        if (e < E) expert_range(offsets, e, R, &lo, &hi);
        tiles = (hi - lo + BM - 1) / BM;
        incl = wave_inclusive_sum(tiles);
    };
    int total = 0;                                     // row tiles of all experts
    int lo0, hi0, tiles0, incl0;                       // the first chunk is kept: with E <= 64 the offsets are read once
    chunk_tiles(0, lo0, hi0, tiles0, incl0);
    total = __shfl(incl0, 63);
    for (int e0 = 64; e0 < E; e0 += 64) {
        int lo, hi, tiles, incl;
        chunk_tiles(e0, lo, hi, tiles, incl);
        total += __shfl(incl, 63);
    }
    const long items = (long)total * ncol;
    const long chunk = (items + kXcds - 1) / kXcds;
    const long s = wg / kXcds;
    const long item = (wg % kXcds) * chunk + s;
    if (s >= chunk || item >= items) return false;
    int base = 0;
    for (int e0 = 0; e0 < E; e0 += 64) {
        int lo = lo0, hi = hi0, tiles = tiles0, incl = incl0;
        if (e0) chunk_tiles(e0, lo, hi, tiles, incl);
        const uint64_t hit = __ballot((long)(base + incl) * ncol > item);
        if (hit) {
            const int src = __ffsll((unsigned long long)hit) - 1;
            const int t_e = __shfl(tiles, src);
            const int excl = __shfl(incl - tiles, src);
            const int local = (int)(item - (long)(base + excl) * ncol);
            const int c = local / t_e, mt = local % t_e;
            const int lo_s = __shfl(lo, src), hi_s = __shfl(hi, src);
            // The expert's rows, in units of UNIT = 32 (one MFMA row tile), are dealt evenly to its t_e
            // tiles: 270 rows become 96 + 96 + 78 rather than 128 + 128 + 14, the same matrix
            // work without a nearly empty tile that streams a whole weight block for 14 rows.
            const int units = (hi_s - lo_s + UNIT - 1) / UNIT, per = units / t_e, extra = units % t_e;
            const int first = lo_s + UNIT * (mt * per + min(mt, extra));
            *e_out = e0 + src;
            *col = c;
            *row0 = first;
            *rows = min(UNIT * (per + (mt < extra ? 1 : 0)), hi_s - first);
            return true;
        }
        base += __shfl(incl, 63);
    }
    return false;
}

// LDS of find_unsorted_item: rows of every expert and where they begin, matches per 64 assignments, the assignments of the tile's rows.
struct IndexScratch {
    int32_t cnt[kUnsortedMaxExperts + 1], off[kUnsortedMaxExperts + 1], match[kUnsortedMaxAssign / 64], row[128];
};

// find_item for a launch of 256-thread blocks that has no index yet: every block counts the gate's output, which gives it the
// offsets and its item, and ranks the item's expert, which gives it the assignments of its rows (s.row).  The blocks of a tile's first column write
// perm_src and inv_perm for the tile's rows, block 0 the offsets and the pruned rows, as moe_permute does.
// What bounds a small batch is its chain of launches, and the index as one of its own is the link that does least.  Here it costs barriers and
// code that no block has run before, so each step over 256 assignments ends the loops that are done with them all.
template <int UNIT = 32>
__device__ inline bool find_unsorted_item(const GemmArgs &p, int BM, int ncol, IndexScratch &s, int *e_out, int *col, int *row0, int *rows)
{
    constexpr int STEPS = kUnsortedMaxAssign / 256;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n = p.n_assign, E = p.E;
    int key[STEPS];
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        if (256 * j >= n) break;
        key[j] = p.gate_idx[min(256 * j + tid, n - 1)];
    }
    for (int i = tid; i <= E; i += 256) s.cnt[i] = 0;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < STEPS; ++j) {
        if (256 * j >= n) break;
        const bool live = 256 * j + tid < n;
        key[j] = live ? min(max(key[j], 0), E) : -1;
        if (live) atomicAdd(&s.cnt[key[j]], 1);
    }
    __syncthreads();
    for (int e0 = 0, carry = 0; e0 <= E; e0 += 64) {            // (every wavefront writes the same for itself: no barrier)
        const int c = e0 + lane <= E ? s.cnt[e0 + lane] : 0, incl = wave_inclusive_sum(c);
        if (e0 + lane <= E) s.off[e0 + lane] = carry + incl - c;
        carry += __shfl(incl, 63);
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // f(assignment, its place among those of expert `target`)
    auto ranks = [&](int target, auto f) {
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            if (256 * j >= n) break;
            const uint64_t m = __ballot(key[j] == target);
            if (lane == 0) s.match[4 * j + wave] = __popcll(m);
        }
        __syncthreads();
        const int c = 64 * lane < n + 255 - (n + 255) % 256 ? s.match[lane] : 0, before = wave_inclusive_sum(c) - c;
#pragma unroll
        for (int j = 0; j < STEPS; ++j) {
            if (256 * j >= n) break;
            const bool hit = key[j] == target;
            const uint64_t m = __ballot(hit);
            const int r = __shfl(before, 4 * j + wave) + __popcll(m & ((1ull << lane) - 1));
            if (hit) f(256 * j + tid, r);
        }
        __syncthreads();
    };
    if (blockIdx.x == 0) {
        for (int i = tid; i <= E; i += 256) p.offsets_out[i] = s.off[i];
        const int active = s.off[E];
        if (active < n) ranks(E, [&](int a, int r) { p.perm_src_out[active + r] = a, p.inv_perm_out[a] = active + r; });
    }
    if (!find_item<UNIT>(s.off, E, n, BM, ncol, blockIdx.x, e_out, col, row0, rows)) return false;
    const int first = *row0 - s.off[*e_out];
    ranks(*e_out, [&](int a, int r) {
        if (r < first || r >= first + *rows) return;
        s.row[r - first] = a;
        if (*col == 0) p.perm_src_out[*row0 + r - first] = a, p.inv_perm_out[a] = *row0 + r - first;
    });
    return true;
}

// Row of `a` that row i of a block's tile is.
__device__ inline int source_row(const GemmArgs &p, const IndexScratch &s, int row0, int i)
{
    if (p.gate_idx) return s.row[i] >> (p.gate_k - 1);              // one or two experts per token
    return p.a_src ? p.a_src[row0 + i] / p.a_div : row0 + i;        // (a_src: gather fused into the loads)
}

}  // namespace moe
