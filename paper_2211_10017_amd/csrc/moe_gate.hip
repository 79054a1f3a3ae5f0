// moe_gate_topk: router logits, top-k selection and gate probabilities (Sec. 3.3).
//
// The logits of many tokens are a matrix product, and the fp32 matrix instructions of this chip round like a chain of fp32
// fused multiply-adds, so the contract's sequential partial sums (128-element blocks of the feature axis dealt round-robin to
// four sums) run on the matrix cores bit for bit: a wavefront owns one of the four partial sums for a tile of tokens and
// experts, the four meet in LDS, and sixteen lanes finish a token.  Two tilings: gate_mfma_kernel (16 tokens x 16 experts
// per instruction) and gate_quad_kernel (4 tokens x 64 experts); few tokens take the vector ALU with a lane per expert or several
// experts per lane (gate_token_kernel, gate_lanes_kernel and their other forms).  T = 8192, d = 4096, 64 experts: 196 -> 48 us (bf16 208 ->
// 47), T = 4096, d = 2048, 128 experts: 76 -> 28.6 us, T = 16384, d = 1024, 64 experts: 55 -> 32 us against multiply-adds in
// the vector ALU with a lane per expert or per token.
#include <math.h>

#include <type_traits>

#include "moe_ffn_common.h"

namespace moe {

constexpr int kGateBlk = 128;    // feature block of one partial-sum turn

template <bool BF16>
__device__ inline float act_to_float(uint16_t v)
{
    if (BF16) return __uint_as_float((uint32_t)v << 16);
    __half h;
    *reinterpret_cast<uint16_t *>(&h) = v;
    return __half2float(h);
}

// Value of the partner lane of butterfly step `off`: quad permutes for 1 and 2, the half-row and row mirrors for 4 and 8 (the same
// partner sets once the value is uniform over 4 resp. 8 lanes, which the earlier steps have made it), all in the VALU's
// data-parallel primitives, the steps across rows of sixteen lanes and halves of 32 the row and half swaps.  Used in ascending
// order of `off` by reductions whose operation is commutative.
template <int OFF, typename V>
__device__ inline V butterfly_partner(V v)
{
    const uint32_t b = __builtin_bit_cast(uint32_t, v);
    if constexpr (OFF >= 16) {      // (a swap leaves the lower rows' resp. half's values in [0] of both sides and the upper ones' in [1])
        const auto sw = OFF == 16 ? __builtin_amdgcn_permlane16_swap(b, b, false, false) : __builtin_amdgcn_permlane32_swap(b, b, false, false);
        return __builtin_bit_cast(V, (threadIdx.x & OFF) ? sw[0] : sw[1]);
    } else {
        constexpr int CTRL = OFF == 1 ? 0xB1 : OFF == 2 ? 0x4E : OFF == 4 ? 0x141 : 0x140;    // quad_perm [1,0,3,2], [2,3,0,1], row_half_mirror, row_mirror
        return __builtin_bit_cast(V, __builtin_amdgcn_update_dpp(0, (int)b, CTRL, 0xf, 0xf, false));
    }
}

// The outputs of one token: its k chosen experts (logits selv, descending) and their gate probabilities, den = the sum of
// exp(logit - largest logit) over all experts.
__device__ inline void store_choice(int t, int T, int E, int k, int renorm, const int (&sel)[2], const float (&selv)[2], float den,
                                    const uint8_t *__restrict__ finished, int32_t *__restrict__ expert_idx,
                                    float *__restrict__ expert_scale)
{
    if (finished && finished[t]) {
        // batch pruning (Sec. 3.5): the row gets an expert index past the real experts, so the
        // sort moves it behind every active row, and a zero scale
        for (int j = 0; j < k; ++j) {
            expert_idx[k * t + j] = E;
            expert_scale[k * t + j] = 0.0f;
        }
    } else if (k == 1) {
        expert_idx[t] = sel[0];
        expert_scale[t] = 1.0f / den;
    } else {
        const float e2 = expf(selv[1] - selv[0]);
        if (renorm) den = 1.0f + e2;
        const float s0 = 1.0f / den, s1 = e2 / den;
        expert_idx[2 * t] = sel[0];
        expert_idx[2 * t + 1] = sel[1];
        expert_scale[2 * t] = s0;
        expert_scale[2 * t + 1] = s1;
    }
}

// Logits, top-k, softmax and the stores of the NT tokens of a block (a multiple of 64 / LANES) from the four partial sums in LDS,
// part[p][token][ld].  LANES lanes finish a token, 64 / LANES tokens per wavefront at a time: lane (j, kk) of a wavefront holds
// the logits of NB neighbouring experts (of each of S slices of LANES NB experts) of token kk, so a reduction is a few
// comparisons in the lane and four data-parallel steps within the row of sixteen lanes (six with a wavefront per token, which
// blocks of few tokens and many experts take: a lane then has four logits instead of sixteen).
template <int S, int NB, int LANES = 16>
__device__ inline void finish_tokens(const float *part, int NT, int ld, int t0, int wave, int nwave,
                                     const float *__restrict__ bias, const uint8_t *__restrict__ finished, int T, int E,
                                     int k, int renorm, int32_t *__restrict__ expert_idx, float *__restrict__ expert_scale)
{
    constexpr int TPW = 64 / LANES;                     // tokens per wavefront at a time
    const int j = threadIdx.x % LANES, kk = threadIdx.x / LANES % TPW;
    for (int b0 = TPW * wave; b0 < NT; b0 += TPW * nwave) {
        const int b = b0 + kk, t = t0 + b;
        float lg[S][NB];
#pragma unroll
        for (int s = 0; s < S; ++s)
#pragma unroll
            for (int q = 0; q < NB; ++q) {
                const int e = (s * LANES + j) * NB + q;
                const float *src = part + (size_t)b * ld + e;
                float l = ((src[0] + src[(size_t)NT * ld]) + src[(size_t)2 * NT * ld]) + src[(size_t)3 * NT * ld];
                if (bias) l = l + bias[min(e, E - 1)];
                lg[s][q] = e < E ? l : -INFINITY;
            }
        auto steps = [](auto &&f) __attribute__((always_inline)) {
            f(std::integral_constant<int, 1>{});
            f(std::integral_constant<int, 2>{});
            f(std::integral_constant<int, 4>{});
            f(std::integral_constant<int, 8>{});
            if constexpr (LANES == 64) {
                f(std::integral_constant<int, 16>{});
                f(std::integral_constant<int, 32>{});
            }
        };
        // best (value, index) with ties to the lower index
        int sel[2] = {0, 0};
        float selv[2] = {0.0f, 0.0f};
        for (int r = 0; r < k; ++r) {
            float bv = -INFINITY;
            int be = 0x7fffffff;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int q = 0; q < NB; ++q) {
                    const int e = (s * LANES + j) * NB + q;
                    const bool taken = r == 1 && e == sel[0];
                    if (e < E && !taken && (lg[s][q] > bv || be == 0x7fffffff)) { bv = lg[s][q]; be = e; }
                }
            steps([&](auto off) {
                constexpr int OFF = decltype(off)::value;
                const float ov = butterfly_partner<OFF>(bv);
                const int oe = butterfly_partner<OFF>(be);
                if (oe != 0x7fffffff && (be == 0x7fffffff || ov > bv || (ov == bv && oe < be))) { bv = ov; be = oe; }
            });
            sel[r] = be;
            selv[r] = bv;
        }
        float den = 1.0f;
        if (k == 1 || !renorm) {                        // (two experts renormalised: their own two terms are all there is to it)
            const float lmax = selv[0];
            den = 0.0f;
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int q = 0; q < NB; ++q)
                    if ((s * LANES + j) * NB + q < E) den += expf(lg[s][q] - lmax);
            steps([&](auto off) { den += butterfly_partner<decltype(off)::value>(den); });
        }
        if (j == 0 && t < T) store_choice(t, T, E, k, renorm, sel, selv, den, finished, expert_idx, expert_scale);
    }
}

// f(integral_constant<I>) for I = 0 .. N-1
template <int I, int N, class F>
__device__ inline void gate_static_for(F &&f)
{
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        gate_static_for<I + 1, N>(f);
    }
}

// Eight 16-bit values per lane, (x0, x1, y0, y1) and (z0, z1, w0, w1): value i of the first four is paired with value i of the
// last four, and the 4 x 4 matrix of pairs over (row of sixteen lanes r, i) is transposed across the rows: q[s] of row r is then
// pair r of row s.
__device__ inline void transpose_quads(uint32_t x, uint32_t y, uint32_t z, uint32_t w, uint32_t (&q)[4])
{
    q[0] = __builtin_amdgcn_perm(z, x, 0x05040100u);
    q[1] = __builtin_amdgcn_perm(z, x, 0x07060302u);
    q[2] = __builtin_amdgcn_perm(w, y, 0x05040100u);
    q[3] = __builtin_amdgcn_perm(w, y, 0x07060302u);
    const auto a = __builtin_amdgcn_permlane16_swap(q[0], q[1], false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(q[2], q[3], false, false);
    const auto c = __builtin_amdgcn_permlane32_swap(a[0], b[0], false, false);
    const auto e = __builtin_amdgcn_permlane32_swap(a[1], b[1], false, false);
    q[0] = c[0]; q[1] = e[0]; q[2] = c[1]; q[3] = e[1];
}

// Loads of the gate weight, whose rows are E values of two bytes: WIDE, all experts of a lane at once (E a multiple of their
// number); PAIRS, two experts per 4-byte load (E even); ODD_PAIRS, the same for odd E, where every other row starts in the
// middle of a dword: its dwords are read from one value earlier, one more of them, and shifted into place in registers.
// (One 2-byte load per expert instead of pairs, d = 1024, caches warm: 4096 tokens, 129 / 250 / 255 experts 57 / 79 / 78 us against
// 37 / 42 / 51; experts in lanes, 16 tokens, 255 experts 22.7 against 13.5.)
enum GateLoads { WIDE, PAIRS, ODD_PAIRS };

// The logits on the matrix cores.  v_mfma_f32_16x16x4_f32 adds its four products to the accumulator one after
// the other, each with the rounding (and the subnormal numbers) of an fp32 fma, so a chain of them over ascending
// features IS the contract's sequential partial sum, bit for bit, at twice the rate of v_fma_mix_f32 (256 flops
// per clock and CU) and with far fewer operand reads: 16 tokens x 16 experts x 4 features per instruction.
// A wavefront owns 16 TT tokens x 16 NB experts of ONE partial sum; the block's first four wavefronts are the four
// partial sums (S slices of 128 experts each when E > 128).  Lane (j, kk) = (lane & 15, lane >> 4) supplies
// feature 4 n + kk of token j and of NB neighbouring experts j NB ..: these sit side by side in the row of the gate
// weight, so one load of 2 NB bytes feeds NB instructions, and nothing is staged through LDS.  A token's features
// come 64 bytes at a time, 16 per lane, and change lanes in registers.  R groups of 32 features are in flight per
// wavefront (a ring).  LOADS: how the gate weight's rows can be read, see GateLoads.
template <bool BF16, int NB, int S, int TT, int R, GateLoads LOADS>
__global__ __launch_bounds__(256 * S) void gate_mfma_kernel(const uint16_t *__restrict__ x,
                                                        const uint16_t *__restrict__ wg,
                                                        const float *__restrict__ bias,
                                                        const uint8_t *__restrict__ finished, int T, int d,
                                                        int E, int k, int renorm,
                                                        int32_t *__restrict__ expert_idx,
                                                        float *__restrict__ expert_scale)
{
    typedef float f4_t __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    constexpr int EP = 16 * NB;                         // experts of a slice
    constexpr int NT = 16 * TT;                         // tokens of the block
    extern __shared__ __align__(16) unsigned char smem[];
    float *part = reinterpret_cast<float *>(smem);      // [4][NT][ld]
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    constexpr int nwave = 4 * S, ld = S * EP + 4;
    const int p = wave & 3, slice = wave >> 2;
    const int j = lane & 15, kk = lane >> 4;
    const int t0 = blockIdx.x * NT;

    const int nblk = (d + kGateBlk - 1) / kGateBlk;
    // quads (four features) of this partial sum: its 128-feature blocks are p, p + 4, ...; only the last block of all may be short
    const int mine = p < nblk ? (nblk - p + 3) / 4 : 0;
    const int nquad = mine * 32 - (mine && (nblk - 1) % 4 == p ? (nblk * kGateBlk - d) / 4 : 0);

    // loads through buffer descriptors; every address is clamped into the row (what lies past the end is not used)
    const int rows = min(NT, T - t0);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x + (size_t)t0 * d), 0, rows * d * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wg), 0, d * E * 2, 0x00020000);
    int x_row[TT];
#pragma unroll
    for (int t = 0; t < TT; ++t) x_row[t] = min(16 * t + j, rows - 1) * d;
    const int e0 = slice * EP + j * NB;                 // this lane's experts e0 .. e0 + NB - 1 (clamped where they do not exist)
    const int odd = LOADS == ODD_PAIRS ? kk & 1 : 0;    // this lane's rows start in the middle of a dword
    const int w_off = (kk * E - odd + (LOADS == WIDE ? min(e0, E - NB) : 0)) * 2;

    constexpr int WD = NB >= 2 ? NB / 2 : 1;            // dwords of a lane's weights for one feature
    constexpr int WL = WD + (LOADS == ODD_PAIRS ? 1 : 0);
    struct Group { u32x4 x[TT]; uint32_t w[8][WL]; } ring[R];
    auto load = [&](Group &c, int g) __attribute__((always_inline)) {
        const int f = (p + 4 * (g >> 2)) * kGateBlk + (g & 3) * 32;
        const int fl = min(f + 8 * kk, d - 8);
#pragma unroll
        for (int t = 0; t < TT; ++t) c.x[t] = __builtin_amdgcn_raw_buffer_load_b128(rx, (x_row[t] + fl) * 2, 0, 0);
#pragma unroll
        for (int n = 0; n < 8; ++n) {
            const int so = min(f + 4 * n, d - 4) * E * 2;
            if constexpr (LOADS != WIDE) {      // (clamped: at most one value into the next row, and none past the last one)
#pragma unroll
                for (int u = 0; u < WL; ++u)
                    c.w[n][u] = __builtin_amdgcn_raw_buffer_load_b32(rw, w_off + 2 * min(e0 + 2 * u, LOADS == PAIRS ? E - 2 : E - 1), so, 0);
            } else if constexpr (NB == 1) {
                c.w[n][0] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rw, w_off, so, 0);
            } else if constexpr (NB == 2) {
                c.w[n][0] = __builtin_amdgcn_raw_buffer_load_b32(rw, w_off, so, 0);
            } else if constexpr (NB == 4) {
                const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rw, w_off, so, 0);
                c.w[n][0] = v.x; c.w[n][1] = v.y;
            } else {
                const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(rw, w_off, so, 0);
                c.w[n][0] = v.x; c.w[n][1] = v.y; c.w[n][2] = v.z; c.w[n][3] = v.w;
            }
        }
    };
    // A lane's 16 bytes hold features 8 kk .. 8 kk + 7 of the group; quad n wants feature 4 n + kk.  Halves i and
    // 4 + i are paired (i = 0 .. 3), and the 4 x 4 matrix of pairs over (kk, i) is transposed across the four rows of
    // sixteen lanes: dword s then holds features 8 s + kk and 8 s + 4 + kk, the operands of quads 2 s and 2 s + 1.
    auto spread = [&](u32x4 v, uint32_t (&q)[4]) __attribute__((always_inline)) { transpose_quads(v.x, v.y, v.z, v.w, q); };
    f4_t acc[TT][NB];
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int q = 0; q < NB; ++q) acc[t][q] = f4_t{0.f, 0.f, 0.f, 0.f};
    // All operands of a group are widened to fp32 in one go, then its 8 NB TT matrix instructions run back to back: fp32
    // matrix instructions share their pipe with the vector ALU, and every change between the two costs (one
    // conversion between any two of them: 44 clocks instead of 32 each).
    struct Ops { float x[8][TT], w[8][NB]; };
    auto widen = [&](const Group &c, Ops &o) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < TT; ++t) {
            uint32_t q[4];
            spread(c.x[t], q);
#pragma unroll
            for (int n = 0; n < 8; ++n) o.x[n][t] = act_to_float<BF16>((uint16_t)(q[n >> 1] >> (16 * (n & 1))));
        }
#pragma unroll
        for (int n = 0; n < 8; ++n)
#pragma unroll
            for (int u = 0; u < WD; ++u) {
                const uint32_t w = LOADS == ODD_PAIRS ? __builtin_amdgcn_alignbit(c.w[n][u + WL - WD], c.w[n][u], 16 * odd) : c.w[n][u];
#pragma unroll
                for (int b = 2 * u; b < NB && b < 2 * u + 2; ++b) o.w[n][b] = act_to_float<BF16>((uint16_t)(w >> (16 * (b & 1))));
            }
    };
    auto multiply = [&](const Ops &o, int n) __attribute__((always_inline)) {
#pragma unroll
        for (int q = 0; q < NB; ++q)
#pragma unroll
            for (int t = 0; t < TT; ++t) acc[t][q] = __builtin_amdgcn_mfma_f32_16x16x4f32(o.x[n][t], o.w[n][q], acc[t][q], 0, 0, 0);
    };
    gate_static_for<0, R>([&](auto o) {
        load(ring[decltype(o)::value], decltype(o)::value);
        __builtin_amdgcn_sched_barrier(0);              // the loads stay in the loop's order: the wait counts of the first trip fit all of them
    });
    const int ng = (nquad + 7) / 8;
    int g0 = 0;
    for (; (g0 + R) * 8 <= nquad; g0 += R) {
        gate_static_for<0, R>([&](auto gc) {
            constexpr int g = decltype(gc)::value;
            Ops o;
            widen(ring[g], o);
            __builtin_amdgcn_sched_barrier(0);
            load(ring[g], g0 + g + R);                  // (past the end: in-bounds loads that are not used)
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int n = 0; n < 8; ++n) multiply(o, n);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    gate_static_for<0, R>([&](auto gc) {                // fewer than 8 R quads are left, all of them in the ring
        constexpr int g = decltype(gc)::value;
        if (g0 + g < ng) {
            Ops o;
            widen(ring[g], o);
#pragma unroll
            for (int n = 0; n < 8; ++n)
                if ((g0 + g) * 8 + n < nquad) multiply(o, n);
        }
    });
    // acc[t][q][i]: token 16 t + 4 kk + i, expert slice EP + j NB + q
#pragma unroll
    for (int t = 0; t < TT; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float *dst = part + ((size_t)p * NT + 16 * t + 4 * kk + i) * ld + slice * EP + j * NB;
#pragma unroll
            for (int q = 0; q < NB; ++q) dst[q] = acc[t][q][i];
        }
    __syncthreads();

    finish_tokens<S, NB>(part, NT, ld, t0, wave, nwave, bias, finished, T, E, k, renorm, expert_idx, expert_scale);
}

// Few tokens and 33 to 64 experts: the same chains in v_mfma_f32_4x4x1_16b_f32, sixteen 4 x 4 x 1 products that make up
// 4 tokens x 64 experts x 1 feature.  A block takes four tokens instead of sixteen, so the batch spreads over four times
// as many compute units at the same rate of the matrix pipe.  An octet of features is one 16-byte load of the tokens and two
// 8-byte loads of the gate weight: lane (j, r) = (lane & 15, lane >> 4) brings experts 4 j .. 4 j + 3 of features r and 4 + r, and
// the same 4 x 4 transposition that spreads the tokens' features above leaves it with expert 4 j + r of all eight.  (VEC; numbers
// of experts that are no multiple of four: a lane per expert, one 2-byte load per feature.)  A ring of R octets.
template <bool BF16, int R, bool VEC>
__global__ __launch_bounds__(256) void gate_quad_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wg,
                                                            const float *__restrict__ bias,
                                                            const uint8_t *__restrict__ finished, int T, int d, int E,
                                                            int k, int renorm, int32_t *__restrict__ expert_idx,
                                                            float *__restrict__ expert_scale)
{
    typedef float f4_t __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    constexpr int NT = 4, ld = 64 + 4;
    __shared__ float part[4 * NT * ld];
    const int lane = threadIdx.x & 63;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int own = VEC ? 4 * (lane & 15) + (lane >> 4) : lane;      // this lane's expert
    const int t0 = blockIdx.x * NT;
    const int nblk = (d + kGateBlk - 1) / kGateBlk;
    const int mine = p < nblk ? (nblk - p + 3) / 4 : 0;
    const int nq = mine * 16 - (mine && (nblk - 1) % 4 == p ? (nblk * kGateBlk - d) / 8 : 0);     // octets of this partial sum
    auto feature = [&](int q) { return min((p + 4 * (q >> 4)) * kGateBlk + (q & 15) * 8, d - 8); };   // clamped into the row
    const int rows = min(NT, T - t0);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x + (size_t)t0 * d), 0, rows * d * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wg), 0, d * E * 2, 0x00020000);
    const int x_off = min(lane & 3, rows - 1) * d * 2;
    const int w_off = VEC ? ((lane >> 4) * E + min(4 * (lane & 15), E - 4)) * 2 : min(own, E - 1) * 2;   // (experts clamped where they do not exist)

    struct Octet { u32x4 x; uint32_t w[VEC ? 4 : 8]; } ring[R];
    auto load = [&](Octet &c, int q) __attribute__((always_inline)) {
        const int f = feature(q);
        c.x = __builtin_amdgcn_raw_buffer_load_b128(rx, x_off, f * 2, 0);
        if constexpr (VEC) {
            const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(rw, w_off, f * E * 2, 0), b = __builtin_amdgcn_raw_buffer_load_b64(rw, w_off, (f + 4) * E * 2, 0);
            c.w[0] = a.x; c.w[1] = a.y; c.w[2] = b.x; c.w[3] = b.y;
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) c.w[u] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rw, w_off, (f + u) * E * 2, 0);
        }
    };
    f4_t acc = {0.f, 0.f, 0.f, 0.f};
    struct Ops { float x[8], w[8]; };
    auto widen = [&](const Octet &c, Ops &o) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const uint32_t v = u < 2 ? c.x.x : u < 4 ? c.x.y : u < 6 ? c.x.z : c.x.w;
            o.x[u] = act_to_float<BF16>((uint16_t)(v >> (16 * (u & 1))));
        }
        if constexpr (VEC) {
            uint32_t q[4];
            transpose_quads(c.w[0], c.w[1], c.w[2], c.w[3], q);     // dword u: features u and 4 + u of expert `own`
#pragma unroll
            for (int u = 0; u < 8; ++u) o.w[u] = act_to_float<BF16>((uint16_t)(q[u & 3] >> (16 * (u >> 2))));
        } else {
#pragma unroll
            for (int u = 0; u < 8; ++u) o.w[u] = act_to_float<BF16>((uint16_t)c.w[u]);
        }
    };
    auto multiply = [&](const Ops &o) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u) acc = __builtin_amdgcn_mfma_f32_4x4x1f32(o.x[u], o.w[u], acc, 0, 0, 0);
    };
    gate_static_for<0, R>([&](auto o) {
        load(ring[decltype(o)::value], decltype(o)::value);
        __builtin_amdgcn_sched_barrier(0);              // the loads stay in the loop's order
    });
    int q0 = 0;
    for (; q0 + R <= nq; q0 += R) {
        gate_static_for<0, R / 2>([&](auto oc) {        // two octets at a time: conversions and matrix instructions in longer runs
            constexpr int o = 2 * decltype(oc)::value;
            Ops a, b;
            widen(ring[o], a);
            widen(ring[o + 1], b);
            __builtin_amdgcn_sched_barrier(0);
            load(ring[o], q0 + o + R);                  // (past the end: in-bounds loads that are not used)
            load(ring[o + 1], q0 + o + 1 + R);
            __builtin_amdgcn_sched_barrier(0);
            multiply(a);
            multiply(b);
            __builtin_amdgcn_sched_barrier(0);
        });
    }
    gate_static_for<0, R - 1>([&](auto oc) {
        constexpr int o = decltype(oc)::value;
        if (q0 + o < nq) {
            Ops a;
            widen(ring[o], a);
            multiply(a);
        }
    });
#pragma unroll
    for (int i = 0; i < NT; ++i) part[(p * NT + i) * ld + own] = acc[i];
    __syncthreads();
    finish_tokens<1, 4>(part, NT, ld, t0, p, 4, bias, finished, T, E, k, renorm, expert_idx, expert_scale);
}

// Few tokens and more than 32 experts: NE experts per lane and the partial sums as plain fp32 fused multiply-adds.  Up to a few
// tokens per compute unit the matrix instructions above work on rows and experts of one block alone, sixteen or four tokens by all
// experts, and a compute unit's matrix pipe is the bound; here a block takes TB tokens, each feature costs a wavefront
// NE TB fused multiply-adds and one load of a row of the gate weight per VW experts of a lane, and R octets of features are in flight.
// (Caches warm, 16 / 512 tokens, d = 1024: 127 experts 9.5 / 12.5 us, 256 12.2 / 14.2, 255 13.5 / 18.1; on the matrix
// cores 14.8 to 16 us with 64 to 512 tokens and 65 to 128 experts, 25 with 256, 51 with 255.)
template <bool BF16, int NE, GateLoads LOADS, int TB, int R>
__global__ __launch_bounds__(256) void gate_lanes_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wg,
                                                         const float *__restrict__ bias,
                                                         const uint8_t *__restrict__ finished, int T, int d, int E,
                                                         int k, int renorm, int32_t *__restrict__ expert_idx,
                                                         float *__restrict__ expert_scale)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    constexpr bool ODD = LOADS == ODD_PAIRS;
    constexpr int VW = LOADS == WIDE ? NE : 2, NL = NE / VW;           // experts per load, loads per feature
    constexpr int NT = NE <= 2 && TB < 4 ? 4 : TB, ld = 64 * NE + 4;   // (sixteen lanes per token: four tokens at a time, the ones past TB are not stored)
    __shared__ float part[4 * NT * ld];
    const int lane = threadIdx.x & 63;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int t0 = blockIdx.x * TB;
    const int nblk = (d + kGateBlk - 1) / kGateBlk;
    const int mine = p < nblk ? (nblk - p + 3) / 4 : 0;
    const int nq = mine * 16 - (mine && (nblk - 1) % 4 == p ? (nblk * kGateBlk - d) / 8 : 0);     // octets of this partial sum
    auto feature = [&](int q) { return min((p + 4 * (q >> 4)) * kGateBlk + (q & 15) * 8, d - 8); };   // clamped into the row
    const int rows = min(TB, T - t0);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x + (size_t)t0 * d), 0, rows * d * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wg), 0, d * E * 2, 0x00020000);
    int w_off[NL];                                      // experts VW (64 s + lane) .. (clamped where they do not exist; odd E: at most one value into the next row)
#pragma unroll
    for (int s = 0; s < NL; ++s) w_off[s] = min(VW * (64 * s + lane), ODD ? E - 1 : E - VW) * 2;

    struct Octet { u32x4 x[TB]; uint32_t w[8][NL][VW < 2 ? 1 : VW / 2]; } ring[R];
    auto load = [&](Octet &c, int q) __attribute__((always_inline)) {
        const int f = feature(q);
#pragma unroll
        for (int b = 0; b < TB; ++b) c.x[b] = __builtin_amdgcn_raw_buffer_load_b128(rx, min(b, rows - 1) * d * 2, f * 2, 0);
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int s = 0; s < NL; ++s) {
                const int so = ((f + u) * E - (ODD ? u & 1 : 0)) * 2;
                if constexpr (VW == 1) c.w[u][s][0] = (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(rw, w_off[s], so, 0);
                else if constexpr (VW == 2) c.w[u][s][0] = __builtin_amdgcn_raw_buffer_load_b32(rw, w_off[s], so, 0);
                else {
                    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(rw, w_off[s], so, 0);
                    c.w[u][s][0] = v.x; c.w[u][s][1] = v.y;
                }
            }
    };
    float acc[TB][NE];
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int e = 0; e < NE; ++e) acc[b][e] = 0.0f;
    auto multiply = [&](const Octet &c) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 8; ++u)
#pragma unroll
            for (int b = 0; b < TB; ++b) {
                const float xf = act_to_float<BF16>((uint16_t)(c.x[b][u >> 1] >> (16 * (u & 1))));
#pragma unroll
                for (int e = 0; e < NE; ++e)
                    acc[b][e] = fmaf(xf, act_to_float<BF16>((uint16_t)(c.w[u][e / VW][(e % VW) >> 1] >> (16 * (e % VW & 1)))), acc[b][e]);
            }
    };
    // odd E: a lane's dword of an odd feature holds the value before its first expert and that expert; the other one is the lower half
    // of the next lane's dword (of lane 0's of the next slice in the last lane)
    auto shift = [&](Octet &c) __attribute__((always_inline)) {
        if constexpr (ODD) {
#pragma unroll
            for (int u = 1; u < 8; u += 2) {
                uint32_t up[NL];
#pragma unroll
                for (int s = 0; s < NL; ++s) up[s] = __builtin_amdgcn_update_dpp(0, (int)c.w[u][s][0], 0x134, 0xf, 0xf, false);   // wave_rol:1
#pragma unroll
                for (int s = 0; s < NL; ++s)
                    c.w[u][s][0] = __builtin_amdgcn_alignbit(s + 1 < NL && lane == 63 ? up[s + 1 < NL ? s + 1 : s] : up[s], c.w[u][s][0], 16);
            }
        }
    };
    gate_static_for<0, R>([&](auto o) { load(ring[decltype(o)::value], decltype(o)::value); });
    int q0 = 0;
    for (; q0 + R <= nq; q0 += R) {
        gate_static_for<0, R>([&](auto oc) {
            constexpr int o = decltype(oc)::value;
            Octet c = ring[o];
            load(ring[o], q0 + o + R);                  // (past the end: in-bounds loads that are not used)
            shift(c);
            multiply(c);
        });
    }
    gate_static_for<0, R - 1>([&](auto oc) {
        constexpr int o = decltype(oc)::value;
        if (q0 + o < nq) {
            shift(ring[o]);
            multiply(ring[o]);
        }
    });
#pragma unroll
    for (int b = 0; b < TB; ++b)
#pragma unroll
        for (int e = 0; e < NE; ++e) part[(p * NT + b) * ld + VW * (64 * (e / VW) + lane) + e % VW] = acc[b][e];
    __syncthreads();
    finish_tokens<NE == 2 ? 2 : 1, 4, NE <= 2 ? 16 : 64>(part, NT, ld, t0, p, 4, bias, finished, min(T, t0 + TB), E, k, renorm, expert_idx, expert_scale);
}

// The last, short block of features of one partial sum, for the chains below: its rows of the gate weight, as they lie, go into LDS while the chain before it runs.  (Fetched
// at its end, an octet at a time, each octet was a trip to memory: us, then / now, 75 tokens of 112, 32 experts 5.1 / 4.1, 64 of 1000, 16 experts 5.8 / 4.7, 184 of 6248, 8 experts 17.1 /
// 14.1, 64 bf16 tokens of 1016, 128 experts 12.3 / 10.3.)
constexpr int gate_tail_bytes(int EP, int d) { return d % kGateBlk ? EP * 256 : 0; }

__device__ __forceinline__ void gate_tail_load(const uint16_t *block, int bytes, unsigned char *lds)
{
    for (int i = 0; i < bytes; i += 1024)
        load_to_lds16(reinterpret_cast<const unsigned char *>(block) + min((int)(threadIdx.x & 63) * 16 + i, bytes - 16), reinterpret_cast<uint16_t *>(lds + i));
}

__device__ __forceinline__ void gate_tail_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Few tokens, E a multiple of four up to 32: a lane per expert, SUB tokens side by side, TW of them per lane, plain fp32 multiply-adds, the gate weight through
// LDS as it lies in memory: each wavefront copies its own partial sum's rows 64 features at a time (two chunks in LDS, two more on the way), and the transposing
// read gives a lane four features of its expert.  What bounds it are instructions, of which a wavefront alone on its SIMD issues one in 4.4 clocks: an octet of features
// takes eight multiply-adds, a wait state after each whose sum the next one adds to, two reads of weights, one of the token.  (115 clocks an octet.  With FP16 tokens as
// fp32 in LDS, which spares wait states, the reads bound: d = 4096, 16 experts 8.6 -> 10.6 us.  Transposing in registers as below: 10.1.  For 64 experts writes and reads
// of LDS meet the other three wavefronts': 10.9 against 10.1.)  A wavefront waits for nobody before the end.
template <bool BF16, int EP, int TW>
__device__ __forceinline__ void gate_rows(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wg, const float *__restrict__ bias,
                                          const uint8_t *__restrict__ finished, int T, int d, int E, int k, int renorm,
                                          int32_t *__restrict__ expert_idx, float *__restrict__ expert_scale)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    constexpr int SUB = 64 / EP, NT = TW * SUB;
    constexpr int ld = EP + 4, NTP = NT < 4 ? 4 : NT;   // (four tokens finish at a time, those past NT are not stored)
    constexpr int XV = BF16 ? 2 : 1;                    // 16-byte words of an octet of a token
    constexpr int XP = 2;                               // passes of 64 octets of the tokens that are requested ahead of the weights
    constexpr int CW = EP * 8, LD = EP / 8;             // 16-byte words of a chunk (64 features), loads of it per lane
    static_assert(LD <= 6, "a chunk is written before its first octet is read");
    extern __shared__ __align__(16) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    u32x4 *s_w = reinterpret_cast<u32x4 *>(smem) + (size_t)p * 2 * CW;                   // two chunks of this wavefront's
    float *part = reinterpret_cast<float *>(smem + 8 * CW * 16);                         // [4][NTP][ld]
    const int e = lane % EP, sub = lane / EP;           // this lane's expert and token
    const int t0 = blockIdx.x * NT, rows = min(NT, T - t0);
    const int nblk = (d + kGateBlk - 1) / kGateBlk;
    const int full = max((d / kGateBlk - p + 3) / 4, 0);                                // whole 128-feature blocks of this partial sum
    const int rest = (nblk - 1) % 4 == p ? (d % kGateBlk) / 8 : 0, nq = full * 16 + rest;      // octets of the last, short one, and in all
    const int x_words = ((nblk + 3) / 4 * 16 + 2) * NT * XV;                             // (two octets are read past the end)
    u32x4 *s_x = reinterpret_cast<u32x4 *>(smem + 8 * CW * 16 + 4 * NTP * ld * 4) + (size_t)p * x_words;      // [octet][token]
    unsigned char *s_tail = smem + 8 * CW * 16 + 4 * NTP * ld * 4 + (size_t)4 * x_words * 16;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x + (size_t)t0 * d), 0, rows * d * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wg), 0, d * E * 2, 0x00020000);
    int w_off[LD];                                      // (within the chunk: fewer experts than EP read its end again)
#pragma unroll
    for (int i = 0; i < LD; ++i) w_off[i] = min(lane * 16 + i * 1024, 128 * E - 16);

    const int row = E * 2;                              // bytes
    auto x_load = [&](int q, int b) __attribute__((always_inline)) {
        return __builtin_amdgcn_raw_buffer_load_b128(rx, (min(b, rows - 1) * d + min((p + 4 * (q >> 4)) * kGateBlk + (q & 15) * 8, d - 8)) * 2, 0, 0);
    };
    auto x_store = [&](int q, int b, u32x4 v) __attribute__((always_inline)) {
        if (q >= nq) return;
        if constexpr (BF16) {
            s_x[(q * NT + b) * 2] = u32x4{v.x << 16, v.x & 0xffff0000u, v.y << 16, v.y & 0xffff0000u};
            s_x[(q * NT + b) * 2 + 1] = u32x4{v.z << 16, v.z & 0xffff0000u, v.w << 16, v.w & 0xffff0000u};
        } else {
            s_x[q * NT + b] = v;
        }
    };
    float acc[TW];
#pragma unroll
    for (int w = 0; w < TW; ++w) acc[w] = 0.0f;
    struct Octet { u32x4 x[TW][XV]; s16x4 w[2]; };
    // sixteen lanes point at four rows of sixteen experts, four experts each; back comes an expert's four rows
    const int w_read = (((lane & 15) >> 2) * E + (e & 16) + 4 * (lane & 3)) * 2;
    auto x_read = [&](Octet &t, int q) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < TW; ++w)
#pragma unroll
            for (int h = 0; h < XV; ++h) t.x[w][h] = s_x[(q * NT + w * SUB + sub) * XV + h];
    };
    auto w_get = [&](Octet &t, const void *rows_of, int o) __attribute__((always_inline)) {
        typedef __attribute__((address_space(3))) s16x4 *lds_t;
        unsigned char *at = (unsigned char *)rows_of + w_read + o * 8 * row;
#pragma unroll
        for (int h = 0; h < 2; ++h) t.w[h] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_t)(at + h * 4 * row));
    };
    auto feature = [&](const Octet &t, auto uc) __attribute__((always_inline)) {
        constexpr int u = decltype(uc)::value;
#pragma unroll
        for (int w = 0; w < TW; ++w) {
            const float xf = BF16 ? __uint_as_float(t.x[w][XV == 2 ? u >> 2 : 0][u & 3]) : act_to_float<false>((uint16_t)(t.x[w][0][u >> 1] >> (16 * (u & 1))));
            acc[w] = fmaf(xf, act_to_float<BF16>((uint16_t)t.w[u >> 2][u & 3]), acc[w]);
        }
    };
    u32x4 xv[XP][NT];
#pragma unroll
    for (int i = 0; i < XP; ++i)
#pragma unroll
        for (int b = 0; b < NT; ++b) xv[i][b] = x_load(lane + 64 * i, b);
    __builtin_amdgcn_sched_barrier(0);
    auto base = [&](int c) { c = min(c, 2 * full - 1); return ((p + 4 * (c >> 1)) * kGateBlk + (c & 1) * 64) * row; };      // (past the end: the last one again, not used)
    u32x4 W[2][LD];
    auto load = [&](int i, int so) __attribute__((always_inline)) { return __builtin_amdgcn_raw_buffer_load_b128(rw, w_off[i], so, 0); };
    if (full)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int i = 0; i < LD; ++i) W[h][i] = load(i, base(h));
    __builtin_amdgcn_sched_barrier(0);
    if (rest) gate_tail_load(wg + (size_t)(p + 4 * full) * kGateBlk * E, rest * 8 * row, s_tail);
#pragma unroll
    for (int i = 0; i < XP; ++i)
#pragma unroll
        for (int b = 0; b < NT; ++b) x_store(lane + 64 * i, b, xv[i][b]);
    for (int q = lane + 64 * XP; q < nq; q += 64)
#pragma unroll
        for (int b = 0; b < NT; ++b) x_store(q, b, x_load(q, b));
    auto fence = [] {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    };
    if (full) {
#pragma unroll
        for (int i = 0; i < LD; ++i) s_w[i * 64 + lane] = W[0][i];
        const int so = base(2);
#pragma unroll
        for (int i = 0; i < LD; ++i) W[0][i] = load(i, so);
        fence();
        Octet t[4];
        x_read(t[0], 0); w_get(t[0], s_w, 0);
        x_read(t[1], 1); w_get(t[1], s_w, 1);
        for (int b = 0; b < full; ++b) {
            gate_static_for<0, 16>([&](auto oc) {
                // octet oo of chunk h of the block; with its first ones go the writes of the next chunk and the loads of the one two further on
                constexpr int o = decltype(oc)::value, h = o >> 3, oo = o & 7;
                const int so = base(2 * b + h + 3);
                gate_static_for<0, 8>([&](auto u) {
                    constexpr int i = decltype(u)::value;
                    feature(t[o & 3], u);
                    if constexpr (i == 0) x_read(t[(o + 2) & 3], b * 16 + o + 2);
                    if constexpr (i == 1) w_get(t[(o + 2) & 3], s_w + (((o + 2) >> 3) & 1) * CW, (o + 2) & 7);      // (from the sixth octet on in the next chunk: all of it is there)
                    if constexpr (i == 2 && oo < LD) {
                        s_w[(1 - h) * CW + oo * 64 + lane] = W[1 - h][oo];
                        W[1 - h][oo] = load(oo, so);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
                if constexpr (oo == 5) fence();
            });
        }
    }
    if (rest) {
        gate_tail_wait();
        fence();
        Octet t;
        x_read(t, full * 16); w_get(t, s_tail, 0);
#pragma unroll 1
        for (int o = 0; o < rest; ++o) {
            Octet next;
            x_read(next, full * 16 + o + 1); w_get(next, s_tail, o + 1);
            gate_static_for<0, 8>([&](auto u) { feature(t, u); });
            t = next;
        }
    }
#pragma unroll
    for (int w = 0; w < TW; ++w) part[(p * NTP + w * SUB + sub) * ld + e] = acc[w];
    __syncthreads();
    finish_tokens<1, EP / 16>(part, NTP, ld, t0, p, 4, bias, finished, min(T, t0 + NT), E, k, renorm, expert_idx, expert_scale);
}

// Few tokens and 36 to 128 experts, a multiple of four: the same with a lane per expert (two with more than 64) and the gate weight
// from memory straight into registers.  A lane (j, r) brings experts 4 j .. 4 j + 3 of features r and 4 + r in two 8-byte loads, and the 4 x 4
// transposition that spreads the tokens' features above leaves it with expert 4 j + r of an octet of features.  Its eight instructions for the next octet
// are dealt out one by one between the multiply-adds, where each stands in for a wait state, and so are the loads and the reads of the tokens (in the order
// spread, additions, loads 3 % slower).  130 clocks an octet, the swaps issuing at half rate.  Eight octets in flight: with 4, warm launches are 0.2 us shorter and
// layers' steps, whose gate weight comes from memory, 0.3 % longer; with 16, 1.8 % longer.
template <bool BF16, int EP, int TW>
__device__ __forceinline__ void gate_chains(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wg, const float *__restrict__ bias,
                                            const uint8_t *__restrict__ finished, int T, int d, int E, int k, int renorm,
                                            int32_t *__restrict__ expert_idx, float *__restrict__ expert_scale)
{
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
    constexpr int EW = EP / 64, NT = TW, R = 8;
    constexpr int ld = EP + 4, NTP = NT < 4 ? 4 : NT;   // (four tokens finish at a time, those past NT are not stored)
    constexpr int XV = BF16 ? 2 : 1;                    // 16-byte words of an octet of a token
    constexpr int XP = 2;                               // passes of 64 octets of the tokens that are requested ahead of the weights
    extern __shared__ __align__(16) unsigned char smem[];
    float *part = reinterpret_cast<float *>(smem);      // [4][NTP][ld]
    const int lane = threadIdx.x & 63;
    const int p = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int j = lane & 15, r = lane >> 4;
    const int t0 = blockIdx.x * NT, rows = min(NT, T - t0);
    const int nblk = (d + kGateBlk - 1) / kGateBlk;
    const int full = max((d / kGateBlk - p + 3) / 4, 0);                                // whole 128-feature blocks of this partial sum
    const int rest = (nblk - 1) % 4 == p ? (d % kGateBlk) / 8 : 0, nq = full * 16 + rest;      // octets of the last, short one, and in all
    const int x_words = ((nblk + 3) / 4 * 16 + 2) * NT * XV;                             // (two octets are read past the end)
    u32x4 *s_x = reinterpret_cast<u32x4 *>(smem + 4 * NTP * ld * 4) + (size_t)p * x_words;      // [octet][token]
    unsigned char *s_tail = smem + 4 * NTP * ld * 4 + (size_t)4 * x_words * 16;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x + (size_t)t0 * d), 0, rows * d * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(wg), 0, d * E * 2, 0x00020000);
    int w_off[EW][2];                                   // features r, 4 + r
#pragma unroll
    for (int s = 0; s < EW; ++s) {
        w_off[s][0] = (r * E + min(64 * s + 4 * j, E - 4)) * 2;         // (experts clamped where they do not exist)
        w_off[s][1] = w_off[s][0] + 8 * E;
    }

    auto x_load = [&](int q, int b) __attribute__((always_inline)) {
        return __builtin_amdgcn_raw_buffer_load_b128(rx, (min(b, rows - 1) * d + min((p + 4 * (q >> 4)) * kGateBlk + (q & 15) * 8, d - 8)) * 2, 0, 0);
    };
    auto x_store = [&](int q, int b, u32x4 v) __attribute__((always_inline)) {
        if (q >= nq) return;
        if constexpr (BF16) {
            s_x[(q * NT + b) * 2] = u32x4{v.x << 16, v.x & 0xffff0000u, v.y << 16, v.y & 0xffff0000u};
            s_x[(q * NT + b) * 2 + 1] = u32x4{v.z << 16, v.z & 0xffff0000u, v.w << 16, v.w & 0xffff0000u};
        } else {
            s_x[q * NT + b] = v;
        }
    };
    struct Raw { uint32_t w[EW][4]; } ring[R];
    auto load = [&](Raw &c, int so) __attribute__((always_inline)) {        // so: bytes of the octet's first row
#pragma unroll
        for (int s = 0; s < EW; ++s) {
            const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(rw, w_off[s][0], so, 0), b = __builtin_amdgcn_raw_buffer_load_b64(rw, w_off[s][1], so, 0);
            c.w[s][0] = a.x; c.w[s][1] = a.y; c.w[s][2] = b.x; c.w[s][3] = b.y;
        }
    };
    // one of the eight instructions that spread an octet (transpose_quads)
    struct Spread { uint32_t q[EW][4]; };
    auto spread = [&](const Raw &c, Spread &v, auto ic) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
#pragma unroll
        for (int s = 0; s < EW; ++s) {
            uint32_t(&q)[4] = v.q[s];
            if constexpr (i < 4) {
                q[i] = __builtin_amdgcn_perm(c.w[s][2 + (i >> 1)], c.w[s][i >> 1], i & 1 ? 0x07060302u : 0x05040100u);
            } else if constexpr (i < 6) {
                const auto a = __builtin_amdgcn_permlane16_swap(q[2 * i - 8], q[2 * i - 7], false, false);
                q[2 * i - 8] = a[0]; q[2 * i - 7] = a[1];
            } else {
                const auto a = __builtin_amdgcn_permlane32_swap(q[i - 6], q[i - 4], false, false);
                q[i - 6] = a[0]; q[i - 4] = a[1];
            }
        }
    };
    // after the swaps: dword 0, 1, 2, 3 holds features (0, 4), (1, 5), (2, 6), (3, 7)
    float acc[TW][EW];
#pragma unroll
    for (int w = 0; w < TW; ++w)
#pragma unroll
        for (int s = 0; s < EW; ++s) acc[w][s] = 0.0f;
    struct Tok { u32x4 v[TW][XV]; };
    auto x_read = [&](Tok &t, int q) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < TW; ++w)
#pragma unroll
            for (int h = 0; h < XV; ++h) t.v[w][h] = s_x[(q * NT + w) * XV + h];
    };
    auto feature = [&](const Tok &t, const Spread &v, auto uc) __attribute__((always_inline)) {
        constexpr int u = decltype(uc)::value;
#pragma unroll
        for (int w = 0; w < TW; ++w) {
            const float xf = BF16 ? __uint_as_float(t.v[w][XV == 2 ? u >> 2 : 0][u & 3]) : act_to_float<false>((uint16_t)(t.v[w][0][u >> 1] >> (16 * (u & 1))));
#pragma unroll
            for (int s = 0; s < EW; ++s) acc[w][s] = fmaf(xf, act_to_float<BF16>((uint16_t)(v.q[s][u & 3] >> (16 * (u >> 2)))), acc[w][s]);
        }
    };
    u32x4 xv[XP][NT];
#pragma unroll
    for (int i = 0; i < XP; ++i)
#pragma unroll
        for (int b = 0; b < NT; ++b) xv[i][b] = x_load(lane + 64 * i, b);
    __builtin_amdgcn_sched_barrier(0);
    const int step = 16 * E, turn = 4 * kGateBlk * E * 2, first = p * kGateBlk * E * 2;   // bytes of an octet of rows, between this partial sum's blocks, before the first of them
    if (full)
        gate_static_for<0, R>([&](auto o) {
            load(ring[decltype(o)::value], first + decltype(o)::value * step);
            __builtin_amdgcn_sched_barrier(0);
        });
    if (rest) gate_tail_load(wg + (size_t)(p + 4 * full) * kGateBlk * E, rest * step, s_tail);
#pragma unroll
    for (int i = 0; i < XP; ++i)
#pragma unroll
        for (int b = 0; b < NT; ++b) x_store(lane + 64 * i, b, xv[i][b]);
    for (int q = lane + 64 * XP; q < nq; q += 64)
#pragma unroll
        for (int b = 0; b < NT; ++b) x_store(q, b, x_load(q, b));
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");

    if (full) {
        Tok tok[4];
        Spread sp[2];
        x_read(tok[0], 0);
        x_read(tok[1], 1);
        gate_static_for<0, 8>([&](auto i) { spread(ring[0], sp[0], i); });
        int ahead = first + R * step;       // the octet R past the one at hand
        load(ring[0], ahead);
        for (int b = 0; b < full; ++b) {
            gate_static_for<0, 16>([&](auto oc) {
                constexpr int o = decltype(oc)::value;
                auto spr = [&](auto i) __attribute__((always_inline)) { spread(ring[(o + 1) % R], sp[(o + 1) & 1], i); };
                gate_static_for<0, 8>([&](auto u) {
                    constexpr int i = decltype(u)::value;
                    feature(tok[o & 3], sp[o & 1], u);
                    if constexpr (i == 0) {
                        spr(std::integral_constant<int, 0>{});
                        spr(std::integral_constant<int, 1>{});
                    } else if constexpr (i == 1) {
                        spr(std::integral_constant<int, 2>{});
                        x_read(tok[(o + 2) & 3], b * 16 + o + 2);
                    } else if constexpr (i == 5) {      // the octet o + 1 + R: in this block or the next (the last block again where there is none)
                        constexpr int n = o + 1 + R;
                        if constexpr (n % 16 == 0) ahead = first + min(b + n / 16, full - 1) * turn;
                        else ahead += step;
                        load(ring[(o + 1) % R], ahead);
                    } else {
                        spr(std::integral_constant<int, i == 2 ? 3 : i < 5 ? i + 1 : i>{});
                    }
                    __builtin_amdgcn_sched_barrier(0);
                });
            });
        }
    }
    if (rest) {
        auto from_lds = [&](Raw &c, int o) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 0; s < EW; ++s)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const u32x2 v = *reinterpret_cast<const u32x2 *>(s_tail + w_off[s][h] + o * step);
                    c.w[s][2 * h] = v.x; c.w[s][2 * h + 1] = v.y;
                }
        };
        gate_tail_wait();
        Raw c;
        from_lds(c, 0);
#pragma unroll 1
        for (int o = 0; o < rest; ++o) {
            Raw next;
            Spread v;
            Tok t;
            x_read(t, full * 16 + o);
            from_lds(next, o + 1);
            gate_static_for<0, 8>([&](auto i) { spread(c, v, i); });
            gate_static_for<0, 8>([&](auto u) { feature(t, v, u); });
            c = next;
        }
    }
#pragma unroll
    for (int w = 0; w < TW; ++w)
#pragma unroll
        for (int s = 0; s < EW; ++s) part[(p * NTP + w) * ld + 64 * s + 4 * j + r] = acc[w][s];
    __syncthreads();
    finish_tokens<EW, 4>(part, NTP, ld, t0, p, 4, bias, finished, min(T, t0 + NT), E, k, renorm, expert_idx, expert_scale);
}

template <bool BF16, int EP, int TW>      // up to 64 experts
__global__ __launch_bounds__(256) void gate_token_kernel(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wg, const float *__restrict__ bias,
                                                         const uint8_t *__restrict__ finished, int T, int d, int E, int k, int renorm,
                                                         int32_t *__restrict__ expert_idx, float *__restrict__ expert_scale)
{
    if constexpr (EP <= 32) gate_rows<BF16, EP, TW>(x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale);
    else gate_chains<BF16, EP, TW>(x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale);
}

template <bool BF16, int TW>              // up to 128
__global__ __launch_bounds__(256) void gate_lanes_kernel_wide(const uint16_t *__restrict__ x, const uint16_t *__restrict__ wg, const float *__restrict__ bias,
                                                              const uint8_t *__restrict__ finished, int T, int d, int E, int k, int renorm,
                                                              int32_t *__restrict__ expert_idx, float *__restrict__ expert_scale)
{
    gate_chains<BF16, 128, TW>(x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale);
}

template <bool BF16, int NB, int S, int TT, int R, GateLoads LOADS>
static void launch_gate_mfma(const uint16_t *x, const uint16_t *wg, const float *bias, const uint8_t *finished, int T, int d, int E,
                                 int k, int renorm, int32_t *expert_idx, float *expert_scale, hipStream_t s)
{
    const size_t smem = (size_t)4 * 16 * TT * (S * 16 * NB + 4) * sizeof(float);
    static std::atomic<uint64_t> raised;
    raise_lds_limit(reinterpret_cast<const void *>(&gate_mfma_kernel<BF16, NB, S, TT, R, LOADS>), 144 * 1024, raised);
    hipLaunchKernelGGL((gate_mfma_kernel<BF16, NB, S, TT, R, LOADS>), dim3((T + 16 * TT - 1) / (16 * TT)), dim3(256 * S), smem, s, x, wg, bias,
                       finished, T, d, E, k, renorm, expert_idx, expert_scale);
}

// False where a block's tokens have too many features for the LDS.
template <bool BF16, int EP, int TW>
static bool launch_gate_chains(const uint16_t *x, const uint16_t *wg, const float *bias, const uint8_t *finished, int T, int d, int E,
                              int k, int renorm, int32_t *expert_idx, float *expert_scale, hipStream_t s)
{
    constexpr int NT = TW * (EP < 64 ? 64 / EP : 1), NTP = NT < 4 ? 4 : NT;
    const size_t smem = (EP <= 32 ? EP * 1024 : 0) + (size_t)4 * NTP * (EP + 4) * sizeof(float) + (size_t)4 * ((d + 511) / 512 * 16 + 2) * NT * (BF16 ? 32 : 16) + gate_tail_bytes(EP, d);
    if (smem > 152 * 1024) return false;
    auto launch = [&](auto kernel) {
        static std::atomic<uint64_t> raised;
        raise_lds_limit(reinterpret_cast<const void *>(kernel), 152 * 1024, raised);
        hipLaunchKernelGGL(kernel, dim3((T + NT - 1) / NT), dim3(256), smem, s, x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale);
    };
    if constexpr (EP > 64) launch(&gate_lanes_kernel_wide<BF16, TW>);
    else launch(&gate_token_kernel<BF16, EP, TW>);
    return true;
}

template <bool BF16>
static void launch_gate(const uint16_t *x, const uint16_t *wg, const float *bias, const uint8_t *finished, int T, int d, int E,
                        int k, int renorm, int32_t *expert_idx, float *expert_scale, hipStream_t s)
{
    const GateLoads pairs = E % 2 ? ODD_PAIRS : PAIRS;
    // A multiple of four experts up to 128 and few tokens: chains, more tokens per lane rather than more than a block
    // per compute unit (64 experts, d = 4096, 512 tokens, one / two per lane 17.9 / 12.4 us).  (us, caches warm, d = 512 / 1024 / 2048 / 4096, before -> after.  FP16: up to 16
    // experts on the matrix cores, 1 to 1024 tokens 4.1 / 5.3 / 7.3 / 11.3 -> 3.5 / 4.3 / 5.7 / 8.8; 32 experts, 64 tokens, the weight transposed into LDS for the whole block 3.9 / 5.1 / 7.3 / 11.8 ->
    // 3.9 / 4.7 / 6.2 / 9.4, 1024 tokens, matrix cores 4.5 / 6.0 / 9.1 / 15.7 -> 4.5 / 5.4 / 7.4 / 11.5; 64 experts, 64 tokens 4.5 / 6.2 / 9.3 / 15.8 -> 4.0 / 4.9 / 6.6 / 10.2, 1024 tokens, four-token
    // blocks 6.5 / 9.0 / 14.5 / 24.7 -> 5.0 / 6.7 / 9.9 / 17.5; 128 experts, 64 tokens, gate_lanes_kernel 5.9 / 8.4 / 13.2 / 22.1 -> 5.8 / 7.4 / 10.9 / 17.9, 1024 tokens 8.5 / 13.1 / 22.9 / 41.4 ->
    // 7.4 / 10.5 / 17.2 / 30.3.  bf16, 64 tokens: 16 experts 4.5 / 5.6 / 7.6 / 11.6 -> 4.0 / 5.0 / 7.0 / 11.1, 32 4.2 / 5.6 / 8.4 / 14.4 -> 4.2 / 5.2 / 7.0 / 11.0, 64 4.8 / 6.9 / 10.6 / 18.0 -> 4.2 /
    // 5.5 / 7.6 / 12.2.  Not: 513 to 1024 bf16 tokens on 17 to 32 experts, 6.0 / 6.3 at d = 1024; 2048 tokens on 64 experts, d = 4096, 25 / 28.)
    // Features past the last whole block of 128 run after the chain, slower than within it.  Left to the forms below, these / chains: 65 to 127 such features of fewer than 256 with more
    // than 64 experts (133 tokens of 112, 128 experts, 4.9 / 5.9); more than eight of them with more than 512 bf16 tokens on 33 to 64 experts (683 of 1016, 60 experts, 7.9 / 9.0, 993 of 656, 40
    // experts, 7.7 / 8.3).  Long bf16 tokens on up to 16 experts (878 of 6144, 15.8 / 17.5, 443 of 5120 13.6 / 14.3, 770 of 4096 11.7 / 12.3).  Tokens whose fp32 copies
    // the LDS does not hold: more than 512 bf16 tokens on 33 to 64 experts three to a lane while these are a block per compute unit (600 of
    // 10240, 64 experts, two to a lane 70, three 42, four-token blocks 56; 998 of 11416, 36 experts, two to a lane 80, four-token blocks 53).
    if (E % 4 == 0 && E <= 128 && T <= 1024) {
#define MOE_GATE_CHAINS(EP, TW) launch_gate_chains<BF16, EP, TW>(x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale, s)
        const int past = d % kGateBlk;
        bool done = false;
        if (E > 64) done = !(past > 64 && d < 256) && (T <= 256 ? MOE_GATE_CHAINS(128, 1) : T <= 512 ? MOE_GATE_CHAINS(128, 2) : MOE_GATE_CHAINS(128, 4));
        else if (E > 32 && T <= 512) done = T <= 256 ? MOE_GATE_CHAINS(64, 1) : MOE_GATE_CHAINS(64, 2);
        else if (E > 32) done = !(BF16 && past > 8) && (MOE_GATE_CHAINS(64, 4) || (T <= 768 && MOE_GATE_CHAINS(64, 3)));
        else if (E <= 16) done = (!BF16 || d <= (T <= 512 ? 4352 : 3072)) && MOE_GATE_CHAINS(16, 1);
        else if (T <= 512) done = MOE_GATE_CHAINS(32, 1);
        else if constexpr (!BF16) done = MOE_GATE_CHAINS(32, 2);
#undef MOE_GATE_CHAINS
        if (done) return;
    }
    // 33 to 64 experts else and up to four tokens per compute unit: four-token blocks on the matrix
    // cores; FP16 tokens, more than one such block and up to a token per compute unit: a lane per expert.  (Lane per expert / four-token /
    // sixteen-token blocks, warm, 36 to 60 experts, d = 1024: T = 64 8.4 / 9.2 / 9.9 us, 300 11.9 / 9.2 / 10.2, 1000 20.5 / 9.3 / 10.1,
    // 2000 37 / 15.9 / 10.1; d = 4096, T = 64 21.0 / 24.9 / 25.3; bf16 27.6 / 24.9 / 25.3.  Odd numbers of experts: one token 7.4 / 8.3 / 11.3,
    // 2000 37 / 15.8 / 12.2.)
    if (E > 32 && E <= 64 && T <= 1024) {
        if (!BF16 && T > 4 && T <= 256)
            hipLaunchKernelGGL((gate_lanes_kernel<BF16, 1, WIDE, 1, 2>), dim3(T), dim3(256), 0, s, x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale);
        else if (E % 4) hipLaunchKernelGGL((gate_quad_kernel<BF16, 8, false>), dim3((T + 3) / 4), dim3(256), 0, s, x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale);
        else hipLaunchKernelGGL((gate_quad_kernel<BF16, 8, true>), dim3((T + 3) / 4), dim3(256), 0, s, x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale);
        return;
    }
    // More than 64 experts else: a block per token up to one per compute unit, then two, then four, as far as that is faster than the
    // matrix cores (d = 1024, T = 1024, FP16, lanes / matrix cores: 127 experts 15.4 / 21.9 us, 256 22.7 / 24.9; T = 1500: 255 33.2 / 51, 250 30 / 41, 256 32.5 / 25;
    // multiples of four up to 128 experts, as far as they come here, bf16, T = 1024, 17.0 / 15.0, d = 4096 48 / 42).
    const int few = E > 128 ? (E % 8 ? 2048 : 1024) : E % 2 ? (d <= 1024 ? 2048 : 1024) : !BF16 && d <= 2048 ? 1024 : 512;
    if (E > 64 && T <= few) {
#define MOE_GATE_LANES(NE, LOADS, TB, R) \
    hipLaunchKernelGGL((gate_lanes_kernel<BF16, NE, LOADS, TB, R>), dim3((T + TB - 1) / TB), dim3(256), 0, s, x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale)
#define MOE_GATE_LANES_TB(NE, LOADS) \
    do { \
        constexpr int R = NE == 2 ? 3 : 2; \
        if (T <= 256) MOE_GATE_LANES(NE, LOADS, 1, R); \
        else if (T <= 512) MOE_GATE_LANES(NE, LOADS, 2, R); \
        else MOE_GATE_LANES(NE, LOADS, 4, 2); \
    } while (0)
        if (E <= 128) {
            if (pairs == PAIRS) MOE_GATE_LANES_TB(2, WIDE);
            else MOE_GATE_LANES_TB(2, ODD_PAIRS);
        } else {
            if (E % 4 == 0) MOE_GATE_LANES_TB(4, WIDE);
            else if (pairs == PAIRS) MOE_GATE_LANES_TB(4, PAIRS);
            else MOE_GATE_LANES_TB(4, ODD_PAIRS);
        }
#undef MOE_GATE_LANES_TB
#undef MOE_GATE_LANES
        return;
    }
    // Two row tiles per wavefront (one load and conversion of the gate weight for 32 tokens) once that still gives every
    // compute unit a block.  (T = 8192, d = 4096, 64 experts: 48.5 against 52 us; T = 4096: 45 against 30 us.)  With up to 16
    // experts the conversions of the tokens, not of the weights, are the larger part: one tile always.
    const bool two = (T + 31) / 32 >= 256;
#define MOE_GATE_MFMA(NB, S, TT, R, LOADS) launch_gate_mfma<BF16, NB, S, TT, R, LOADS>(x, wg, bias, finished, T, d, E, k, renorm, expert_idx, expert_scale, s)
    if (E <= 16) MOE_GATE_MFMA(1, 1, 1, 8, WIDE);
    else if (E <= 32) {
        if (E % 2) MOE_GATE_MFMA(2, 1, 1, 4, ODD_PAIRS);
        else if (two) MOE_GATE_MFMA(2, 1, 2, 4, WIDE);
        else MOE_GATE_MFMA(2, 1, 1, 4, WIDE);
    } else if (E <= 64) {
        if (E % 2) MOE_GATE_MFMA(4, 1, 1, 4, ODD_PAIRS);
        else if (E % 4) MOE_GATE_MFMA(4, 1, 1, 4, PAIRS);
        else if (two) MOE_GATE_MFMA(4, 1, 2, 4, WIDE);
        else MOE_GATE_MFMA(4, 1, 1, 6, WIDE);
    } else if (E <= 128) {
        if (E % 2) MOE_GATE_MFMA(4, 2, 1, 4, ODD_PAIRS);
        else if (E % 4) MOE_GATE_MFMA(4, 2, 1, 4, PAIRS);
        else if (two) MOE_GATE_MFMA(4, 2, 2, 4, WIDE);
        else MOE_GATE_MFMA(4, 2, 1, 4, WIDE);
    } else {
        if (E % 2 && two) MOE_GATE_MFMA(8, 2, 2, 1, ODD_PAIRS);
        else if (E % 2) MOE_GATE_MFMA(8, 2, 1, 2, ODD_PAIRS);
        else if (E % 8 && two) MOE_GATE_MFMA(8, 2, 2, 1, PAIRS);
        else if (E % 8) MOE_GATE_MFMA(8, 2, 1, 3, PAIRS);
        else MOE_GATE_MFMA(8, 2, 1, 3, WIDE);
    }
#undef MOE_GATE_MFMA
}

}  // namespace moe

extern "C" int moe_gate_topk(const void *x, int act_dtype, const void *wg, const float *bias,
                             const uint8_t *finished, int T, int d, int E, int k, int renormalize,
                             int32_t *expert_idx, float *expert_scale, void *stream)
{
    using namespace moe;
    if (T == 0 && d > 0 && E > 0) return MOE_OK;         // nothing to route (empty buffers may be NULL)
    if (!x || !wg || !expert_idx || !expert_scale) return fail(MOE_ERR_INVALID_ARG, "moe_gate_topk: NULL pointer");
    if (T < 0 || d <= 0 || E <= 0) return fail(MOE_ERR_INVALID_ARG, "moe_gate_topk: T >= 0, d > 0, E > 0 required");
    if (d % 8) return fail(MOE_ERR_INVALID_ARG, "moe_gate_topk: d %% 8 != 0 (d=%d)", d);
    if (k < 1 || k > 2 || k > E) return fail(MOE_ERR_INVALID_ARG, "moe_gate_topk: k must be 1 or 2 and <= E (k=%d E=%d)", k, E);
    if (E > 256) return fail(MOE_ERR_UNSUPPORTED, "moe_gate_topk: E=%d above 256", E);
    if (act_dtype != MOE_F16 && act_dtype != MOE_BF16) return fail(MOE_ERR_UNSUPPORTED, "moe_gate_topk: act_dtype must be fp16 or bf16");
    if (!aligned16(x) || !aligned16(wg)) return fail(MOE_ERR_INVALID_ARG, "moe_gate_topk: x and wg must be 16-byte aligned");
    hipStream_t s = as_stream(stream);
    const uint16_t *xp = (const uint16_t *)x, *wp = (const uint16_t *)wg;
    if (act_dtype == MOE_BF16) launch_gate<true>(xp, wp, bias, finished, T, d, E, k, renormalize, expert_idx, expert_scale, s);
    else launch_gate<false>(xp, wp, bias, finished, T, d, E, k, renormalize, expert_idx, expert_scale, s);
    return check_launch("moe_gate_topk");
}
