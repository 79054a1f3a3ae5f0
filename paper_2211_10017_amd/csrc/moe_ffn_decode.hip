// The expert FFN of a decode-sized batch (Sec. 3.3 steps 2-4 with the fused dequantisation of
// Sec. 3.4) in one streaming launch plus a small reduction: the stable sort by expert is rebuilt from
// the gate's output, and fc1, the activation and fc2 run in one grid.
//
// Such a batch (the decoder-like case of Table 1: a few rows per expert) is bound by pulling every
// active expert's packed weights through the chip once.  The work is cut along d_ff: a work item is (expert that has rows,
// sixteen or thirty-two of its rows, slice of 64 CW channels of d_ff), one block of eight wavefronts, and the grid holds a
// block per item for any routing, dealt out by the hardware as blocks end (the few without an item find that out and end).  The block
// computes its slice of h = act(x W1 + b1) - a wavefront 64 channels over a CW-th part of an eighth of K, the parts meet in LDS -, keeps it in LDS
// in the rows' type and multiplies it at once with the matching rows of W2 (a wavefront an eighth of the output channels): h never goes to memory.
// What is left over is a partial sum of y per slice, stored as fp32 rows; decode_reduce_kernel then adds the
// slices in a fixed order, applies W2's channel scale, the bias and the gate scale, and sums a token's experts in slot
// order into the layer output (no atomics, nothing to clear, nothing to wait for inside a launch).
//
// What bounds it: one token, the latencies in a row (the gate's indices 1 us, the weights 2, each phase's instructions, which no
// block has run before: about 100 clocks per 64 bytes of code), 64 tokens, the weight stream and the unpacking beside it.  Small
// blocks are dealt out as others end, so no compute unit's share is fixed, and one token's two experts of 1024 x 4096 are 128 blocks
// over the chip: kernel and reduction 10.8 us where sixteen workgroups of sixteen wavefronts, one per slice of 512
// channels, took 22; 64 tokens 34.6 against 33; a step of 64 tokens, 64 experts of 4096 x 16384, group scales, 803 -> 732 against two launches in
// row tiles.  Fewer registers beat longer rings (4-bit, FP16: 24 wavefronts per compute unit with two 1 KB blocks of fc1 and four of fc2
// in flight 28.8 us, sixteen with six and eight 31.1), and two fc2 units at a time one (12 against 17 us for a block's 512 channels).
//
// The rows of an item (sixteen, thirty-two where experts are expected to have more than eight) are the A operand of
// v_mfma_f32_16x16x32_f16, fetched from the tokens in operand order; an expert with more rows has several items, whose blocks read its weights
// at about the same time.  (As passes of one block they left most of a crowded batch's chip idle: 64 tokens on two of 64 experts of 4096 x 16384,
// group scales, 383 -> 133 us a step, 143 in row tiles; on two of 32 of 1024 x 4096, bf16, 78 -> 29 and 44; 192 on two 190 -> 43 and 40, on
// four of 64 of 4096 x 16384, 64 tokens, 298 -> 197 and 184.  Even routing gains what a kernel without the loop has in registers: 0 to 3 %.)
// Where items may have thirty-two rows those of up to sixteen run the code for sixteen: half the products, more of fc2 in flight (192 tokens,
// two of 32 of 1024 x 4096, a third of them ended 43.1 -> 41.6, none 43.7 and 43.9; 71, two of 16, group scales 32.7 -> 28.0).
// The weights go through the magic-number conversion into the B operand.  Group scales multiply the fp32 sums of 64 K values of exact
// codes.  bf16 rows, and the slice of h rounded to bf16, are operands as they are, the codes being exact in bf16 too (codes_to_bf16).  Where rows
// come sixteen at a time and meet group scales they are scaled per row and 64 K values by a power of two into the FP16 range (exact) instead, and so is the slice of h per row, after its
// rounding to bf16: the unpacking of the codes then costs less than the searches for each row's largest.  (us a step, scaled / as they are: 64 tokens, two of 32 experts of
// 1024 x 4096, group scales 41.8 / 43.1, 16 37.9 / 38.6; channel scales 40.7 / 40.7; 20, two of 32 of 2048 x 8192 113.7 / 109.3, 40, two of 16 of 768 x 3072 25.7 / 25.0, 20, one
// of 32 of 1024 x 4096, 8-bit, 36.2 / 34.0; same bits.)
#include <math.h>

#include <type_traits>

#include "moe_ffn_common.h"

// Hook for timing studies: a harness that includes this file may define it to record a time stamp per block at the named points;
// the library builds it empty.
#ifndef MOE_DEC_STAMP
#define MOE_DEC_STAMP(slot)
#endif

namespace moe {

constexpr int kDecWaves = 8;             // wavefronts per block
constexpr int kDecThreads = kDecWaves * 64;
constexpr int kDecFit = 16;              // rows of an item (one 16-row matrix tile)

typedef float float4_t __attribute__((ext_vector_type(4)));
typedef uint32_t dec_u32x4 __attribute__((ext_vector_type(4)));

// Loads through buffer descriptors: what changes per load is in the descriptor (scalar registers), the lane's offset in one vector
// register for all of them.  The hardware compares a lane's offset with the extent LESS the instruction's scalar offset, which wraps
// for an extent of zero, so no load here has a scalar offset: the base is moved instead.
__device__ inline __amdgpu_buffer_rsrc_t dec_rsrc(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, (int)bytes, 0x00020000);
}

// 16 bytes per lane of one 1 KB fragment block, non-temporal: the weights of a launch are read once and must not push the small
// hot arrays out of the caches.  Not `live`: the descriptor has no extent, the load returns zero without touching memory, and
// the number of loads in flight does not depend on how long a wavefront's stream is.
__device__ inline uint4 dec_load(const uint8_t *block, bool live, uint32_t lane_off)
{
    const __amdgpu_buffer_rsrc_t r = dec_rsrc(block, live ? kFragBytes : 0);
    const dec_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, lane_off, 0, 2 /* nt */);
    return make_uint4(v.x, v.y, v.z, v.w);
}

// Value of lane `first + (lane's byte offset / 4)`, both from registers (first: a constant).
__device__ inline float dec_lane(float v, int byte_off, int first)
{
    return __int_as_float(__builtin_amdgcn_ds_bpermute(byte_off + 4 * first, __float_as_int(v)));
}

// Rows 1 and 3 (of sixteen lanes each) of `a` change places with rows 0 and 2 of `b`.  A fragment
// block holds, per MFMA step j of the 32-row layout, [ch 0-15 | ch 16-31 | ch 0-15 | ch 16-31] x
// [k 0-7, k 0-7, k 8-15, k 8-15]; swapping steps j and j+1 this way leaves `a` with channels 0-15
// and `b` with channels 16-31, each over the four k octets {0-7, 16-23, 8-15, 24-31} of the two
// steps: the B operand of a 16x16x32 instruction whose A operand reads its k octets in that order.
__device__ inline void swap_rows(uint32_t &a, uint32_t &b)
{
    const auto r = __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// RT x 16 rows x 32 channels x 64 K values: one fragment block of 4-bit or two of 8-bit weights, a[] the two 32-deep operands of
// each sixteen rows.
template <int BITS, int RT, bool BF16>
__device__ inline void dec_mac(const uint4 (&w)[BITS / 4], const uint4 (&a)[RT][2], float4_t (&lo)[RT], float4_t (&hi)[RT])
{
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        auto products = [&](const uint32_t (&bw)[4], float4_t (&acc)[RT]) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) {
                if constexpr (BF16) acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[rt][q]), __builtin_bit_cast(bf16x8_t, frag_from(bw)), acc[rt], 0, 0, 0);
                else acc[rt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a[rt][q]), frag_from(bw), acc[rt], 0, 0, 0);
            }
        };
        uint32_t bw[4];
        auto convert = [&](uint32_t c0, uint32_t c1) {
            const uint32_t c[2] = {c0, c1};
            if constexpr (BF16) codes_to_bf16<BITS>(c, bw);
            else if constexpr (BITS == 4) dequant4(c0, bw);
            else dequant8(c0, c1, bw);
        };
        if constexpr (BITS == 4) {
            uint32_t r0 = q ? w[0].z : w[0].x, r1 = q ? w[0].w : w[0].y;
            swap_rows(r0, r1);
            convert(r0, 0);
            products(bw, lo);
            convert(r1, 0);
            products(bw, hi);
        } else {
            uint32_t r0 = w[q].x, r1 = w[q].y, r2 = w[q].z, r3 = w[q].w;
            swap_rows(r0, r2);
            swap_rows(r1, r3);
            convert(r0, r1);
            products(bw, lo);
            convert(r2, r3);
            products(bw, hi);
        }
    }
}

// Power of two that brings a bf16 magnitude `amax` (bits, sign cleared) into [2^14, 2^15), and its reciprocal.
__device__ inline void dec_row_pow(uint32_t amax, float &down, float &up)
{
    int ex = (int)(amax >> 7);
    if (ex == 255) ex = 141;                            // inf/nan: factor 1 (the result is nan anyway)
    const int fe = min(max(268 - ex, 1), 253);
    down = __uint_as_float((uint32_t)fe << 23);
    up = __uint_as_float((uint32_t)(254 - fe) << 23);
}

__device__ inline uint32_t dec_max_bf16(uint32_t amax, uint32_t pair)
{
    return max(amax, max(pair & 0x7fffu, (pair >> 16) & 0x7fffu));
}

// The same wavefront-wide for values that sixteen-lane rows share: maximum over lanes l, l ^ 16, l ^ 32, l ^ 48.
__device__ inline uint32_t dec_max_over_rows(uint32_t v)
{
    v = max(v, (uint32_t)__shfl_xor((int)v, 16));
    return max(v, (uint32_t)__shfl_xor((int)v, 32));
}

__device__ inline uint32_t dec_bf16_pair_to_f16(uint32_t pair, float down)
{
    const half2_t h = {(_Float16)__builtin_fmaf(__uint_as_float(pair << 16), down, 0.0f),
                       (_Float16)__builtin_fmaf(__uint_as_float(pair & 0xffff0000u), down, 0.0f)};
    return h2_bits(h);
}

// The stable sort by expert, for the callers: perm_src, inv_perm and expert_offsets (pruned rows, key E, come last).  One block;
// up to 512 keys, every thread counts what precedes its own.
__device__ inline void dec_write_index(const DecodeArgs &p, int32_t *s_key, int v)
{
    const int tid = threadIdx.x, n = p.n_assign;
    s_key[tid] = v;
    __syncthreads();
    auto count = [&](auto less) {
        int r = 0;
        for (int i = 0; i < n; i += 4) {
            const int4 q = *reinterpret_cast<const int4 *>(s_key + i);
            r += less(q.x, i) + less(q.y, i + 1) + less(q.z, i + 2) + less(q.w, i + 3);
        }
        return r;
    };
    if (tid < n) {
        const int r = count([&](int key, int i) { return (int)(key < v || (key == v && i < tid)); });
        p.inv_perm_out[tid] = r;
        p.perm_src_out[r] = tid;
    }
    for (int e = tid; e <= p.E; e += kDecThreads) p.offsets_out[e] = count([&](int key, int) { return (int)(key < e); });
}

// BITS: weight width.  GROUPED: group scales (groups of a multiple of 64 K values).  BF: bf16 rows.  CW: 64-channel parts of a slice.
// MOST: sixteens of rows per item at most; with two, items of up to sixteen rows run the code for one.
template <int BITS, bool GROUPED, bool BF, int CW, int MOST>
__global__ __launch_bounds__(kDecThreads, !GROUPED && MOST == 1 && (BITS == 4 || CW > 1) ? 6 : 4) void decode_ffn_kernel(DecodeArgs p)
{
    constexpr int NW = BITS / 4;                        // fragment blocks of a slab per 64 K values (a "unit")
    constexpr int KP = kDecWaves / CW, CH = 64 * CW;    // parts of K in fc1; channels of the slice
    constexpr int FIT = kDecFit * MOST;
    constexpr int LDR = CH + 4, LDH = CH + 8;
    // How bf16 rows meet the codes: as they are, or (group scales, one sixteen of rows per item) scaled to FP16
    constexpr bool SCALED = BF && GROUPED && MOST == 1, CODES = BF && !SCALED;
    constexpr float UNIT = CODES ? kBf16CodeUnit : 1.0f;                 // (bf16 codes are q / kBf16CodeUnit)
    __shared__ __align__(16) float s_red[KP * kDecFit * LDR];
    __shared__ __align__(16) uint16_t s_h[FIT * LDH];
    __shared__ __align__(16) int32_t s_row[kDecMaxAssign];      // assignments of the block's expert
    __shared__ int s_wave[kDecWaves];                           // rows of the expert among each wavefront's assignments
    __shared__ float s_pow[SCALED ? FIT : 1];
    int *const s_cnt = reinterpret_cast<int *>(s_red);          // rows of every expert, until fc1's sums need the place
    static_assert(sizeof(s_red) >= kDecMaxExperts * sizeof(int), "the experts' counters fit");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int E = p.E, F = p.F, d = p.d, S = F / CH;
    MOE_DEC_STAMP(0);
    const int v_exp = tid < p.n_assign ? p.gate_idx[tid] : 0x7fffffff;
    if (blockIdx.x == 0) {
        dec_write_index(p, s_row, v_exp);
        return;
    }
    const int c = (int)(blockIdx.x - 1) % S;
    // ---- the block's item: the (blockIdx - 1) / S -th (expert that has rows, FIT of its rows), experts in ascending order.
    // A lane sums the items of `span` neighbouring experts; more than 64 experts: the lanes then look into the span that was hit.
    const int span = (E + 63) / 64;
    for (int i = tid; i < 64 * span; i += kDecThreads) s_cnt[i] = 0;
    __syncthreads();
    if ((uint32_t)v_exp < (uint32_t)E) atomicAdd(&s_cnt[v_exp], 1);
    __syncthreads();
    int e, rows, z0;
    {
        int item = (int)(blockIdx.x - 1) / S, first = 0;
        auto find = [&](int cnt) {                      // the lane that holds the item; `item` becomes its number there
            const int incl = wave_inclusive_sum(cnt);
            const uint64_t hit = __ballot(incl > item);
            if (!hit) return -1;
            const int src = __ffsll((unsigned long long)hit) - 1;
            item -= __shfl(incl - cnt, src);
            return src;
        };
        auto groups = [&](int i) { return (s_cnt[i] + FIT - 1) / FIT; };
        int cnt = 0;
        for (int i = 0; i < span; ++i) cnt += groups(lane * span + i);
        int src = find(cnt);
        if (src < 0) return;                            // fewer items than there are blocks for
        if (span > 1) {
            first = src * span;
            src = find(lane < span ? groups(first + lane) : 0);
        }
        e = __builtin_amdgcn_readfirstlane(first + src);
        z0 = __builtin_amdgcn_readfirstlane(item) * FIT;
        rows = min(FIT, __builtin_amdgcn_readfirstlane(s_cnt[e]) - z0);
    }

    MOE_DEC_STAMP(1);
    auto run = [&](auto rt_c) __attribute__((always_inline)) {
        constexpr int RT = decltype(rt_c)::value;           // sixteens of rows of this item
        // units of fc2 in flight per wavefront (and one of fc1); two of 8-bit weights leave room for a third block per compute unit (20 tokens, one of
        // 32 experts of 1024 x 4096, a step 30.3 -> 28.8 us; for slices of 64 channels, few blocks at all, 15.8 and 15.9, four)
        constexpr int U2 = (RT > 1 && GROUPED) || (BITS == 8 && !GROUPED && CW > 1) ? 2 : 4;
        // ---- weight streams
        const uint32_t lane_off = (uint32_t)lane * 16u;
        const int cg = wave % CW, kp = wave / CW;
        const int nk = d / 64, per = (nk + KP - 1) / KP, u0 = kp * per, n1 = max(min(nk - u0, per), 0);
        const int ktot = F / 64;                            // units of a slab of W2
        const int nslab = d / 32, spw = (nslab + kDecWaves - 1) / kDecWaves, slab0 = wave * spw;
        const int n2 = max(min(nslab - slab0, spw), 0) * CW;
        const uint8_t *w1 = p.w1 + (size_t)e * packed_bytes_per_expert(d, F, BITS) + ((size_t)(c * CW + cg) * 2 * nk + u0) * NW * kFragBytes;
        const uint8_t *w2 = p.w2 + (size_t)e * packed_bytes_per_expert(F, d, BITS) + ((size_t)slab0 * ktot + c * CW) * NW * kFragBytes;
        const uint16_t *s1 = reinterpret_cast<const uint16_t *>(p.s1) + (size_t)e * (GROUPED ? d / p.g : 1) * F + c * CH;
        const uint16_t *s2 = reinterpret_cast<const uint16_t *>(p.s2) + (size_t)e * (GROUPED ? F / p.g : 1) * d + slab0 * 32;

        auto group_of = [&](int u) { return p.group_inv ? (int)__umulhi((uint32_t)u, p.group_inv) : u; };      // unit -> group
        uint4 W[2][NW], A[RT][2], V[U2][NW];
        uint16_t gs1, gs2[GROUPED ? U2 : 1];        // group scales: lane l brings channel l of the wavefront's 64, l % 32 of the slab's 32
        auto load_w1 = [&](int u) {
#pragma unroll
            for (int s = 0; s < 2; ++s)
#pragma unroll
                for (int w = 0; w < NW; ++w) W[s][w] = dec_load(w1 + ((size_t)s * nk + u) * NW * kFragBytes + w * kFragBytes, u < n1, lane_off);
            if constexpr (GROUPED) gs1 = __builtin_amdgcn_raw_buffer_load_b16(dec_rsrc(s1 + (size_t)group_of(u0 + u) * F + cg * 64, u < n1 ? 128 : 0), lane * 2, 0, 0);
        };
        auto load_w2 = [&](int slot, int j) {
            const int slab = j / CW, unit = j % CW;
#pragma unroll
            for (int w = 0; w < NW; ++w) V[slot][w] = dec_load(w2 + ((size_t)slab * ktot + unit) * NW * kFragBytes + w * kFragBytes, j < n2, lane_off);
            if constexpr (GROUPED) {
                gs2[slot] = __builtin_amdgcn_raw_buffer_load_b16(dec_rsrc(s2 + (size_t)group_of(c * CW + unit) * d + slab * 32, j < n2 ? 64 : 0), (lane & 31) * 2, 0, 0);
            }
        };
        // (the weights depend on the expert alone: the rows are found under their flight)
        load_w1(0);
#pragma unroll
        for (int i = 0; i < U2; ++i) load_w2(i, i);
        __builtin_amdgcn_sched_barrier(0);
        // ---- the item's rows, in the order of the assignments: blocks of other slices and of the expert's other items share them out alike
        const bool mine = v_exp == e;
        const uint64_t wave_rows = __ballot(mine);
        if (lane == 0) s_wave[wave] = __popcll(wave_rows);
        __syncthreads();
        if (mine) {
            int r = __popcll(wave_rows & ((1ull << lane) - 1)) - z0;
            for (int w = 0; w < wave; ++w) r += s_wave[w];
            if ((uint32_t)r < (uint32_t)FIT) s_row[r] = tid;
        }
        // channel factors of the thread's part of h: row tid / 32, 2 CW channels
        constexpr int HC = 2 * CW;
        const int h_row = tid >> 5, h_ch = (tid & 31) * HC;
        uint32_t hs[CW], hb[CW];
        auto load_factors = [&]() {
#pragma unroll
            for (int i = 0; i < CW; ++i) {
                hs[i] = GROUPED ? 0 : reinterpret_cast<const uint32_t *>(s1 + h_ch)[i];
                hb[i] = p.b1 ? reinterpret_cast<const uint32_t *>(reinterpret_cast<const uint16_t *>(p.b1) + (size_t)e * F + c * CH + h_ch)[i] : 0;
            }
        };
        if constexpr (CW <= 2) load_factors();              // (wider slices have no registers to carry them through fc1)
        __syncthreads();
        MOE_DEC_STAMP(2);
        const uint32_t x_bytes = (uint32_t)(p.n_assign >> (p.gate_k - 1)) * d * 2u;
        const int lane16 = (lane & 15) * 4, lane_row = (lane >> 4) * 16;     // byte offsets of dec_lane
        // k octet this lane's quarter of the wavefront reads within a 32-deep step (see swap_rows)
        const int koct = ((lane >> 4) & 1) * 16 + (lane >> 5) * 8;
        // rows of x in operand order: only the lanes of live rows read (the others are past the tokens, which reads as zero)
        uint32_t a_off[RT];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int m = 16 * rt + (lane & 15), tok = s_row[min(m, rows - 1)] >> (p.gate_k - 1);      // one or two experts per token
            a_off[rt] = m < rows ? ((uint32_t)tok * d + koct) * 2u : 0x7fffff00u;
        }
        auto load_a = [&](int u) {
            const __amdgpu_buffer_rsrc_t r = dec_rsrc(p.x + (u0 + u) * 64, u < n1 ? x_bytes - (u0 + u) * 128 : 0);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const dec_u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(r, a_off[rt] + 64 * q, 0, 0);
                    A[rt][q] = make_uint4(v.x, v.y, v.z, v.w);
                }
        };
        load_a(0);

        // ---- fc1: the rows x 64 channels over the wavefront's part of K
        float4_t acc[4][RT];
        auto clear = [&](float4_t (&t)[RT]) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) t[rt] = float4_t{0.f, 0.f, 0.f, 0.f};
        };
#pragma unroll
        for (int t = 0; t < 4; ++t) clear(acc[t]);
        for (int u = 0; u < n1; ++u) {
            float up[RT];
            if constexpr (SCALED) {
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    uint32_t amax = 0;
#pragma unroll
                    for (int q = 0; q < 2; ++q) {
                        amax = dec_max_bf16(dec_max_bf16(amax, A[rt][q].x), A[rt][q].y);
                        amax = dec_max_bf16(dec_max_bf16(amax, A[rt][q].z), A[rt][q].w);
                    }
                    float down;
                    dec_row_pow(dec_max_over_rows(amax), down, up[rt]);
#pragma unroll
                    for (int q = 0; q < 2; ++q)
                        A[rt][q] = make_uint4(dec_bf16_pair_to_f16(A[rt][q].x, down), dec_bf16_pair_to_f16(A[rt][q].y, down),
                                              dec_bf16_pair_to_f16(A[rt][q].z, down), dec_bf16_pair_to_f16(A[rt][q].w, down));
                }
            }
            if constexpr (GROUPED || BF) {              // the unit's sums, folded with the group's scale in fp32 (bf16: short sums, as h keeps few bits)
#pragma unroll
                for (int t = 0; t < 4; t += 2) {        // (one slab, then the other)
                    float4_t part[2][RT];
                    clear(part[0]), clear(part[1]);
                    dec_mac<BITS, RT, CODES>(W[t / 2], A, part[0], part[1]);
                    float sf[2];
#pragma unroll
                    for (int i = 0; i < 2; ++i) sf[i] = GROUPED ? dec_lane((float)__builtin_bit_cast(_Float16, gs1) * UNIT, lane16, 16 * (t + i)) : 1.0f;
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const float pw = SCALED ? dec_lane(up[rt], lane_row, r) : 1.0f;
#pragma unroll
                            for (int i = 0; i < 2; ++i) acc[t + i][rt][r] = GROUPED ? fmaf(part[i][rt][r], sf[i] * pw, acc[t + i][rt][r]) : part[i][rt][r] + acc[t + i][rt][r];
                        }
                    if (RT > 1) __builtin_amdgcn_sched_barrier(0);
                }
            } else {
                dec_mac<BITS, RT, false>(W[0], A, acc[0], acc[1]);
                dec_mac<BITS, RT, false>(W[1], A, acc[2], acc[3]);
            }
            load_w1(u + 1);
            load_a(u + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        MOE_DEC_STAMP(3);
        if constexpr (CW > 2) load_factors();
        // ---- the parts of K meet, sixteen rows at a time: rows 16 rt + 4 (lane / 16) + r, channels 64 cg + 16 t + lane % 16
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            if (rt) __syncthreads();                    // the sixteen rows before have been read
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) s_red[(kp * kDecFit + 4 * (lane >> 4) + r) * LDR + cg * 64 + 16 * t + (lane & 15)] = acc[t][rt][r];
            __syncthreads();
            float v[HC];
#pragma unroll
            for (int i = 0; i < HC; ++i) v[i] = s_red[h_row * LDR + h_ch + i];
#pragma unroll
            for (int q = 1; q < KP; ++q)
#pragma unroll
                for (int i = 0; i < HC; ++i) v[i] += s_red[(q * kDecFit + h_row) * LDR + h_ch + i];
#pragma unroll
            for (int i = 0; i < HC; ++i) {
                const half2_t s2v = bits_h2(hs[i >> 1]), b2v = bits_h2(hb[i >> 1]);
                v[i] = fmaf(v[i], GROUPED ? 1.0f : (float)s2v[i & 1] * UNIT, (float)b2v[i & 1]);
            }
            if (p.act == MOE_ACT_GELU) {
#pragma unroll
                for (int i = 0; i < HC; ++i) v[i] = activate(v[i], MOE_ACT_GELU);
            } else {
#pragma unroll
                for (int i = 0; i < HC; ++i) v[i] = activate(v[i], MOE_ACT_RELU);
            }
            if constexpr (SCALED) {
                uint32_t amax = 0;
                float down, up;
#pragma unroll
                for (int i = 0; i < HC; ++i) {
                    v[i] = __uint_as_float((uint32_t)to_bf16_rne(v[i]) << 16);
                    amax = max(amax, (__float_as_uint(v[i]) >> 16) & 0x7fffu);
                }
#pragma unroll
                for (int off = 16; off > 0; off >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, off));
                dec_row_pow(amax, down, up);
                if ((tid & 31) == 0) s_pow[16 * rt + h_row] = up;
#pragma unroll
                for (int i = 0; i < HC; ++i) v[i] *= down;
            }
#pragma unroll
            for (int i = 0; i < HC; i += 2) {
                const half2_t hv = {(_Float16)v[i], (_Float16)v[i + 1]};
                *reinterpret_cast<uint32_t *>(s_h + (16 * rt + h_row) * LDH + h_ch + i) = CODES ? to_bf16_rne(v[i]) | (uint32_t)to_bf16_rne(v[i + 1]) << 16 : h2_bits(hv);
            }
        }
        __syncthreads();

        MOE_DEC_STAMP(4);
        // ---- fc2 on the slice: the rows x 32 output channels per slab, K = the slice's channels
        const uint16_t *h_ptr = s_h + (lane & 15) * LDH + koct;
        float *const part_c = p.partial + (size_t)c * p.n_assign * d + slab0 * 32;
        int row_off[RT][4];
        float pw[RT][4];
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = 16 * rt + 4 * (lane >> 4) + r;
                row_off[rt][r] = m < rows ? s_row[m] * d + (lane & 15) : -1;
                pw[rt][r] = SCALED ? s_pow[m] : 1.0f;
            }
        float4_t y0[RT], y1[RT];
        clear(y0), clear(y1);
        auto read_h = [&](int unit, uint4 (&a)[RT][2]) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int q = 0; q < 2; ++q) a[rt][q] = *reinterpret_cast<const uint4 *>(h_ptr + 16 * rt * LDH + unit * 64 + 32 * q);
        };
        auto unit_mac = [&](int i, const uint4 (&a)[RT][2], float4_t (&lo)[RT], float4_t (&hi)[RT]) {
            if constexpr (GROUPED) {
                float4_t p0[RT], p1[RT];
                clear(p0), clear(p1);
                dec_mac<BITS, RT, CODES>(V[i], a, p0, p1);
                const float sl = (float)__builtin_bit_cast(_Float16, gs2[i]) * UNIT, f0 = dec_lane(sl, lane16, 0), f1 = dec_lane(sl, lane16, 16);
#pragma unroll
                for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                    for (int r = 0; r < 4; ++r) lo[rt][r] = fmaf(p0[rt][r], f0, lo[rt][r]), hi[rt][r] = fmaf(p1[rt][r], f1, hi[rt][r]);
            } else {
                dec_mac<BITS, RT, CODES>(V[i], a, lo, hi);
            }
        };
        auto store = [&](int n, const float4_t (&lo)[RT], const float4_t (&hi)[RT]) {       // this slice's part of y, channels n .. n + 31
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row_off[rt][r] >= 0) {
                        part_c[row_off[rt][r] + n] = SCALED ? lo[rt][r] * pw[rt][r] : lo[rt][r];
                        part_c[row_off[rt][r] + n + 16] = SCALED ? hi[rt][r] * pw[rt][r] : hi[rt][r];
                    }
        };
        // two units at a time, whose chains of unpacking and products the wavefront interleaves: two slabs (slices of 64 channels)
        // or two units of a slab
        for (int base = 0; base < n2; base += U2) {
#pragma unroll
            for (int i = 0; i < U2; i += 2) {
                const int j = base + i, unit = CW == 1 ? 0 : U2 % CW == 0 ? i % CW : j % CW;
                if (j < n2) {
                    uint4 a0[RT][2];
                    read_h(unit, a0);
                    if constexpr (CW == 1) {
                        float4_t z0v[RT], z1v[RT];
                        clear(y0), clear(y1), clear(z0v), clear(z1v);
                        unit_mac(i, a0, y0, y1);
                        unit_mac(i + 1, a0, z0v, z1v);
                        store(j * 32, y0, y1);
                        if (j + 1 < n2) store(j * 32 + 32, z0v, z1v);
                    } else {
                        uint4 a1[RT][2];
                        read_h(unit + 1, a1);
                        unit_mac(i, a0, y0, y1);
                        unit_mac(i + 1, a1, y0, y1);
                        if (unit == CW - 2) {
                            store(j / CW * 32, y0, y1);
                            clear(y0), clear(y1);
                        }
                    }
                }
                load_w2(i, j + U2);
                load_w2(i + 1, j + 1 + U2);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        MOE_DEC_STAMP(5);
    };
    if (MOST > 1 && rows > kDecFit) run(std::integral_constant<int, MOST>{});
    else run(std::integral_constant<int, 1>{});
}

// Sum of the d_ff slices and of a token's experts: out[t] = sum_j scale[a] * (W2-scale * sum_c partial[c][a] + b2),
// a = t k + j in ascending j; pruned assignments (expert index E) add nothing, so a pruned token's row is zero.
// A block is a token and 1024 / SG channels, four per thread; SG threads share an element's slices, NV of each expert at a time.
// CODES: the partial sums are in units of bf16 codes (bf16 rows, channel scales).
template <int SG, int NV, bool CODES>
__device__ __forceinline__ void decode_reduce(const DecodeArgs &p)
{
    constexpr int LANES = 256 / SG;
    __shared__ float4 s_sum[SG > 1 ? 2 * 256 : 1];
    const int t = blockIdx.x, S = p.F / (64 * p.cw), d = p.d;
    const int sg = threadIdx.x / LANES, ln = threadIdx.x % LANES, n = (blockIdx.y * LANES + ln) * 4;
    const bool in = n < d;
    // the token's experts and what their rows of W2 are scaled with are requested with the slices: found after their sum they are two more
    // trips to memory in a row
    const int J = p.gate_k > 1 ? 2 : 1;
    int e[2];
    float sc[2];
    uint2 s2[2], b2[2];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        e[j] = p.gate_idx[t * J + min(j, J - 1)];
        sc[j] = p.gate_scale[t * J + min(j, J - 1)];
    }
    auto load_factors = [&]() {
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            if (j >= J || (uint32_t)e[j] >= (uint32_t)p.E) e[j] = -1;      // (pruned: nothing of it was written)
            s2[j] = make_uint2(0x3c003c00u, 0x3c003c00u), b2[j] = make_uint2(0, 0);
            if (sg == 0 && in && e[j] >= 0) {
                if (!p.g) s2[j] = *reinterpret_cast<const uint2 *>(p.s2 + (size_t)e[j] * d + n);       // (group scales are in the partial sums)
                if (p.b2) b2[j] = *reinterpret_cast<const uint2 *>(p.b2 + (size_t)e[j] * d + n);
            }
        }
    };
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    float4 y[2] = {acc, acc};
    const float *src = p.partial + (size_t)t * p.gate_k * d + (in ? n : 0);     // (a token's rows of a slice are neighbours)
    const int second = p.gate_k > 1 ? d : 0;
    const size_t step = (size_t)p.n_assign * d;
    for (int c = sg; c - sg < S; c += NV * SG) {
        float4 v[2][NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            v[0][i] = v[1][i] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (c - sg + i * SG < S) {                  // (the same for the whole block)
                const float *q = src + min(c + i * SG, S - 1) * step;
                v[0][i] = *reinterpret_cast<const float4 *>(q);
                v[1][i] = *reinterpret_cast<const float4 *>(q + second);
            }
        }
        if (c == sg) load_factors();
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const bool live = c + i * SG < S;
                y[j].x += live ? v[j][i].x : 0.0f; y[j].y += live ? v[j][i].y : 0.0f; y[j].z += live ? v[j][i].z : 0.0f; y[j].w += live ? v[j][i].w : 0.0f;
            }
    }
    if constexpr (SG > 1) {
        s_sum[threadIdx.x] = y[0];
        s_sum[256 + threadIdx.x] = y[1];
        __syncthreads();
        if (sg) return;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 1; g < SG; ++g) {
                const float4 v = s_sum[j * 256 + g * LANES + ln];
                y[j].x += v.x; y[j].y += v.y; y[j].z += v.z; y[j].w += v.w;
            }
    }
    if (!in) return;
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        if (e[j] < 0) continue;
        const half2_t s01 = bits_h2(s2[j].x), s23 = bits_h2(s2[j].y), b01 = bits_h2(b2[j].x), b23 = bits_h2(b2[j].y);
        constexpr float unit = CODES ? kBf16CodeUnit : 1.0f;
        acc.x += sc[j] * (y[j].x * ((float)s01[0] * unit) + (float)b01[0]);
        acc.y += sc[j] * (y[j].y * ((float)s01[1] * unit) + (float)b01[1]);
        acc.z += sc[j] * (y[j].z * ((float)s23[0] * unit) + (float)b23[0]);
        acc.w += sc[j] * (y[j].w * ((float)s23[1] * unit) + (float)b23[1]);
    }
    if (p.out_dtype == MOE_F32) {
        *reinterpret_cast<float4 *>((float *)p.out + (size_t)t * d + n) = acc;
    } else {
        const float v[4] = {acc.x, acc.y, acc.z, acc.w};
        for (int i = 0; i < 4; ++i) store_out(p.out, p.out_dtype, (size_t)t * d + n + i, v[i]);
    }
}

template <int SG, int NV>
__global__ __launch_bounds__(256) void decode_reduce_kernel(DecodeArgs p)
{
    decode_reduce<SG, NV, false>(p);
}

template <int SG, int NV>
__global__ __launch_bounds__(256) void decode_reduce_codes_kernel(DecodeArgs p)
{
    decode_reduce<SG, NV, true>(p);
}

// ---- host side -----------------------------------------------------------------------------------

template <int SG, int NV>
static void launch_reduce(const DecodeArgs &p, bool codes, hipStream_t s)
{
    const dim3 grid(p.n_assign / p.gate_k, (p.d + 1024 / SG - 1) / (1024 / SG));
    if (codes) hipLaunchKernelGGL((decode_reduce_codes_kernel<SG, NV>), grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL((decode_reduce_kernel<SG, NV>), grid, dim3(256), 0, s, p);
}

template <int BITS, bool GROUPED, bool BF, int RT>
static void launch_decode_rows(const DecodeArgs &p, dim3 grid, hipStream_t s)
{
    if (p.cw == 1) hipLaunchKernelGGL((decode_ffn_kernel<BITS, GROUPED, BF, 1, RT>), grid, dim3(kDecThreads), 0, s, p);
    else if (p.cw == 2) hipLaunchKernelGGL((decode_ffn_kernel<BITS, GROUPED, BF, 2, RT>), grid, dim3(kDecThreads), 0, s, p);
    else if (p.cw == 4) hipLaunchKernelGGL((decode_ffn_kernel<BITS, GROUPED, BF, 4, RT>), grid, dim3(kDecThreads), 0, s, p);
    else hipLaunchKernelGGL((decode_ffn_kernel<BITS, GROUPED, BF, 8, RT>), grid, dim3(kDecThreads), 0, s, p);
}

template <int BITS, bool GROUPED, bool BF>
static void launch_decode(const DecodeArgs &p, dim3 grid, hipStream_t s)
{
    if constexpr (BITS == 4)
        if (p.row_tiles > 1) return launch_decode_rows<BITS, GROUPED, BF, 2>(p, grid, s);
    launch_decode_rows<BITS, GROUPED, BF, 1>(p, grid, s);
}

template <int BITS>
static void launch_decode_bits(const DecodeArgs &p, bool bf, dim3 grid, hipStream_t s)
{
    if (p.g) bf ? launch_decode<BITS, true, true>(p, grid, s) : launch_decode<BITS, true, false>(p, grid, s);
    else bf ? launch_decode<BITS, false, true>(p, grid, s) : launch_decode<BITS, false, false>(p, grid, s);
}

// Sizes the kernel takes.
bool decode_ffn_supports(int n_assign, int k, int E, int d, int F, int bits, int group_size)
{
    if (n_assign < 1 || n_assign > kDecMaxAssign || k < 1 || k > 2 || E < 1 || E > kDecMaxExperts || d <= 0 || F <= 0 || d % 64 || F % 64) return false;
    if ((bits != 4 && bits != 8) || group_size < 0 || (group_size && (group_size % 64 || d % group_size || F % group_size))) return false;
    return (long)n_assign * d < (1l << 29) && (long)d * F * bits / 8 < (1l << 31);      // offsets into x and the partial sums have 31 bits
}

// Experts that n_assign assignments are expected to touch under uniform routing.
double decode_active_experts(int n_assign, int E)
{
    return E * (1.0 - pow(1.0 - 1.0 / E, n_assign));
}

// Channels of d_ff per slice, in 64s: the widest slice that still gives every compute unit a block, give or take.  Narrow slices
// spread few experts over the chip; each slice leaves a partial sum of every row behind, so wide ones move less.  (us a step, slices
// of 64 / 128 / 256 / 512: 1 token, two of 32 experts of 1024 x 4096, 4-bit 15.2 / 17.8 / 22.4 / 31.2; 16 tokens 31.5 / 30.7 / 30.5 / 34.6; 64 tokens 49.4 /
// 42.4 / 35.4 / 38.0; 80 tokens on 16 experts of 4096 x 16384, group scales 357 / 281 / 264 / 227.  Over 390 drawn sizes this rule is 2 %
// slower than the best width of each, at most 17 %.)
int decode_slice_width(int n_assign, int E, int F)
{
    const double blocks64 = decode_active_experts(n_assign, E) * (F / 64);
    int w = 1;
    for (int c = 2; c <= 8; c *= 2)
        if (F % (64 * c) == 0 && blocks64 / c >= 254) w = c;
    return w;
}

size_t decode_ffn_partial_bytes(int n_assign, int d, int F, int cw)
{
    return (size_t)(F / (64 * cw)) * n_assign * d * sizeof(float);
}

int launch_decode_ffn(const DecodeArgs &q, int bits, bool bf, hipStream_t s)
{
    DecodeArgs p = q;
    const uint32_t units = p.g ? p.g / 64 : 1;
    // two sixteens of rows per item where experts are expected to have more than eight, 4-bit codes: with fewer the second
    // sixteen's products are idle, with wider codes it takes the registers that loads in flight need
    p.row_tiles = p.n_assign > 8 * p.E && bits == 4 ? 2 : 1;
    p.group_inv = units > 1 ? (uint32_t)(((1ull << 32) + units - 1) / units) : 0;
    const int S = p.F / (64 * p.cw);
    // the most items that a routing can make: one per expert with rows, one more for every further `fit` rows (the first block writes the index arrays)
    const int fit = kDecFit * p.row_tiles, items = p.n_assign <= p.E ? p.n_assign : p.E + (p.n_assign - p.E) / fit;
    const dim3 grid(1 + (unsigned)items * S);
    if (bits == 4) launch_decode_bits<4>(p, bf, grid, s);
    else launch_decode_bits<8>(p, bf, grid, s);
    int rc = check_launch("moe_grouped_ffn_wq (decode kernel)");
    if (rc || !p.out) return rc;                // (no output buffer: the partial sums are all the caller wants)
    const bool codes = bf && !p.g;
    if (S > 32) launch_reduce<16, 4>(p, codes, s);
    else if (S > 8) launch_reduce<8, 4>(p, codes, s);
    else launch_reduce<4, 2>(p, codes, s);
    return check_launch("moe_grouped_ffn_wq (slice reduction)");
}

}  // namespace moe
