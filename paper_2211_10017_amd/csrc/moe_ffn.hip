// moe_grouped_ffn_wq: grouped expert GEMM pair with weight-only int4/int8 experts
// (Sec. 3.3 grouped GEMM, Sec. 3.4 fused dequantisation).  This file holds the entry point:
// argument checks, workspace layout and the choice between the weight-streaming kernel
// (experts with few rows, HBM-bound) and the LDS-tiled kernel (experts with many rows,
// MFMA-bound).
#include <mutex>

#include "moe_ffn_common.h"

namespace moe {

// bf16 rows -> FP16 rows scaled by a power of two per row: pow.x = 2^-p brings the row's largest magnitude
// into [2^14, 2^15), so that every element converts to FP16 without overflow; the GEMM takes the result like
// FP16 rows (straight from memory into LDS) and multiplies its output rows by pow.y = 2^p.  A value keeps its 8-bit significand unless it is more than 2^-28 below the row's largest, where FP16
// runs out of exponent.  `out` may be `in`: a lane reads what it converts before it writes it, and the row's
// largest magnitude is known before the first write.
//
// LANES lanes share a row (a wavefront, or a block of 256 for long rows) and hold it in registers, NV 16-byte vectors each,
// between the search for its largest magnitude and the conversion: a row is read once.  (Read twice, with a wavefront per
// row, the rows in flight on the chip were many times its L2s and the second read went to memory again: h of 16384 rows of
// 16384, 262 us against 163.)  NV = 0: rows of any length, read twice.
template <int LANES, int NV>
__global__ __launch_bounds__(256) void rows_to_f16_kernel(const uint16_t *in, uint16_t *out, int R, int K, float2 *__restrict__ row_pow)
{
    __shared__ uint32_t s_max[4];
    const int i0 = threadIdx.x % LANES;
    const int r = blockIdx.x * (256 / LANES) + threadIdx.x / LANES;
    if (r >= R) return;                            // (with a row per block: the whole block)
    const uint4 *row = reinterpret_cast<const uint4 *>(in + (size_t)r * K);
    uint4 *dst = reinterpret_cast<uint4 *>(out + (size_t)r * K);
    uint32_t amax = 0;
    auto largest = [&](const uint4 q) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            amax = max(amax, w[i] & 0x7fffu);
            amax = max(amax, (w[i] >> 16) & 0x7fffu);
        }
    };
    uint4 v[NV ? NV : 1];
    if constexpr (NV > 0) {
#pragma unroll
        for (int j = 0; j < NV; ++j) v[j] = i0 + j * LANES < K / 8 ? row[i0 + j * LANES] : make_uint4(0, 0, 0, 0);
#pragma unroll
        for (int j = 0; j < NV; ++j) largest(v[j]);
    } else {
        for (int i = i0; i < K / 8; i += LANES) largest(row[i]);
    }
    for (int off = 32; off > 0; off >>= 1) amax = max(amax, (uint32_t)__shfl_xor((int)amax, off));
    if constexpr (LANES > 64) {
        if ((threadIdx.x & 63) == 0) s_max[threadIdx.x >> 6] = amax;
        __syncthreads();
        amax = max(max(s_max[0], s_max[1]), max(s_max[2], s_max[3]));
    }
    int ex = (int)(amax >> 7);                     // biased exponent of the largest magnitude
    if (ex == 255) ex = 141;                       // inf/nan rows: factor 1 (the result is nan anyway)
    int fe = 268 - ex;                             // biased exponent of 2^(14 - (ex - 127))
    fe = min(max(fe, 1), 253);
    const float down = __uint_as_float((uint32_t)fe << 23);
    if (i0 == 0) row_pow[r] = make_float2(down, __uint_as_float((uint32_t)(254 - fe) << 23));
    auto convert = [&](const uint4 q) {
        const uint32_t w[4] = {q.x, q.y, q.z, q.w};
        uint32_t o[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const half2_t h = {(_Float16)(__uint_as_float(w[i] << 16) * down), (_Float16)(__uint_as_float(w[i] & 0xffff0000u) * down)};
            o[i] = h2_bits(h);
        }
        return make_uint4(o[0], o[1], o[2], o[3]);
    };
    if constexpr (NV > 0) {
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (i0 + j * LANES < K / 8) dst[i0 + j * LANES] = convert(v[j]);
    } else {
        for (int i = i0; i < K / 8; i += LANES) dst[i] = convert(row[i]);
    }
}

static int rows_to_f16(const uint16_t *in, uint16_t *out, int R, int K, float2 *row_pow, hipStream_t s)
{
    if (K <= 64 * 8 * 2) hipLaunchKernelGGL((rows_to_f16_kernel<64, 2>), dim3((R + 3) / 4), dim3(256), 0, s, in, out, R, K, row_pow);
    else if (K <= 64 * 8 * 8) hipLaunchKernelGGL((rows_to_f16_kernel<64, 8>), dim3((R + 3) / 4), dim3(256), 0, s, in, out, R, K, row_pow);
    else if (K <= 256 * 8 * 8) hipLaunchKernelGGL((rows_to_f16_kernel<256, 8>), dim3(R), dim3(256), 0, s, in, out, R, K, row_pow);
    else hipLaunchKernelGGL((rows_to_f16_kernel<64, 0>), dim3((R + 3) / 4), dim3(256), 0, s, in, out, R, K, row_pow);
    return check_launch("moe_grouped_ffn_wq (bf16 rows to scaled FP16)");
}

// Sizes for which the gated call runs the decode kernel instead of two streaming launches: the ones it was measured to be the faster way
// for in this call (one K range per weight width; other sizes have moe_grouped_ffn_wq_sliced, which takes any).
static bool gated_decode(int R, int E, int d, int F, int bits)
{
    if (R < 1 || R > kGatedMaxAssign || E < 1 || E > kDecMaxExperts) return false;
    if (d != (bits == 4 ? 1024 : 512) || F % 512 || F / 512 > 8 || F < 512) return false;
    return (long)R <= 8L * E && (long)E * (F / 512) >= 64;
}

struct FfnWorkspace {
    size_t h_off, pow_x_off, pow_h_off, x16_off;
    size_t own;             // what the two GEMMs need
    size_t total;           // with the decode kernel's partial sums of y, which that kernel keeps at the start of the workspace
};

static FfnWorkspace ffn_workspace(int R, int E, int d, int F, int act_dtype)
{
    FfnWorkspace w;
    size_t o = 0;
    w.h_off = o;
    o += round_up((size_t)R * F * 2, 256);
    w.pow_x_off = o;
    if (act_dtype == MOE_BF16) o += round_up((size_t)R * sizeof(float2), 256);
    w.pow_h_off = o;
    if (act_dtype == MOE_BF16) o += round_up((size_t)R * sizeof(float2), 256);
    w.x16_off = o;                               // bf16 rows: x converted to scaled FP16 (h is converted in place)
    if (act_dtype == MOE_BF16) o += round_up((size_t)R * d * 2, 256);
    w.own = w.total = o < 256 ? 256 : o;
    if (gated_decode(R, E, d, F, 4) || gated_decode(R, E, d, F, 8)) w.total += round_up(decode_ffn_partial_bytes(R, d, F, decode_slice_width(R, E, F)), 256);
    return w;
}

}  // namespace moe

extern "C" size_t moe_grouped_ffn_wq_workspace_bytes(int R, int d, int F, int E, int act_dtype)
{
    if (R <= 0 || d <= 0 || F <= 0) return 256;
    return moe::ffn_workspace(R, E, d, F, act_dtype).total;
}

// Which kernel can take one GEMM of the FFN, from what the host knows about the routed loads: an upper bound on the rows of any
// expert and the mean rows per expert.  The gated call and the answers of the _supported queries follow this rule; a GEMM of
// permuted rows runs in the streaming kernel it names only where that is the faster one as well (stream_pays).
enum GemmKernel { GEMM_TILED, GEMM_STREAM_UNROLLED, GEMM_STREAM_LOOP };

static GemmKernel choose_kernel(int R, int E, int max_rows, int K, int N, int bits, int smode, bool bf)
{
    using namespace moe;
    if (bf || !stream_gemm_supports(K, bits, smode)) return GEMM_TILED;
    const int mean = (R + E - 1) / E;
    const bool unrolled = stream_unrolled_supports(K, bits, smode);
    // rows of an expert one block of the streaming kernel holds; an expert with more rows takes further
    // blocks (row groups), each of which streams the expert's weights again
    const int fit = unrolled ? stream_unrolled_fit(K, max_rows) : stream_gemm_fit_rows(K);
    // Streaming takes a row bound that needs few row groups: at most 64 rows, or at most 32 rows per
    // expert on average and at most sixteen groups ...
    const bool few = unrolled && mean <= 32 && max_rows <= 16 * fit;
    if (!(max_rows <= 64 || few)) return GEMM_TILED;
    // ... and, further, that the typical expert is one row group, the batch is decode-sized, or row tiles would leave most
    // of the chip idle (one tile per expert and column block).
    const long tiles = (long)(E < R ? E : R) * ((N + 255) / 256);
    if (R <= 256 || mean <= fit || tiles < 128) return unrolled ? GEMM_STREAM_UNROLLED : GEMM_STREAM_LOOP;
    return GEMM_TILED;
}

// Whether one of the streaming kernels is the faster one for a GEMM that choose_kernel gives it, rows permuted beforehand.  A
// streaming block takes one row group of an expert (`fit` rows) and one or two slabs of 32 channels and has its whole ring in flight
// from the start; further row groups of the expert stream its weights again.  Row tiles read them once, but a launch of few
// tiles waits for its chain of K steps.  So streaming pays
//  - while all slabs of all row groups run at once, about 1280 of 4-bit or 1200 of 8-bit weights: 40 rows on 8 experts of
//    1024 x 4096, 4-bit, 16.0 us a pair of GEMMs against 25.0 in row tiles, 256 rows 39 against 29; in the run-loop kernel 1300 of 4-bit
//    or 650 of 8-bit weights, from N = 2048 on (32 experts of 1024 x 4096, 8-bit, 64 rows: its fc2 takes 5 us longer than row tiles),
//  - for few tiles (64 rows on one expert of 2048 x 8192, 8-bit: 45 against 61 us, of 512 x 2048 11 against 22; on four of 2048 x 8192
//    70 against 47, which the lines above leave to row tiles),
//  - for experts of mostly well under one row group, 8-bit, or 4-bit with many tiles (200 rows on 128 experts of 1024 x 1024: 43
//    against 54, 33 against 40).
// (8681 GEMMs of such calls, even and skewed loads: row tiles for every R > E cost up to 88 % of a call, streaming wherever
// choose_kernel allows it up to 68 %; this rule up to 13 %, or 28 % where the load is skewed, which it does not see.)
static bool stream_pays(int R, int E, int K, int N, int bits, bool unrolled)
{
    using namespace moe;
    if (R <= E) return true;
    const long experts = E < R ? E : R, tiles = experts * ((N + 255) / 256);
    const int fit = unrolled ? stream_unrolled_fit(K, R) : stream_gemm_fit_rows(K);
    const long slabs = (experts + R / fit) * (N / 32);
    if (unrolled) return slabs <= (bits == 4 ? 1280 : 1200) || tiles <= 40 || (8L * R <= 5L * fit * E && (bits == 8 || tiles > 448));
    return (slabs * bits <= 4 * 1300 && N >= 2048) || (tiles <= 28 && R > 32L * E && R <= 16L * fit * E);
}

// The kernel of one GEMM whose rows come permuted.
static GemmKernel four_call_kernel(int R, int E, int max_rows, int K, int N, int bits, int smode, bool bf)
{
    const GemmKernel kernel = choose_kernel(R, E, max_rows, K, N, bits, smode, bf);
    return kernel == GEMM_TILED || stream_pays(R, E, K, N, bits, kernel == GEMM_STREAM_UNROLLED) ? kernel : GEMM_TILED;
}

// bf: the rows were bf16 (they come in as they are, smode SCALE_CHANNEL_BF16, or converted to scaled FP16, with their factors in
// g.row_pow; only the row tiles take either)
// tiles_only: rows go through the routing index, which only the row tiles do
static int run_gemm(moe::GemmArgs g, int bits, int smode, bool bf, bool tiles_only, int max_rows, hipStream_t s)
{
    using namespace moe;
    // (the permutation inside the launch and the added rows of the gated call are built for the straight-line kernel only)
    const GemmKernel kernel = tiles_only                ? GEMM_TILED
                              : g.gate_idx || g.out_add ? choose_kernel(g.R, g.E, max_rows, g.K, g.N, bits, smode, bf)
                                                        : four_call_kernel(g.R, g.E, max_rows, g.K, g.N, bits, smode, bf);
    if (kernel != GEMM_TILED) note_kernel(kernel == GEMM_STREAM_UNROLLED ? "stream_unrolled_kernel" : "stream_gemm_kernel");
    if (kernel == GEMM_STREAM_UNROLLED) return launch_stream_unrolled(g, bits, max_rows, s);
    if (!tiles_only && (g.gate_idx || g.out_add)) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_gated: K=%d does not run in the straight-line kernel with these sizes", g.K);
    if (kernel == GEMM_STREAM_LOOP) return launch_stream_gemm(g, bits, smode, max_rows, s);
    // Everything else runs in row tiles, experts with a handful of rows included: their tiles skip
    // the row blocks that hold no rows and stream the weights as fast as the streaming kernel would
    // (sending them there in a launch of their own measured 2-25 % slower on skewed loads).
    return launch_tiled_gemm(g, bits, smode, s);
}

// true when a call with these sizes runs both GEMMs in the tiled kernel (the only kernel that takes
// rows through the routing index)
static bool tiled_only(int R, int E, int max_rows, int d, int F, int bits, bool grouped, bool bf)
{
    using namespace moe;
    const int smode = grouped ? SCALE_GROUP : SCALE_CHANNEL;
    return choose_kernel(R, E, max_rows, d, F, bits, smode, bf) == GEMM_TILED &&
           choose_kernel(R, E, max_rows, F, d, bits, smode, bf) == GEMM_TILED;
}

// How fc1's weights meet group scales.  bf16 rows, groups of 128: exact codes, group sums folded in fp32; other group sizes: the two-term form, in the LDS ring exact
// codes as well.
static int fc1_group_mode(bool bf, int group_size)
{
    return !bf ? moe::SCALE_GROUP : group_size == 128 ? moe::SCALE_GROUP_ACC : moe::SCALE_GROUP_SPLIT;
}

static int ffn_impl(const void *x_perm, int act_dtype, const int32_t *expert_offsets, int R,
                    int E, int max_rows_per_expert, int d, int F, int bits, int group_size, int activation,
                    const void *w1_packed,
                    const void *s1, const void *b1, const void *w2_packed, const void *s2,
                    const void *b2, void *y_perm, int y_dtype, void *workspace,
                    size_t workspace_bytes, void *stream,
                    const int32_t *perm_src, int k, const float *expert_scale,
                    const int32_t *gate_idx = nullptr, int32_t *perm_src_out = nullptr, int32_t *inv_perm_out = nullptr,
                    int32_t *offsets_out = nullptr, bool unsorted = false, bool stream_fc1 = false)
{
    using namespace moe;
    // decode-sized batch with everything fused: one streaming launch for the sort and both GEMMs, then the slice reduction
    const bool decode = gate_idx && !unsorted && expert_scale && act_dtype == MOE_F16 && group_size == 0 && gated_decode(R, E, d, F, bits);
    const bool partial_only = !y_perm && decode;        // (on that path NULL means "leave out the slice reduction")
    if (!expert_offsets || !w1_packed || !s1 || !w2_packed || !s2 || (R != 0 && (!x_perm || (!y_perm && !partial_only))))
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq: NULL pointer");
    if (R < 0 || E <= 0 || d <= 0 || F <= 0 || max_rows_per_expert < 0)
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq: R >= 0, max_rows_per_expert >= 0 and E, d, F > 0 required");
    if (d % 64 || F % 64) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq: d and F must be multiples of 64 (d=%d F=%d)", d, F);
    if (bits != 4 && bits != 8) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq: bits must be 4 or 8 (got %d)", bits);
    if (activation != MOE_ACT_RELU && activation != MOE_ACT_GELU) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq: unknown activation %d", activation);
    if (act_dtype != MOE_F16 && act_dtype != MOE_BF16) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq: act_dtype must be fp16 or bf16");
    if (y_dtype != MOE_F16 && y_dtype != MOE_BF16 && y_dtype != MOE_F32) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq: unknown y_dtype %d", y_dtype);
    if (group_size < 0 || (group_size && (group_size % 64 || d % group_size || F % group_size)))
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq: group_size %d must be 0 or a multiple of 64 dividing d and F", group_size);
    if (E > 4096) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq: E=%d above 4096", E);
    const void *ptrs[] = {x_perm, w1_packed, s1, b1, w2_packed, s2, b2, y_perm, workspace};
    for (const void *q : ptrs)
        if (!aligned16(q)) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq: buffers must be 16-byte aligned");
    const FfnWorkspace ws = ffn_workspace(R, E, d, F, act_dtype);
    const size_t least = decode ? decode_ffn_partial_bytes(R, d, F, 8) : ws.own;
    if (!workspace || workspace_bytes < least)
        return fail(MOE_ERR_WORKSPACE, "moe_grouped_ffn_wq: workspace of %zu bytes needed, %zu given", least, workspace_bytes);
    reset_kernel_notes();
    if (R == 0) return MOE_OK;

    hipStream_t s = as_stream(stream);
    const bool bf = act_dtype == MOE_BF16;
    const int max_rows = max_rows_per_expert > 0 && max_rows_per_expert < R ? max_rows_per_expert : R;
    unsigned char *wsb = (unsigned char *)workspace;
    void *h = wsb + ws.h_off;
    if (decode) {
        // (a workspace asked for with more rows may hold fewer slices than this batch would take: they are then wider)
        int cw = decode_slice_width(R, E, F);
        while (cw < 8 && decode_ffn_partial_bytes(R, d, F, cw) > workspace_bytes) cw *= 2;
        DecodeArgs q{};
        q.x = (const uint16_t *)x_perm; q.gate_idx = gate_idx; q.gate_scale = expert_scale; q.n_assign = R; q.gate_k = k;
        q.E = E; q.d = d; q.F = F; q.act = activation;
        q.w1 = (const uint8_t *)w1_packed; q.w2 = (const uint8_t *)w2_packed;
        q.s1 = (const __half *)s1; q.s2 = (const __half *)s2; q.b1 = (const __half *)b1; q.b2 = (const __half *)b2;
        q.cw = cw; q.partial = (float *)wsb; q.out = y_perm; q.out_dtype = MOE_F32;
        q.perm_src_out = perm_src_out; q.inv_perm_out = inv_perm_out; q.offsets_out = offsets_out;
        note_kernel("decode_ffn_kernel");
        return launch_decode_ffn(q, bits, false, s);
    }
    float2 *pow_x = (float2 *)(wsb + ws.pow_x_off), *pow_h = (float2 *)(wsb + ws.pow_h_off);
    const bool grouped = group_size != 0 && !(group_size == d && group_size == F);

    // fc1: h = relu(x_perm @ deq(W1) + b1), stored in the activation dtype.  With bf16
    // activations and group scales the weights go in as an exact two-term FP16 sum, because h
    // is rounded to 8 bits afterwards and a 2^-11 weight rounding would show through.
    GemmArgs g1{};
    const bool tiles_only = perm_src || unsorted;
    const int tokens = tiles_only ? R / k : R;                  // rows of x
    const bool convert = bf && (grouped || !bf16_codes_pay(R, tokens, E, d, F, bits, tiles_only));
    g1.a = (const uint16_t *)x_perm; g1.row_pow = convert ? pow_x : nullptr; g1.offsets = expert_offsets;
    g1.wq = (const uint8_t *)w1_packed; g1.scales = (const __half *)s1; g1.bias = (const __half *)b1;
    g1.out = h; g1.E = E; g1.R = R; g1.K = d; g1.N = F; g1.g = grouped ? group_size : d;
    g1.out_dtype = act_dtype; g1.act = activation;
    g1.a_src = perm_src; g1.a_div = k; g1.indexed = tiles_only;
    if (gate_idx) {     // decode-sized: fc1 rebuilds the permutation from the gate's output and writes the index arrays
        g1.gate_idx = gate_idx; g1.n_assign = R; g1.gate_k = k;
        g1.perm_src_out = perm_src_out; g1.inv_perm_out = inv_perm_out; g1.offsets_out = offsets_out;
        if (expert_scale && !unsorted) { g1.zero_out = (float *)y_perm; g1.zero_count = (long)(R / k) * d; }   // fc2 adds into it
    }
    if (convert) {      // bf16 rows of group-scaled or large layers: converted to power-of-two scaled FP16 rows first, then the GEMM of FP16 rows
        uint16_t *x16 = (uint16_t *)(wsb + ws.x16_off);
        // (through the routing index: every token's row once, R / k of them)
        int rc = rows_to_f16((const uint16_t *)x_perm, x16, tokens, d, pow_x, s);
        if (rc) return rc;
        g1.a = x16;
    }
    const int channel = bf && !convert ? SCALE_CHANNEL_BF16 : SCALE_CHANNEL, smode1 = grouped ? fc1_group_mode(bf, group_size) : channel;
    int rc = run_gemm(g1, bits, smode1, bf, tiles_only && !stream_fc1, max_rows, s);
    if (rc) return rc;

    // fc2: y = h @ deq(W2) + b2
    GemmArgs g2 = g1;
    g2.a = (const uint16_t *)h; g2.row_pow = convert ? pow_h : nullptr;
    g2.wq = (const uint8_t *)w2_packed; g2.scales = (const __half *)s2; g2.bias = (const __half *)b2;
    g2.out = y_perm; g2.K = F; g2.N = d; g2.g = grouped ? group_size : F;
    g2.out_dtype = y_dtype; g2.act = MOE_ACT_NONE;
    g2.a_src = nullptr;
    g2.gate_idx = nullptr; g2.zero_out = nullptr;
    if (gate_idx && expert_scale && !unsorted) {     // un-permute fused into fc2: fc1 clears out, fc2 adds scale * y into the tokens' rows
        g2.out_dst = perm_src_out; g2.out_scale = expert_scale; g2.out_add = 1; g2.out_div = k;
    } else if (expert_scale) {
        g2.out_dst = unsorted ? perm_src_out : perm_src; g2.out_scale = expert_scale;
    }
    if (convert) {      // h, which fc1 rounded to bf16 (A13), in place
        rc = rows_to_f16((const uint16_t *)h, (uint16_t *)h, R, F, pow_h, s);
        if (rc) return rc;
    }
    return run_gemm(g2, bits, grouped ? SCALE_GROUP : channel, bf, tiles_only, max_rows, s);
}

extern "C" int moe_grouped_ffn_wq(const void *x_perm, int act_dtype, const int32_t *expert_offsets, int R,
                                  int E, int max_rows_per_expert, int d, int F, int bits, int group_size,
                                  int activation, const void *w1_packed,
                                  const void *s1, const void *b1, const void *w2_packed, const void *s2,
                                  const void *b2, void *y_perm, int y_dtype, void *workspace,
                                  size_t workspace_bytes, void *stream)
{
    return ffn_impl(x_perm, act_dtype, expert_offsets, R, E, max_rows_per_expert, d, F, bits, group_size, activation, w1_packed,
                    s1, b1, w2_packed, s2, b2, y_perm, y_dtype, workspace, workspace_bytes, stream, nullptr, 1, nullptr);
}

// ---- the entry point for callers that cannot allocate ------------------------------------------
// moe_grouped_ffn_wq with its workspace (h, and for bf16 rows the per-row factors) in a fixed array in
// the library's own device memory.  Every GPU the library runs on holds its own copy of the array
// until the process ends.
constexpr size_t kScratchBytes = (size_t)8 << 20;
constexpr int kScratchMaxDevices = 64;
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// Device address of `scratch` on the current device, looked up once per device (0 on failure, with
// the error message set).  In host code the array's name is only a handle for this lookup.
static void *scratch_address()
{
    using namespace moe;
    static std::mutex lock;
    static void *address[kScratchMaxDevices];           // zero-initialised: not looked up yet
    int dev = -1;
    hipError_t err = hipGetDevice(&dev);
    if (err != hipSuccess || dev < 0 || dev >= kScratchMaxDevices) {
        fail(MOE_ERR_HIP, "moe_grouped_ffn_wq_noalloc: no current device (%s)", hipGetErrorString(err));
        return nullptr;
    }
    std::lock_guard<std::mutex> guard(lock);
    if (!address[dev]) {
        void *ptr = nullptr;
        err = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (err != hipSuccess || !ptr) {
            fail(MOE_ERR_HIP, "moe_grouped_ffn_wq_noalloc: hipGetSymbolAddress failed on device %d (%s)", dev, hipGetErrorString(err));
            return nullptr;
        }
        address[dev] = ptr;
    }
    return address[dev];
}

extern "C" size_t moe_grouped_ffn_wq_noalloc_max_bytes(void) { return kScratchBytes; }

extern "C" int moe_grouped_ffn_wq_noalloc(const void *x_perm, int act_dtype, const int32_t *expert_offsets, int R,
                                          int E, int max_rows_per_expert, int d, int F, int bits, int group_size,
                                          int activation, const void *w1_packed,
                                          const void *s1, const void *b1, const void *w2_packed, const void *s2,
                                          const void *b2, void *y_perm, int y_dtype, void *stream)
{
    using namespace moe;
    if (R > 0 && d > 0 && F > 0) {
        const size_t need = ffn_workspace(R, E, d, F, act_dtype).own;
        if (need > kScratchBytes)
            return fail(MOE_ERR_WORKSPACE, "moe_grouped_ffn_wq_noalloc: R=%d rows of F=%d need %zu bytes of scratch, the built-in "
                                           "array holds %zu: use moe_grouped_ffn_wq with a workspace", R, F, need, kScratchBytes);
    }
    void *ws = scratch_address();
    if (!ws) return MOE_ERR_HIP;
    return ffn_impl(x_perm, act_dtype, expert_offsets, R, E, max_rows_per_expert, d, F, bits, group_size, activation, w1_packed,
                    s1, b1, w2_packed, s2, b2, y_perm, y_dtype, ws, kScratchBytes, stream, nullptr, 1, nullptr);
}

// The same pair of GEMMs with the row gather (and, for k = 1, the un-permute and gate scale) fused
// into them; built on the tiled kernel only.
extern "C" int moe_grouped_ffn_wq_routed_supported(int R, int E, int max_rows_per_expert, int d, int F,
                                                   int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (R <= 0 || E <= 0 || d <= 0 || F <= 0 || act_dtype != MOE_F16) return 0;
    const int max_rows = max_rows_per_expert > 0 && max_rows_per_expert < R ? max_rows_per_expert : R;
    const bool grouped = group_size != 0 && !(group_size == d && group_size == F);
    return tiled_only(R, E, max_rows, d, F, bits, grouped, false) ? 1 : 0;
}

extern "C" int moe_grouped_ffn_wq_routed(const void *x, int act_dtype, const int32_t *perm_src, int k,
                                         const float *expert_scale, const int32_t *expert_offsets, int R,
                                         int E, int max_rows_per_expert, int d, int F, int bits,
                                         int group_size, int activation, const void *w1_packed, const void *s1,
                                         const void *b1, const void *w2_packed, const void *s2,
                                         const void *b2, void *out, int out_dtype, void *workspace,
                                         size_t workspace_bytes, void *stream)
{
    using namespace moe;
    if (!perm_src) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_routed: perm_src must not be NULL");
    if (k < 1 || k > 2) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_routed: k must be 1 or 2 (k=%d)", k);
    if (expert_scale && k != 1)
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_routed: the fused un-permute needs k = 1 (one expert per token)");
    if (!moe_grouped_ffn_wq_routed_supported(R, E, max_rows_per_expert, d, F, bits, group_size, act_dtype))
        return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_routed: only fp16 batches too large for the streaming kernels are taken: use "
                                         "moe_grouped_ffn_wq_indexed, or moe_permute + moe_grouped_ffn_wq + moe_combine");
    return ffn_impl(x, act_dtype, expert_offsets, R, E, max_rows_per_expert, d, F, bits, group_size, activation, w1_packed, s1, b1,
                    w2_packed, s2, b2, out, out_dtype, workspace, workspace_bytes, stream, perm_src, k, expert_scale);
}

// The routed call for every size and both row types: both GEMMs run in row tiles.
extern "C" int moe_grouped_ffn_wq_indexed(const void *x, int act_dtype, const int32_t *perm_src, int k,
                                          const float *expert_scale, const int32_t *expert_offsets, int R,
                                          int E, int max_rows_per_expert, int d, int F, int bits,
                                          int group_size, int activation, const void *w1_packed, const void *s1,
                                          const void *b1, const void *w2_packed, const void *s2,
                                          const void *b2, void *out, int out_dtype, void *workspace,
                                          size_t workspace_bytes, void *stream)
{
    using namespace moe;
    if (!perm_src) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_indexed: perm_src must not be NULL");
    if (k < 1 || k > 2 || R % k) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_indexed: k must be 1 or 2 and divide R (k=%d, R=%d)", k, R);
    if (expert_scale && k != 1)
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_indexed: the fused un-permute needs k = 1 (one expert per token)");
    return ffn_impl(x, act_dtype, expert_offsets, R, E, max_rows_per_expert, d, F, bits, group_size, activation, w1_packed, s1, b1,
                    w2_packed, s2, b2, out, out_dtype, workspace, workspace_bytes, stream, perm_src, k, expert_scale);
}

// Decode-sized batches: moe_permute and moe_grouped_ffn_wq in one call.  fc1 runs in the straight-line
// streaming kernel, whose blocks rebuild the permutation from the gate's expert indices, fetch their
// rows from the tokens and write perm_src / inv_perm / expert_offsets on the way; fc2 and moe_combine
// then read those arrays as after moe_permute.
static int gated_shapes(int T, int k, int E, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (T <= 0 || k < 1 || k > 2 || E <= 0 || d <= 0 || F <= 0 || act_dtype != MOE_F16) return 0;
    if ((long)T * k > kGatedMaxAssign || (bits != 4 && bits != 8) || d % 64 || F % 64) return 0;
    if (group_size != 0 && !(group_size == d && group_size == F)) return 0;
    if (!stream_unrolled_takes_gate(d, bits)) return 0;
    // fc1 must run in the straight-line streaming kernel (row bound T) ...
    const int R = T * k;
    if (choose_kernel(R, E, T, d, F, bits, SCALE_CHANNEL, false) != GEMM_STREAM_UNROLLED) return 0;
    // ... and fc2 as well, if it is to add its rows straight into the layer output
    const bool fc2 = choose_kernel(R, E, T, F, d, bits, SCALE_CHANNEL, false) == GEMM_STREAM_UNROLLED;
    return fc2 ? 2 : 1;
}

// Whether a layer should take the gated call where it is supported: yes for the decode kernel; with the streaming kernels
// while a weight matrix's active experts are small enough for the saved launch to count (16.8 MB, 256 rows of 512 x 2048:
// 20 us against 25 in permute + row tiles; 134 MB, 64 rows on 32 experts of 1024 x 4096 8-bit: 64 and 68), or for at most
// one row per expert on average (16 tokens on 32 experts of 2048 x 8192 8-bit: 142 and 151), two with 8-bit weights and two experts
// per token (128 rows on 64 experts of 1024 x 4096 93 and 100, 192 on 128 of 1024 x 2048 88 and 106); otherwise the row tiles
// stream faster (64 tokens, 2048 x 8192: 4-bit 146 and 115, 8-bit 228 and 190).
extern "C" int moe_grouped_ffn_wq_gated_pays(int T, int k, int E, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (!gated_shapes(T, k, E, d, F, bits, group_size, act_dtype)) return 0;
    const int R = T * k;
    return gated_decode(R, E, d, F, bits) || R <= E || (bits == 8 && k == 2 && R <= 2 * E) || (double)E * d * F * bits / 8 <= 150e6;
}

// moe_permute's index and moe_grouped_ffn_wq_indexed in one call: fc1's row tiles sort for themselves (find_unsorted_item).
extern "C" int moe_grouped_ffn_wq_unsorted_supported(int T, int k, int E, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (T <= 0 || k < 1 || k > 2 || E <= 0 || E > kUnsortedMaxExperts || (long)T * k > kUnsortedMaxAssign || d <= 0 || F <= 0 || d % 64 || F % 64) return 0;
    if ((bits != 4 && bits != 8) || group_size < 0 || (group_size && (group_size % 64 || d % group_size || F % group_size))) return 0;
    return act_dtype == MOE_F16 || act_dtype == MOE_BF16;
}

// ... or, for the batches whose fc1 the gated call would run in the streaming kernel and whose fc2 runs in row tiles, that kernel, which sorts for itself as well.
static bool unsorted_streams(int T, int k, int E, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    return gated_shapes(T, k, E, d, F, bits, group_size, act_dtype) == 1 && moe_grouped_ffn_wq_gated_pays(T, k, E, d, F, bits, group_size, act_dtype) &&
           four_call_kernel(T * k, E, T, F, d, bits, SCALE_CHANNEL, false) == GEMM_TILED;
}

// Whether a layer that takes the indexed call should take this one: the launch that it saves is 2 to 3.5 us, and every round of fc1's blocks pays for
// sorting, the more the more assignments there are.  us a step, with the index in a launch / in fc1, by fc1's blocks per compute unit: 62 tokens, one of 8 experts of 512 x
// 2048 8-bit (0.5) 30.6 / 28.7; 683, two of 32 of 512 x 2048 (1.0) 35.4 / 32.3; 1270, two of 16 of 1024 x 4096 8-bit (3.0) 87.2 / 83.9; 1555, one of 8 of 2048 x 8192
// 8-bit (3.6) 158.1 / 158.6; few assignments, 31, two of 64 of 2048 x 8192 (5.5) 173.1 / 170.8; 107, two (7.5) 217.9 / 217.3; left out 1215, two of 64 of 2048 x 8192 (8)
// 292 / 295; 387, two of 128 of 1024 x 4096 8-bit (15.8) 207 / 212.
extern "C" int moe_grouped_ffn_wq_unsorted_pays(int T, int k, int E, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (!moe_grouped_ffn_wq_unsorted_supported(T, k, E, d, F, bits, group_size, act_dtype)) return 0;
    // one expert per token, fc1 streaming: fc2 stores the output, where the gated call leaves it to moe_combine (40 tokens, one of 32 experts of 1024 x 4096, 8-bit,
    // 45.0 / 43.1 us a step; 200, one of 8, 41.3 / 39.4)
    if (moe_grouped_ffn_wq_gated_pays(T, k, E, d, F, bits, group_size, act_dtype)) return k == 1 && unsorted_streams(T, k, E, d, F, bits, group_size, act_dtype);
    GemmArgs g{};
    g.R = T * k, g.E = E, g.K = d, g.N = F, g.indexed = 1;
    const bool grouped = group_size != 0 && !(group_size == d && group_size == F);
    return row_tile_blocks(g, bits, grouped ? fc1_group_mode(act_dtype == MOE_BF16, group_size) : SCALE_CHANNEL) <= 256 * (g.R <= 512 ? 8 : 3.5);
}

extern "C" int moe_grouped_ffn_wq_unsorted(const void *x, int act_dtype, const int32_t *expert_idx, const float *expert_scale, int T, int k, int E,
                                           int d, int F, int bits, int group_size, int activation, const void *w1_packed, const void *s1,
                                           const void *b1, const void *w2_packed, const void *s2, const void *b2, void *out, int out_dtype,
                                           int32_t *perm_src, int32_t *inv_perm, int32_t *expert_offsets, void *workspace,
                                           size_t workspace_bytes, void *stream)
{
    using namespace moe;
    if (!expert_idx || !perm_src || !inv_perm || !expert_offsets) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_unsorted: NULL pointer");
    if (!moe_grouped_ffn_wq_unsorted_supported(T, k, E, d, F, bits, group_size, act_dtype))
        return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_unsorted: only 1 to %d assignments of fp16 or bf16 rows to at most %d experts with k = 1 or 2, d and F "
                                         "multiples of 64, 4- or 8-bit weights and group sizes that are 0 or a multiple of 64 dividing d and F are taken",
                    kUnsortedMaxAssign, kUnsortedMaxExperts);
    if (expert_scale && k != 1) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_unsorted: the fused un-permute needs k = 1 (one expert per token)");
    return ffn_impl(x, act_dtype, expert_offsets, T * k, E, T, d, F, bits, group_size, activation, w1_packed, s1, b1, w2_packed, s2, b2, out, out_dtype,
                    workspace, workspace_bytes, stream, nullptr, k, expert_scale, expert_idx, perm_src, inv_perm, expert_offsets, true,
                    unsorted_streams(T, k, E, d, F, bits, group_size, act_dtype));
}

// Whether a layer should take the indexed call: for bf16 rows, which run in row tiles anyway, and for more rows than experts where
// fc2 runs in row tiles.  Where a streaming kernel is the better one for fc2, permuted copies cost less than row tiles there
// (48 tokens, two of two experts of 2048 x 2048, 8-bit: 29 against 43 us a step).
extern "C" int moe_grouped_ffn_wq_indexed_pays(int R, int E, int max_rows_per_expert, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (R <= 0 || E <= 0 || d <= 0 || F <= 0) return 0;
    if (act_dtype == MOE_BF16) return 1;
    const int max_rows = max_rows_per_expert > 0 && max_rows_per_expert < R ? max_rows_per_expert : R;
    const bool grouped = group_size != 0 && !(group_size == d && group_size == F);
    return R > E && four_call_kernel(R, E, max_rows, F, d, bits, grouped ? SCALE_GROUP : SCALE_CHANNEL, false) == GEMM_TILED;
}

// ---- decode-sized batches of every kind: index, both GEMMs and the un-permute in the decode kernel and its reduction ----
extern "C" size_t moe_grouped_ffn_wq_sliced_workspace_bytes(int T, int k, int E, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (T <= 0 || (act_dtype != MOE_F16 && act_dtype != MOE_BF16)) return 0;
    if ((long)T * k > kDecMaxAssign || !decode_ffn_supports(T * k, k, E, d, F, bits, group_size)) return 0;
    return round_up(decode_ffn_partial_bytes(T * k, d, F, decode_slice_width(T * k, E, F)), 256);
}

// Few experts or small ones, beyond what moe_grouped_ffn_wq_sliced_pays lists: the launches of the other routes, and in wide layers (d_ff of three times d and more) the
// long chain of fc2, are most of their step there, while nothing much is read twice: `over`, the items that a touched expert is expected to make (sixteen rows,
// thirty-two with 4-bit weights and more than eight rows per expert), may be 1.6, with more than 100 MB of weights 1.1, anything up to 17 MB; FP16 rows on 8-bit codes
// with channel scales, which stream well elsewhere, 1.25 and 1.1, and from 100 MB on only up to a row per expert and 430 MB.  Further, us a step, the best other route /
// sliced:
//  - few rows, as every row costs its partial sums: 200, of wide layers that move 10 to 100 MB 256; bf16 rows with group scales, which the other routes convert, 56 more
//    (141 on 16 experts of 768 x 3072, groups of 128, 31.6 / 24.4; 311, groups of 64, bf16, on 32 of 448 x 1792 32.1 / 23.6; left out 476 on 8 of 768 x 3072 35 / 47, 512 on one of 2048 x
//    2048 36.7 / 78.9, of 2048 x 8192 71 / 350);
//  - what moves, the items' weights and the partial sums out and back: wide layers 150 MB (149 on 8 of 1024 x 4096 32.0 / 27.3; left out 226 on 8 of 2048 x 8192 70 / 85), up
//    to a hundred rows 300 and up to forty 500 (23 on 7 of 3904 x 15616 129 / 107), bf16 rows with channel scales 150 and 300 (left out 32, two of 48 of 2048 x 8192 108 / 119); other
//    layers 35 (64 on 9 of 1024 x 1024, groups of 128, 22.3 / 16.5; left out 161 on 8 of 2048 x 1024 25.1 / 31.2), bf16 rows with group scales up to a hundred 100 (98 on 16 of
//    2048 x 1024 38.5 / 28.4); and 35 where the gated call has everything in its two launches (left out 86 on 5 of 1024 x 4096 25.1 / 28.5);
//  - beyond 35 MB, partial sums of at most twice the weights.
// Or at most two rows on each of experts of up to 5 MB (229 on 128 of 768 x 3072, 8-bit bf16, 97 / 77), and FP16 rows on 4-bit codes with channel scales of wide layers at up to
// 1.6 rows per expert, a hundred in all, and 1200 MB (22 on 16 of 4096 x 16384, 814 MB, 180 / 155).
// Slices of 64 channels up to 520 blocks, as far as these were measured.
// (7250 drawn sizes that the lines below leave, one to 256 experts, d_ff of d / 2 to 8 d, every form: this takes 4240 of them, a step 1.42 times as fast on average, 25 more than
// 3 % slower, the worst 0.90; of their steps with all rows on two experts or on a quarter of them 45 of 3400 more than 5 % slower, the worst 0.70.  Without the bounds on rows, what moves and partial
// sums 1370 were more than 3 % slower, up to five times.)
static bool sliced_small(int R, int E, int d, int F, int bits, bool grouped, bool f16, double active, double bytes, double partial, bool narrow, bool fused)
{
    using namespace moe;
    const double expert = 2.0 * d * F * bits / 8, over = R <= E ? 1.0 : expected_row_tiles(R, E, R > 8L * E && bits == 4 ? 32 : 16) / active;
    const bool eight = f16 && bits == 8 && !grouped, four = f16 && bits == 4 && !grouped, bf_groups = grouped && !f16, bf_channels = !grouped && !f16, wide = F >= 3 * d;
    if (narrow || (eight ? over > (bytes > 100e6 ? 1.1 : 1.25) || (bytes > 100e6 && (R > E || bytes > 430e6)) : bytes > 17e6 && over > (bytes > 100e6 ? 1.1 : 1.6))) return false;
    if (R <= 2L * E && expert <= 5e6 && bytes <= 600e6) return true;
    if (wide && four && 5L * R <= 8L * E && R <= 100) return bytes <= 1200e6;
    const double moved = over * bytes + 2 * partial;
    const double most = fused ? 35e6 : !wide ? (bf_groups && R <= 100 ? 100e6 : 35e6) : R <= 40 ? (bf_channels ? 300e6 : 500e6) : R <= 100 && !bf_channels ? 300e6 : 150e6;
    const int rows = 200 + (bf_groups ? 56 : 0) + (wide && moved > 10e6 && moved <= 100e6 ? 56 : 0);
    return R <= rows && moved <= most && (partial <= 2 * bytes || moved <= 35e6);
}

// Whether a layer should take the sliced call: sliced_small, and what these lines take (steps in us of the routes below against it, uniform routing; of 13898 drawn sizes of
// 4 to 512 assignments the lines by themselves take 9964, 1.40 times as fast on average; 263 of them, most with up to one row per expert, are 2 to 41 % slower):
//  - up to eight assignments per expert: a block takes sixteen rows, and experts with more stream their weights again (61 tokens, two of
//    eight experts of 4096 x 16384 8-bit 182 and 320; 5 per expert of 1024 x 4096 8-bit 57 and 61).
//    Rows on 4-bit codes, whose blocks then take thirty-two: up to sixteen, 150 MB of weights and a d_ff of twice d (192 tokens,
//    two of 32 experts of 1024 x 4096 48.1 and 43.1, bf16 52.9 and 50.5; 242 tokens, two of 32 of 2048 x 8192 122 and 138; 191 of 1536 x
//    2048 40.7 and 41.2; left out 144, two of 16 of 1024 x 4096, 40.0 and 33.9, bf16 44.3 and 38.2), with group scales twelve, 110 MB and four times d (71 tokens, two of 16 of
//    1024 x 4096 42.6 and 28.1, bf16 48.5 and 32.1; 96, two of 16 of 2048 x 4096 51.0 and 52.5; left out 154, two of 32 of 1024 x 4096, 53.7 and 45.9), but not where one and a
//    bit blocks per compute unit would keep some busy twice as long as others (250 tokens, two of 60 of 1536 x 1280, 300 blocks, 53.6 and 52.4);
//  - the partial sums of a slice, rows x d x 4 bytes, well below its weights, and no thousands of slices of 64 channels, where d_ff leaves no
//    wider ones: a block's start then costs more than its few weights (218 tokens on 115 of 256 x 5312, group scales, 8100 blocks, 58 and 97;
//    139 on 131 of 640 x 4544, 6100, 81 and 113; 178 on 80 of 384 x 3392, 3800, 40 and 45; 43 on 71 of 448 x 6720, 3400, 48 and 40);
//  - up to 300 MB of weights: beyond, the launch's fixed parts count little and the ring's loads into LDS keep more in flight (30 tokens
//    on 32 experts of 4096 x 16384 8-bit 398 and 388; 240 on 55 of 4096 x 4096 8-bit, 1.8 GB, 314 and 370);
//  - FP16 rows on 8-bit codes with channel scales, more rows than experts: not from 140 MB on where the routes below stream and rows are long
//    enough for that to go well (40 / 60 / 100 / 128 tokens, two of 32 of 1024 x 4096 55.0 / 55.2 / 58.4 / 62.8 and 54.2 / 55.5 / 65.9 / 72.6;
//    40, one of 32, 44.5 and 45.6; 120, two of 22 of 2048 x 1536 52 and 60; but 512 x 4096, 128, two of 64, 61 and 55), from 180 MB on not for the longest rows (64 tokens on 8 of 4096 x
//    4096 63 and 84), and fewer narrow slices (100 tokens, two of 67 of 512 x 2112, 2100 slices, 44 and 49).  Where row tiles run
//    below, sliced at any of these sizes (60 tokens, two of 32 of 1088 x 4096 72 and 56, of 960 x 4096 58 and 49; 160, two of 128 of 512 x 2048 62 and 52);
//  - FP16 rows with group scales, whose scales the ring multiplies into the weights, beyond 300 MB too (64 tokens, 64 experts of 4096 x 16384 755 and 703),
//    but experts of more than 30 MB only up to five rows each: there little is left to gain (256 tokens, two of 64 of 4096 x 8192 445 and 445, 192
//    442 and 431, 128 436 and 419; of 2048 x 8192 237 and 242) and crowded routing, whose blocks read an expert's weights for every sixteen rows, loses most (256 on two of
//    4096 x 8192 137 and 214, 192 130 and 188, 128 115 and 127, on eight 195 and 297, 160 and 221, 150 and 188, by a gate of graded popularity
//    391 and 420, 327 and 362, 258 and 288);
//  - wherever the gated call would run the decode kernel: it is the same one (128 tokens, two of 128 experts of 1024 x 4096, 460 MB, 104 in
//    either call; 60 on 8 21).
extern "C" int moe_grouped_ffn_wq_sliced_pays(int T, int k, int E, int d, int F, int bits, int group_size, int act_dtype)
{
    using namespace moe;
    if (!moe_grouped_ffn_wq_sliced_workspace_bytes(T, k, E, d, F, bits, group_size, act_dtype)) return 0;
    const int R = T * k;
    if (gated_shapes(T, k, E, d, F, bits, group_size, act_dtype) == 2 && group_size == 0 && gated_decode(R, E, d, F, bits)) return 1;
    const double active = decode_active_experts(R, E), bytes = active * 2 * d * F * bits / 8;
    const bool grouped = group_size != 0 && !(group_size == d && group_size == F), f16 = act_dtype == MOE_F16;
    const int cw = decode_slice_width(R, E, F);
    const double blocks = active * (F / 64) / cw;
    if (cw == 1 && blocks > 3600) return 0;
    const bool fused = moe_grouped_ffn_wq_gated_pays(T, k, E, d, F, bits, group_size, act_dtype) && gated_shapes(T, k, E, d, F, bits, group_size, act_dtype) == 2;
    if (sliced_small(R, E, d, F, bits, grouped, f16, active, bytes, (double)decode_ffn_partial_bytes(R, d, F, cw), cw == 1 && blocks > 520, fused)) return 1;
    if (5 * R > 4 * active * cw * bits) return 0;
    if (R > 8L * E) {
        const bool fits = grouped ? R <= 12L * E && F >= 4 * d && bytes <= 110e6 : R <= 16L * E && F >= 2 * d && bytes <= 150e6;
        return bits == 4 && fits && (blocks <= 260 || blocks > 400);
    }
    if (bits == 8 && f16 && !grouped && R > E) {
        const bool streams = moe_grouped_ffn_wq_gated_pays(T, k, E, d, F, bits, group_size, act_dtype) ||
                             !(moe_grouped_ffn_wq_routed_supported(R, E, T, d, F, bits, group_size, act_dtype) ||
                               moe_grouped_ffn_wq_indexed_pays(R, E, T, d, F, bits, group_size, act_dtype));
        if ((streams && d >= 1024 && bytes > 140e6) || (d >= 4096 && bytes > 180e6) || (cw == 1 && blocks > 1250)) return 0;
    }
    return bytes <= 300e6 || (grouped && f16 && (R <= 5L * E || (double)d * F * bits <= 120e6));
}

extern "C" int moe_grouped_ffn_wq_sliced(const void *x, int act_dtype, const int32_t *expert_idx, const float *expert_scale, int T, int k, int E,
                                         int d, int F, int bits, int group_size, int activation, const void *w1_packed, const void *s1,
                                         const void *b1, const void *w2_packed, const void *s2, const void *b2, void *out, int out_dtype,
                                         int32_t *perm_src, int32_t *inv_perm, int32_t *expert_offsets, void *workspace,
                                         size_t workspace_bytes, void *stream)
{
    using namespace moe;
    if (!expert_idx || !expert_scale || !perm_src || !inv_perm || !expert_offsets || !x || !w1_packed || !s1 || !w2_packed || !s2)
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_sliced: NULL pointer");
    if (activation != MOE_ACT_RELU && activation != MOE_ACT_GELU) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_sliced: unknown activation %d", activation);
    if (out_dtype != MOE_F16 && out_dtype != MOE_BF16 && out_dtype != MOE_F32) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_sliced: unknown out_dtype %d", out_dtype);
    const size_t need = moe_grouped_ffn_wq_sliced_workspace_bytes(T, k, E, d, F, bits, group_size, act_dtype);
    if (!need)
        return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_sliced: only batches of 1 to %d assignments with k = 1 or 2, d and F multiples of 64, 4- or 8-bit "
                                         "weights and group sizes that are 0 or a multiple of 64 dividing d and F are taken", kDecMaxAssign);
    const void *ptrs[] = {x, w1_packed, s1, b1, w2_packed, s2, b2, out, workspace};
    for (const void *q : ptrs)
        if (!aligned16(q)) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_sliced: buffers must be 16-byte aligned");
    if (!workspace || workspace_bytes < need)
        return fail(MOE_ERR_WORKSPACE, "moe_grouped_ffn_wq_sliced: workspace of %zu bytes needed, %zu given", need, workspace_bytes);
    reset_kernel_notes();
    DecodeArgs q{};
    q.x = (const uint16_t *)x; q.gate_idx = expert_idx; q.gate_scale = expert_scale; q.n_assign = T * k; q.gate_k = k;
    q.E = E; q.d = d; q.F = F; q.act = activation; q.cw = decode_slice_width(T * k, E, F);
    q.g = group_size == d && group_size == F ? 0 : group_size;
    q.w1 = (const uint8_t *)w1_packed; q.w2 = (const uint8_t *)w2_packed;
    q.s1 = (const __half *)s1; q.s2 = (const __half *)s2; q.b1 = (const __half *)b1; q.b2 = (const __half *)b2;
    q.partial = (float *)workspace; q.out = out; q.out_dtype = out_dtype;
    q.perm_src_out = perm_src; q.inv_perm_out = inv_perm; q.offsets_out = expert_offsets;
    note_kernel("decode_ffn_kernel");
    return launch_decode_ffn(q, bits, act_dtype == MOE_BF16, as_stream(stream));
}

extern "C" int moe_grouped_ffn_wq_gated_supported(int T, int k, int E, int d, int F, int bits, int group_size,
                                                  int act_dtype)
{
    return gated_shapes(T, k, E, d, F, bits, group_size, act_dtype);
}

extern "C" int moe_grouped_ffn_wq_gated(const void *x, int act_dtype, const int32_t *expert_idx,
                                        const float *expert_scale, int T, int k,
                                        int E, int d, int F, int bits, int group_size, int activation,
                                        const void *w1_packed, const void *s1, const void *b1,
                                        const void *w2_packed, const void *s2, const void *b2, void *y_perm,
                                        int y_dtype, int32_t *perm_src, int32_t *inv_perm,
                                        int32_t *expert_offsets, void *workspace, size_t workspace_bytes,
                                        void *stream)
{
    using namespace moe;
    if (!expert_idx || !perm_src || !inv_perm || !expert_offsets)
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_ffn_wq_gated: NULL pointer");
    const int level = gated_shapes(T, k, E, d, F, bits, group_size, act_dtype);
    if (!level)
        return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_gated: only decode-sized fp16 batches with per-channel scales "
                                         "(T*k <= %d) are taken: use moe_permute + moe_grouped_ffn_wq", kGatedMaxAssign);
    if (expert_scale && (level < 2 || y_dtype != MOE_F32))
        return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_ffn_wq_gated: the fused un-permute needs an fp32 output and an fc2 that runs "
                                         "in the straight-line streaming kernel: pass expert_scale = NULL and use moe_combine");
    return ffn_impl(x, act_dtype, expert_offsets, T * k, E, T, d, F, bits, group_size, activation, w1_packed, s1, b1,
                    w2_packed, s2, b2, y_perm, y_dtype, workspace, workspace_bytes, stream, nullptr, k, expert_scale,
                    expert_idx, perm_src, inv_perm, expert_offsets);
}

// One grouped GEMM of the decode-sized case, for the comparison of Table 1 (fp16 / int8 / int4
// weights, magic-number or native conversion).
extern "C" int moe_grouped_gemm_wq(const void *x_perm, const int32_t *expert_offsets, int R, int E,
                                   int max_rows_per_expert, int K, int N, int bits, int native_convert,
                                   const void *w_packed, const void *scales, void *y, int y_dtype,
                                   void *stream)
{
    using namespace moe;
    if (!expert_offsets || !w_packed || (bits != 16 && !scales) || (R != 0 && (!x_perm || !y)))
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_gemm_wq: NULL pointer");
    if (R < 0 || E <= 0 || K <= 0 || N <= 0 || max_rows_per_expert < 0)
        return fail(MOE_ERR_INVALID_ARG, "moe_grouped_gemm_wq: R >= 0, max_rows_per_expert >= 0 and E, K, N > 0 required");
    if (K % 64 || N % 64) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_gemm_wq: K and N must be multiples of 64 (K=%d N=%d)", K, N);
    if (bits != 4 && bits != 8 && bits != 16) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_gemm_wq: bits must be 4, 8 or 16 (got %d)", bits);
    if (y_dtype != MOE_F16 && y_dtype != MOE_BF16 && y_dtype != MOE_F32) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_gemm_wq: unknown y_dtype %d", y_dtype);
    if (E > 4096) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_gemm_wq: E=%d above 4096", E);
    const void *ptrs[] = {x_perm, w_packed, scales, y};
    for (const void *q : ptrs)
        if (!aligned16(q)) return fail(MOE_ERR_INVALID_ARG, "moe_grouped_gemm_wq: buffers must be 16-byte aligned");
    if (R == 0) return MOE_OK;
    const int max_rows = max_rows_per_expert > 0 && max_rows_per_expert < R ? max_rows_per_expert : R;
    if (max_rows > 64) return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_gemm_wq: only the decode-sized case (at most 64 rows per expert) is built");
    if (!stream_unrolled_supports(K, bits, SCALE_CHANNEL))
        return fail(MOE_ERR_UNSUPPORTED, "moe_grouped_gemm_wq: K=%d is not taken with bits=%d", K, bits);
    GemmArgs g{};
    g.a = (const uint16_t *)x_perm; g.offsets = expert_offsets; g.wq = (const uint8_t *)w_packed;
    g.scales = (const __half *)scales; g.bias = nullptr; g.out = y; g.E = E; g.R = R; g.K = K; g.N = N; g.g = K;
    g.out_dtype = y_dtype; g.act = MOE_ACT_NONE;
    hipStream_t s = as_stream(stream);
    if (bits == 16 || native_convert) return launch_stream_unrolled_variant(g, bits, native_convert != 0, max_rows, s);
    return launch_stream_unrolled(g, bits, max_rows, s);
}
