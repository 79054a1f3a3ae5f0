// moe_permute: stable counting sort of the (expert, row) tuples by expert and gather of the
// activation rows into expert-contiguous order (Sec. 3.3).
//
// The assignment list a = 0..R-1 is cut into wave-chunks of CH consecutive assignments; a
// wavefront counts its chunk per expert (integer LDS atomics: order-independent), the
// counts are turned into per-chunk start positions by an exclusive scan over (expert, chunk),
// and each wavefront then ranks its assignments in order with ballot-based match masks, so
// the sort is stable and free of global atomics.  Small problems (up to 4096 assignments) take
// a single launch that also copies the rows; larger ones take a count launch, a rank launch and
// a row-copy launch.
//
// Batch pruning (Sec. 3.5): an expert index equal to E marks a row of a finished sentence.  It is
// one more key of the sort, the last one, so such rows end up behind every active row;
// expert_offsets[E] is then the number of active rows, and pruned rows are not copied.
#include <type_traits>

#include "moe_common.h"

namespace moe {

constexpr int kPermMaxE = 1024;
constexpr int kPermFused = 4096;         // assignments that one launch takes (its blocks all sort them)

__device__ inline uint64_t lanemask_lt() { return (1ull << (threadIdx.x & 63)) - 1ull; }

// lanes of this wavefront holding the same key (keys < 1024), computed with 10 ballots
__device__ inline uint64_t match_key(int key, int key_bits)
{
    uint64_t m = ~0ull;
    for (int b = 0; b < key_bits; ++b) {
        const uint64_t set = __ballot((key >> b) & 1);
        m &= ((key >> b) & 1) ? set : ~set;
    }
    return m;
}

// FUSED: small problems, one launch: every block repeats count + scan + rank for all
// assignments (cheap), keeps perm_src in LDS and then gathers its share of the rows; block 0
// writes the index outputs.  Otherwise PHASE selects count (0) or rank (1), and the per-chunk
// histograms travel through `hist` [nwc][E].
// W: wavefronts of a block; ITERS: the most steps of 64 assignments of a wave-chunk.
template <bool FUSED, int PHASE, int W, int ITERS>
__global__ __launch_bounds__(64 * W) void permute_index_kernel(const int32_t *__restrict__ expert_idx,
                                                            int R, int NB, int iters, int nwc,
                                                            int key_bits, int32_t *__restrict__ hist,
                                                            int32_t *__restrict__ perm_src,
                                                            int32_t *__restrict__ inv_perm,
                                                            int32_t *__restrict__ offsets,
                                                            const uint4 *__restrict__ x, int k, int row_vec,
                                                            uint4 *__restrict__ x_perm)
{
    extern __shared__ int32_t sm[];          // [W][NB] per-wave counters, [NB] scratch, (FUSED) [R] perm_src
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int blk = FUSED ? 0 : blockIdx.x;  // FUSED: every block plays block 0 of the index phase
    const bool writer = !FUSED || blockIdx.x == 0;
    int32_t *perm_l = sm + (W + 1) * NB;
    const int wc = blk * W + wave;           // wave-chunk id
    const int CH = iters * 64;
    int32_t *cnt = sm + wave * NB;
    int32_t *tot = sm + W * NB;

    // The chunk's keys are requested together and kept for both passes over them: a load inside each step's chain of counting,
    // ranking and barriers would cost a memory latency per step and pass.
    int keys[ITERS];
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        const int a = wc * CH + it * 64 + lane;
        if (it < iters) keys[it] = a < R ? min(max(expert_idx[a], 0), NB - 1) : -1;          // clamped: never out of range
    }
    if (FUSED || PHASE == 0) {
        for (int e = threadIdx.x; e < W * NB; e += 64 * W) sm[e] = 0;
        __syncthreads();
#pragma unroll
        for (int it = 0; it < ITERS; ++it)
            if (it < iters && keys[it] >= 0) atomicAdd(&cnt[keys[it]], 1);
        __syncthreads();
        if (!FUSED) {
            for (int e = threadIdx.x; e < W * NB; e += 64 * W) hist[(size_t)blk * W * NB + e] = sm[e];
            return;
        }
    }

    // start position of every (expert, wave-chunk of this block): cnt[w][e] <- base
    for (int e = threadIdx.x; e < NB; e += 64 * W) {
        int before = 0, total = 0;
        int c[W];
        if (FUSED) {
#pragma unroll
            for (int w = 0; w < W; ++w) {
                c[w] = sm[w * NB + e];
                total += c[w];
            }
        } else {
#pragma unroll
            for (int w = 0; w < W; ++w) c[w] = hist[(size_t)(blk * W + w) * NB + e];
#pragma unroll 16
            for (int j = 0; j < nwc; ++j) {              // independent loads: many in flight
                const int v = hist[(size_t)j * NB + e];
                before += j < blk * W ? v : 0;
                total += v;
            }
        }
        tot[e] = total;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            sm[w * NB + e] = before;
            before += c[w];
        }
    }
    __syncthreads();
    // exclusive scan of the totals over experts by wavefront 0 (64 experts per step)
    if (wave == 0) {
        int carry = 0;
        for (int e0 = 0; e0 < NB; e0 += 64) {
            const int e = e0 + lane;
            const int v = e < NB ? tot[e] : 0;
            int incl = v;
            for (int off = 1; off < 64; off <<= 1) {
                const int up = __shfl_up(incl, off);
                if (lane >= off) incl += up;
            }
            if (e < NB) tot[e] = carry + incl - v;
            carry += __shfl(incl, 63);
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < NB; e += 64 * W) {
        const int base = tot[e];
        if (writer && blk == 0) offsets[e] = base;
#pragma unroll
        for (int w = 0; w < W; ++w) sm[w * NB + e] += base;
    }
    __syncthreads();

    // rank: cnt[key] is the next free position of `key` for this wave-chunk
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
        if (it >= iters) break;
        const int a = wc * CH + it * 64 + lane;
        const bool live = keys[it] >= 0;
        const int key = max(keys[it], 0);
        uint64_t m = match_key(live ? key : (1 << key_bits) - 1, key_bits);
        m &= __ballot(live);                 // idle lanes never share a group with live ones
        const int rank = __popcll(m & lanemask_lt());
        int r = 0;
        if (live) {
            r = cnt[key] + rank;
            if (FUSED) perm_l[r] = a;
            if (writer) {
                perm_src[r] = a;
                inv_perm[a] = r;
            }
        }
        // the counters are the wavefront's own: its reads are over before its leaders' writes, and those before the next step
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if (live && rank == 0) cnt[key] += __popcll(m);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    if (FUSED && x) {
        __syncthreads();                     // the whole permutation is there
        // x_perm[r] = x[perm_src[r] / k] for this block's share of the active rows; one wavefront per row
        const int active = tot[NB - 1];
        for (int r = blockIdx.x * W + wave; r < active; r += gridDim.x * W) {
            const uint4 *src = x + (size_t)(perm_l[r] / k) * row_vec;
            uint4 *dst = x_perm + (size_t)r * row_vec;
            for (int v = lane; v < row_vec; v += 64) dst[v] = src[v];
        }
    }
}

// x_perm[r] = x[perm_src[r] / k]; one wavefront per row, 16 bytes per lane per step
__global__ __launch_bounds__(256) void gather_rows_kernel(const uint4 *__restrict__ x,
                                                          const int32_t *__restrict__ perm_src,
                                                          const int32_t *__restrict__ active_rows, int R,
                                                          int k, int row_vec, uint4 *__restrict__ x_perm)
{
    const int lane = threadIdx.x & 63;
    const int active = min(*active_rows, R);
    for (int r = blockIdx.x * 4 + (threadIdx.x >> 6); r < active; r += gridDim.x * 4) {
        const int t = perm_src[r] / k;
        const uint4 *src = x + (size_t)t * row_vec;
        uint4 *dst = x_perm + (size_t)r * row_vec;
        for (int v = lane; v < row_vec; v += 64) dst[v] = src[v];
    }
}

// one block's worth, one launch; beyond: 256 assignments per wavefront
constexpr int kPermSteps = 4;
static int perm_blocks(int R) { return R <= kPermFused ? 1 : (R + 256 * kPermSteps - 1) / (256 * kPermSteps); }

}  // namespace moe

extern "C" size_t moe_permute_workspace_bytes(int T, int k, int E)
{
    if (T <= 0 || k <= 0 || E <= 0) return 16;
    return moe::round_up((size_t)moe::perm_blocks(T * k) * 4 * (E + 1) * sizeof(int32_t), 256);
}

extern "C" int moe_permute(const int32_t *expert_idx, const void *x, int act_dtype, int T, int k, int E,
                           int d, void *x_perm, int32_t *perm_src, int32_t *inv_perm,
                           int32_t *expert_offsets, void *workspace, size_t workspace_bytes,
                           void *stream)
{
    using namespace moe;
    if (!expert_offsets || (T > 0 && (!expert_idx || !perm_src || !inv_perm)))
        return fail(MOE_ERR_INVALID_ARG, "moe_permute: NULL index pointer");
    if (T > 0 && (x == nullptr) != (x_perm == nullptr)) return fail(MOE_ERR_INVALID_ARG, "moe_permute: x and x_perm must both be given or both be NULL");
    if (T < 0 || k <= 0 || E <= 0 || d <= 0) return fail(MOE_ERR_INVALID_ARG, "moe_permute: T >= 0 and k, E, d > 0 required");
    if (E > kPermMaxE) return fail(MOE_ERR_UNSUPPORTED, "moe_permute: E=%d above %d", E, kPermMaxE);
    if (act_dtype != MOE_F16 && act_dtype != MOE_BF16 && act_dtype != MOE_F32) return fail(MOE_ERR_UNSUPPORTED, "moe_permute: unknown act_dtype %d", act_dtype);
    const int elt = act_dtype == MOE_F32 ? 4 : 2;
    if (((size_t)d * elt) % 16) return fail(MOE_ERR_INVALID_ARG, "moe_permute: rows must be a multiple of 16 bytes (d=%d)", d);
    if ((long long)T * k > 0x7fffffffLL) return fail(MOE_ERR_INVALID_ARG, "moe_permute: T*k overflows int32");
    if (!aligned16(x) || !aligned16(x_perm)) return fail(MOE_ERR_INVALID_ARG, "moe_permute: x and x_perm must be 16-byte aligned");
    const int R = T * k;
    const int nblocks = perm_blocks(R);
    const size_t need = moe_permute_workspace_bytes(T, k, E);
    if (nblocks > 1 && (!workspace || workspace_bytes < need))
        return fail(MOE_ERR_WORKSPACE, "moe_permute: workspace of %zu bytes needed, %zu given", need, workspace_bytes);
    const int NB = E + 1;                              // keys: the experts and the pruned-row index E
    int key_bits = 1;
    while ((1 << key_bits) < NB + 1) ++key_bits;       // one spare code for idle lanes
    hipStream_t s = as_stream(stream);
    const size_t smem = (size_t)5 * NB * sizeof(int32_t);
    int32_t *hist = (int32_t *)workspace;
    const int row_vec = (int)((size_t)d * elt / 16);
    if (nblocks == 1) {
        // index and gather in one launch: up to 64 blocks share the row copies
        int gb = x ? (R + 3) / 4 : 1;
        gb = gb < 1 ? 1 : gb > 64 ? 64 : gb;
        // Four, eight or sixteen wavefronts per block, the fewest steps in a row for each that their start-up allows: up to 256, up to 512
        // and more assignments (and at most eight where the counters of sixteen would not fit).  Index / index and copies of rows of 1024,
        // 128 experts: 256 assignments 3.4 / 4.1 us in four wavefronts, 3.6 / 4.4 in eight, 4.0 / 5.2 in sixteen; 400 4.1 / 5.3, 3.7 / 4.5, 4.1 / 5.3;
        // 2000 8.4 / 12.3, 5.8 / 8.2, 5.3 / 7.3 (in a quarter of the blocks 10.2); a step of 64 unrolled sixteen times for all sizes adds 0.15-0.3 us.
        auto launch = [&](auto w_c, auto it_c) {
            constexpr int W = decltype(w_c)::value, ITERS = decltype(it_c)::value;
            const int steps = R > 64 * W ? (R + 64 * W - 1) / (64 * W) : 1;
            hipLaunchKernelGGL((permute_index_kernel<true, 0, W, ITERS>), dim3(gb), dim3(64 * W), ((size_t)(W + 1) * NB + R) * sizeof(int32_t), s, expert_idx, R, NB, steps,
                               W, key_bits, hist, perm_src, inv_perm, expert_offsets, (const uint4 *)x, k, row_vec, (uint4 *)x_perm);
        };
        using std::integral_constant;
        if (R <= 256) launch(integral_constant<int, 4>{}, integral_constant<int, 1>{});
        else if (R <= 512) launch(integral_constant<int, 8>{}, integral_constant<int, 1>{});
        else if (NB <= 512) launch(integral_constant<int, 16>{}, integral_constant<int, kPermFused / 1024>{});
        else launch(integral_constant<int, 8>{}, integral_constant<int, kPermFused / 512>{});
        return check_launch("moe_permute");
    }
    hipLaunchKernelGGL((permute_index_kernel<false, 0, 4, kPermSteps>), dim3(nblocks), dim3(256), smem, s, expert_idx, R, NB, kPermSteps,
                       nblocks * 4, key_bits, hist, perm_src, inv_perm, expert_offsets, (const uint4 *)nullptr, k,
                       row_vec, (uint4 *)nullptr);
    hipLaunchKernelGGL((permute_index_kernel<false, 1, 4, kPermSteps>), dim3(nblocks), dim3(256), smem, s, expert_idx, R, NB, kPermSteps,
                       nblocks * 4, key_bits, hist, perm_src, inv_perm, expert_offsets, (const uint4 *)nullptr, k,
                       row_vec, (uint4 *)nullptr);
    int rc = check_launch("moe_permute (index)");
    if (rc != MOE_OK || !x || R == 0) return rc;
    int gblocks = (R + 3) / 4;
    if (gblocks > 4096) gblocks = 4096;
    hipLaunchKernelGGL(gather_rows_kernel, dim3(gblocks), dim3(256), 0, s, (const uint4 *)x, perm_src, expert_offsets + E, R, k,
                       row_vec, (uint4 *)x_perm);
    return check_launch("moe_permute (gather)");
}
