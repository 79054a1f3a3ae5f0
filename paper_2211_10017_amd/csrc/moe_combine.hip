// moe_combine: un-permute the expert outputs and apply expert_scale (Sec. 3.3, last step).
#include <type_traits>

#include "moe_common.h"

namespace moe {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) u32x4 *global_u32x4;

// Channels of a thread: sixteen bytes of a row of y.
constexpr int combine_channels(int y_dtype) { return y_dtype == MOE_F32 ? 4 : 8; }

template <int DT, int V>
__device__ inline void to_float(u32x4 w, float (&v)[V])
{
#pragma unroll
    for (int i = 0; i < V; ++i) {
        if (DT == MOE_F32) { v[i] = __uint_as_float(w[i & 3]); continue; }
        const uint16_t b = (uint16_t)(w[i >> 1] >> (16 * (i & 1)));
        if (DT == MOE_BF16) v[i] = __uint_as_float((uint32_t)b << 16);
        else { __half h; *reinterpret_cast<uint16_t *>(&h) = b; v[i] = __half2float(h); }
    }
}

__device__ inline uint16_t f32_to_bf16_rne(float f)
{
    uint32_t u = __float_as_uint(f);
    if ((u & 0x7fffffffu) > 0x7f800000u) return (uint16_t)((u >> 16) | 0x40u);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

template <int DT, int V>
__device__ inline void store_channels(void *base, size_t idx, const float (&v)[V])      // the idx-th V channels
{
    typedef uint32_t words_t __attribute__((ext_vector_type(DT == MOE_F32 ? 4 : V / 2)));
    constexpr int PER = DT == MOE_F32 ? V / 4 : 1;
#pragma unroll
    for (int s = 0; s < PER; ++s) {
        words_t w;
#pragma unroll
        for (int i = 0; i < (DT == MOE_F32 ? 4 : V / 2); ++i) {
            if (DT == MOE_F32) { w[i] = __float_as_uint(v[4 * s + i]); continue; }
            uint16_t b[2];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                if (DT == MOE_BF16) b[q] = f32_to_bf16_rne(v[2 * i + q]);
                else { __half h = __float2half_rn(v[2 * i + q]); b[q] = *reinterpret_cast<uint16_t *>(&h); }
            }
            w[i] = (uint32_t)b[0] | ((uint32_t)b[1] << 16);
        }
        reinterpret_cast<words_t *>(base)[PER * idx + s] = w;
    }
}

// What a pruned token's row is read from.
static __device__ const u32x4 no_row = {};

// A thread combines the channels of sixteen bytes of y (of fp32 y four: neighbouring lanes then read whole lines; 8192 tokens of 2048, one expert each, 27.2 us, eight a
// thread 30.0).  K: experts per token, 0 = any number, one after the other.  What bounds small batches is memory
// latencies in a row, so the rows of both experts are requested at once, whether they are active or not: two latencies, index and rows, instead of four (a step of 405
// tokens, two of 64 experts of 512 x 2048, 41.1 -> 40.4 us); large ones, bytes in flight: sixteen-byte loads of both rows (8192 tokens of 4096, FP16 y: 58.7 -> 45.6 us,
// 5.9 TB/s).  Rows of pruned tokens (Sec. 3.5), at or past *active_rows, need not be there: their loads go to one line of zeros
// (8192 tokens of 4096, all / two thirds / 40 % of the rows active, FP16 y 56.6 / 48.3 / 42.1 us a call, loaded whether active or not 56.3 each; launches of 2 to 4 us
// as before, where branches around the loads take 0.4 us more).
template <int YDT, int ODT, int K, class Index>
__global__ __launch_bounds__(256) void combine_kernel(const void *__restrict__ y_perm,
                                                      const int32_t *__restrict__ inv_perm,
                                                      const float *__restrict__ scale,
                                                      const int32_t *__restrict__ active_rows, int T, int k,
                                                      int dv, void *__restrict__ out)
{
    constexpr int N = K ? K : 1, V = combine_channels(YDT);
    const Index total = (Index)T * dv;
    for (Index i = (Index)blockIdx.x * 256 + threadIdx.x; i < total; i += (Index)gridDim.x * 256) {
        const int t = (int)(i / dv), c = (int)(i - (Index)t * dv);
        float acc[V] = {};
        for (int j0 = 0; j0 < (K ? 1 : k); ++j0) {
            const size_t a = K ? (size_t)t * K : (size_t)t * k + j0;
            int r[N];
            float s[N];
            u32x4 y[N];
#pragma unroll
            for (int j = 0; j < N; ++j) r[j] = inv_perm[a + j], s[j] = scale[a + j];
            const int active = active_rows ? *active_rows : 0x7fffffff;
#pragma unroll
            for (int j = 0; j < N; ++j)
                y[j] = *reinterpret_cast<global_u32x4>(r[j] < active ? (uintptr_t)y_perm + ((size_t)r[j] * dv + c) * 16 : (uintptr_t)&no_row);
#pragma unroll
            for (int j = 0; j < N; ++j) {
                float v[V];
                to_float<YDT>(y[j], v);
#pragma unroll
                for (int q = 0; q < V; ++q) acc[q] = r[j] < active ? fmaf(s[j], v[q], acc[q]) : acc[q];
            }
        }
        store_channels<ODT>(out, (size_t)i, acc);
    }
}

}  // namespace moe

extern "C" int moe_combine(const void *y_perm, int y_dtype, const int32_t *inv_perm,
                           const float *expert_scale, const int32_t *active_rows, int T, int k, int d,
                           void *out, int out_dtype, void *stream)
{
    using namespace moe;
    if (T == 0 && k > 0 && d > 0) return MOE_OK;         // empty buffers may be NULL
    if (!y_perm || !inv_perm || !expert_scale || !out) return fail(MOE_ERR_INVALID_ARG, "moe_combine: NULL pointer");
    if (T < 0 || k <= 0 || d <= 0 || d % 8) return fail(MOE_ERR_INVALID_ARG, "moe_combine: need T >= 0, k > 0, d > 0, d %% 8 == 0");
    if (y_dtype < 0 || y_dtype > 2 || out_dtype < 0 || out_dtype > 2) return fail(MOE_ERR_UNSUPPORTED, "moe_combine: unknown dtype");
    if (!aligned16(y_perm) || !aligned16(out)) return fail(MOE_ERR_INVALID_ARG, "moe_combine: buffers must be 16-byte aligned");
    const int dv = d / combine_channels(y_dtype);
    const size_t total = (size_t)T * dv, blocks = (total + 255) / 256;
    hipStream_t s = as_stream(stream);
    auto launch = [&](auto y, auto o) {
        constexpr int Y = decltype(y)::value, O = decltype(o)::value;
        const dim3 grid((unsigned)(blocks > 0x400000 ? 0x400000 : blocks));
        const bool narrow = total < 0x40000000u;        // (indices of 32 bits, a good part of so small a kernel)
        auto run = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, s, y_perm, inv_perm, expert_scale, active_rows, T, k, dv, out); };
        if (!narrow) run(&combine_kernel<Y, O, 0, size_t>);
        else if (k == 1) run(&combine_kernel<Y, O, 1, uint32_t>);
        else if (k == 2) run(&combine_kernel<Y, O, 2, uint32_t>);
        else run(&combine_kernel<Y, O, 0, uint32_t>);
        return check_launch("moe_combine");
    };
    auto with_out = [&](auto y) {
        return out_dtype == MOE_F16 ? launch(y, std::integral_constant<int, MOE_F16>{}) : out_dtype == MOE_BF16 ? launch(y, std::integral_constant<int, MOE_BF16>{})
             : launch(y, std::integral_constant<int, MOE_F32>{});
    };
    return y_dtype == MOE_F16 ? with_out(std::integral_constant<int, MOE_F16>{}) : y_dtype == MOE_BF16 ? with_out(std::integral_constant<int, MOE_BF16>{})
         : with_out(std::integral_constant<int, MOE_F32>{});
}
