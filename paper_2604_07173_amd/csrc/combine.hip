// Routing-weighted combine of the per-pair updates of the down projection into token rows
// (Sec. 4.1: a token activates its top-k experts, pair p = t * k + j; Sec. 3 / Fig. 7b: the
// update is added to the base output):
//   y[t] = bf16( f32(y[t]) + sum over j = 0 .. k-1, ascending, of w[t*k+j] * update[t*k+j] )
// over the pairs that have a valid adapter and expert; a token without any such pair is not
// touched.  The sum runs in a fixed order in fp32, so results are bit-identical run to run.
//
// Every wave works alone on one token and 512 of its columns at a time (a lane on eight, 16 bytes of a bf16 row).  The first
// lanes fetch the ids and weights of the token's pairs together; then the token's row and the pair rows that are added to
// it are on their way at once.  Rows of inactive pairs, and tokens without an active pair, are not read.  Bound by the latency of its
// loads up to some 512 tokens, by the memory beyond.  4096 columns, top-2, layer call of a down projection with 8 inputs,
// a workgroup per token that fetches one thing after the other / pair rows fetched beside the ids, whatever they say / now, us: all
// pairs active 64 tokens 10.9 / 8.6 / 8.9, 2048 tokens 29.3 / 26.3 / 26.8, 8192 tokens 71.5 / 68.1 / 69.2; half of the
// tokens without adapter 10.5 / 8.2 / 8.4, 22.7 / 19.7 / 20.7, 45.7 / 50.1 / 41.2; no token with an adapter 6.1 / 6.0 / 6.0,
// 7.4 / 10.5 / 7.0, 13.6 / 27.1 / 12.1.  The largest loss: 131072 tokens, all pairs active, 1108 / 1148 / 1147.
#include <algorithm>

#include "lora_device.h"
#include "lora_internal.h"

namespace lora {

namespace {

constexpr int kMaxTopK = 16;

// K: pair rows kept, at least top_k
template <int K>
__global__ __launch_bounds__(256) void combine_kernel(CombineParams p)
{
    asm volatile("" ::"s"(p.pair), "s"(p.ld_pair), "s"(p.adapter_id), "s"(p.expert_id), "s"(p.route_w), "s"(p.y), "s"(p.ldy));     // together
    const int lane = threadIdx.x & 63;
    const int item = __builtin_amdgcn_readfirstlane(blockIdx.x * 4 + (threadIdx.x >> 6));
    const int t = item / p.waves_div;
    if (t >= p.T) return;

    const int64_t pr = (int64_t)t * p.top_k + min(lane, p.top_k - 1);
    const int a = p.adapter_id[pr];
    const int e = p.expert_id ? p.expert_id[pr] : 0;
    const float route = p.route_w[pr];
    const uint16_t *rows = p.pair + (int64_t)t * p.top_k * p.ld_pair;
    uint16_t *yrow = p.y + (int64_t)t * p.ldy;
    const unsigned active = (unsigned)__ballot(lane < p.top_k && a >= 0 && a < p.n_adapters && e >= 0 && e < p.n_experts);
    if (!active) return;
#pragma unroll 1
    for (int c0 = (item - t * p.waves) * kCombineCols; c0 < p.h_out; c0 += p.waves * kCombineCols) {
        const int c = c0 + lane * 8;
        const int cc = min(c, p.h_out - 8);
        const u32x4 yv = ld16<false>(yrow + cc);
        u32x4 d[K];
#pragma unroll
        for (int j = 0; j < K; ++j)
            if (active >> j & 1u) d[j] = ld16<true>(rows + j * p.ld_pair + cc);      // wave-uniform, all of them before the first sum
        float acc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) acc[q] = 0.f;
#pragma unroll
        for (int j = 0; j < K; ++j) {
            if (active >> j & 1u) {
                const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(route), j));
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    acc[2 * q] += w * __uint_as_float(d[j][q] << 16);
                    acc[2 * q + 1] += w * __uint_as_float(d[j][q] & 0xFFFF0000u);
                }
            }
        }
        u32x4 o;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            o[q] = pack_bf16_rne(__uint_as_float(yv[q] << 16) + acc[2 * q], __uint_as_float(yv[q] & 0xFFFF0000u) + acc[2 * q + 1]);
        if (c < p.h_out) st16<false>(yrow + cc, o);
    }
}

__global__ __launch_bounds__(256) void fill_zero_kernel(u32x4 *dst, size_t n_vec)
{
    const u32x4 z = {0u, 0u, 0u, 0u};
    for (size_t i = (size_t)blockIdx.x * 256 + threadIdx.x; i < n_vec; i += (size_t)gridDim.x * 256)
        st16<false>(dst + i, z);
}

}  // namespace

int combine_max_top_k() { return kMaxTopK; }

hipError_t launch_combine(const CombineParams &p_in, hipStream_t s)
{
    CombineParams p = p_in;
    if (p.T <= 0) return hipSuccess;
    if (p.top_k < 1 || p.top_k > kMaxTopK || p.h_out < 8) return hipErrorInvalidValue;
    p.waves = combine_waves(p.T, p.h_out);
    p.waves_div = fast_div(p.waves);
    const dim3 grid((unsigned)(((int64_t)p.T * p.waves + 3) / 4));
    if (p.top_k <= 2) hipLaunchKernelGGL(combine_kernel<2>, grid, dim3(256), 0, s, p);
    else if (p.top_k <= 4) hipLaunchKernelGGL(combine_kernel<4>, grid, dim3(256), 0, s, p);
    else if (p.top_k <= 8) hipLaunchKernelGGL(combine_kernel<8>, grid, dim3(256), 0, s, p);
    else hipLaunchKernelGGL(combine_kernel<kMaxTopK>, grid, dim3(256), 0, s, p);
    return hipGetLastError();
}

hipError_t launch_fill_zero(void *dst, size_t bytes, hipStream_t s)
{
    const size_t n_vec = bytes / 16;
    if (n_vec == 0) return hipSuccess;
    const unsigned grid = (unsigned)std::min<size_t>((n_vec + 255) / 256, 4096);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(grid), dim3(256), 0, s, static_cast<u32x4 *>(dst), n_vec);
    return hipGetLastError();
}

}  // namespace lora
