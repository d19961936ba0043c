// Device code shared by the grouped-FFN kernels (ffn.hip, ffn_stream.h).
#pragma once
#include "moe_internal.h"

namespace moe {
namespace ffn_dev {

__device__ __forceinline__ int64_t clamp_row(int32_t v, int64_t cap)
{
    int64_t r = v < 0 ? 0 : v;
    return r > cap ? cap : r;
}

// Row range of expert e in one call's row space: a routed expert e < El holds
// [offsets[e], offsets[e+1]) clamped to [0, cap]; the shared expert (e == El,
// present when the call has shared rows) holds [cap, cap + shared_rows).
__device__ __forceinline__ int64_t expert_begin(const int32_t *__restrict__ offsets, int El, int64_t cap, int e)
{
    return e < El ? clamp_row(offsets[e], cap) : cap;
}

__device__ __forceinline__ int64_t expert_end(const int32_t *__restrict__ offsets, int El, int64_t cap,
                                              int64_t shared_rows, int e)
{
    return e < El ? clamp_row(offsets[e + 1], cap) : cap + shared_rows;
}

// SwiGLU of one gate/up pair: silu(g) * u = g / (1 + e^-g) * u, with the
// hardware reciprocal (the result is rounded to bf16).
__device__ __forceinline__ float silu_mul(float g, float u)
{
    return g * __builtin_amdgcn_rcpf(1.0f + __expf(-g)) * u;
}

__device__ __forceinline__ uint16_t bf16_bits(float f)
{
    __bf16 h = static_cast<__bf16>(f);  // round to nearest even
    return *reinterpret_cast<uint16_t *>(&h);
}

}  // namespace ffn_dev
}  // namespace moe
