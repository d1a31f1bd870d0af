// Operands of the fp32 matrix instruction v_mfma_f32_16x16x4_f32, shared by the fp32 attention and column-mass kernels.
//
// A lane (m = lane & 15, kk = lane >> 4) holds one value of A's row m and one of B's column m per instruction, and four
// results: rows 4 kk .. 4 kk + 3 of column m.  The order of the contraction is free as long as both sides agree, so lane
// kk takes the kk-th quarter of the channels of its row: D / 4 consecutive values, loaded 16 bytes at a time.
#pragma once

#include "kvs_internal.h"

namespace kvs {
namespace {

typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;

// channels kk * D / 4 .. of row `row` (in elements from `base`), widened to fp32
template <int DTYPE, int D>
__device__ __forceinline__ void load_quarter(const void *__restrict__ base, int64_t row, int kk, float (&x)[D / 4])
{
    if constexpr (DTYPE == KVS_F32) {
        const float4 *p = reinterpret_cast<const float4 *>(reinterpret_cast<const float *>(base) + row + kk * (D / 4));
#pragma unroll
        for (int i = 0; i < D / 16; ++i) {
            const float4 v = p[i];
            x[4 * i] = v.x; x[4 * i + 1] = v.y; x[4 * i + 2] = v.z; x[4 * i + 3] = v.w;
        }
    } else {
        const uint4 *p = reinterpret_cast<const uint4 *>(reinterpret_cast<const uint16_t *>(base) + row + kk * (D / 4));
#pragma unroll
        for (int i = 0; i < D / 32; ++i) {
            const uint4 v = p[i];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) { x[8 * i + 2 * u] = bf16_lo(w[u]); x[8 * i + 2 * u + 1] = bf16_hi(w[u]); }
        }
    }
}

// 16 x 16 dot products of D channels: entry r of a lane is row 4 kk + r of `a` with row m of `b`.  Two chains, so that an
// instruction does not wait for the one before.
template <int D>
__device__ __forceinline__ f32x4 dots(const float (&a)[D / 4], const float (&b)[D / 4])
{
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < D / 4; i += 2) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[i], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i + 1], b[i + 1], s1, 0, 0, 0);
    }
    return s0 + s1;
}

} // namespace
} // namespace kvs
