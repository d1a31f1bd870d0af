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

// Sixteen rows on their way to such operands through LDS.  Taken straight from memory a lane's 16 bytes lie a row away from its
// neighbours' and every load is 64 separate requests (16 KB a wave, 8 waves: 3.4 us on one compute unit); here consecutive lanes load
// consecutive bytes, 1 KB an instruction.  Row r's 16-byte piece p lies at place p ^ swizzle(r), which spreads the 16 rows
// that are read at one piece over all banks.
template <int DTYPE, int D>
struct Rows16 {
    static constexpr int ROW_B = D * (DTYPE == KVS_F32 ? 4 : 2), PIECES = ROW_B / 16, BYTES = 16 * ROW_B, LOADS = BYTES / 1024, ROWS_A_LOAD = 1024 / ROW_B;
    static __device__ __forceinline__ int swizzle(int r) { return PIECES >= 16 ? r : r >> 1; }
    // a wave's load `i` of LOADS into the 16 rows at `lds`; row(r) is row r's first element in `base`.  It is under way when this returns:
    // before the rows are read, or their place is used for something else, the wave that asked waits (landed()), and
    // waves that read what another asked for meet it at a barrier after that.
    template <class Row>
    static __device__ __forceinline__ void load(const void *__restrict__ base, Row row, char *lds, int i, int lane)
    {
        const int r = i * ROWS_A_LOAD + lane / PIECES, piece = (lane % PIECES) ^ swizzle(r);
        const char *src = reinterpret_cast<const char *>(base) + row(r) * (ROW_B / D) + piece * 16;
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)src, (__attribute__((address_space(3))) void *)(lds + i * 1024), 16, 0, 0);
    }
    static __device__ __forceinline__ void landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
    // the kk-th quarter of row m's channels, widened
    static __device__ __forceinline__ void read(const char *lds, int m, int kk, float (&x)[D / 4])
    {
#pragma unroll
        for (int i = 0; i < PIECES / 4; ++i) {
            const uint4 v = *reinterpret_cast<const uint4 *>(lds + m * ROW_B + (((kk * (PIECES / 4) + i) ^ swizzle(m)) * 16));
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (DTYPE == KVS_F32) x[4 * i + u] = __uint_as_float(w[u]);
                else { x[8 * i + 2 * u] = bf16_lo(w[u]); x[8 * i + 2 * u + 1] = bf16_hi(w[u]); }
            }
        }
    }
};

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
