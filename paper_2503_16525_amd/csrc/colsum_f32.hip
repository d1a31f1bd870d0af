// kvs_attn_colsum in fp32 for the shapes the bf16 matrix-core kernel does not cover (fp32, head_dim 64, a scale that is not
// positive): the same two sweeps (row statistics, then column sums of the weights; Alg. 1 steps 1-2) on the fp32
// matrix instruction.  A workgroup owns 16 fixed rows of a KV head (query rows, flattened (token, head-in-group), in sweep
// 1; keys in sweep 2); its eight waves deal the streamed 16-row tiles among themselves and read them straight from global
// memory, the next tile while one is worked on.  A lane's results belong to one fixed row, so the running sums are a lane's own and
// the loop has no cross-lane traffic; the 32 shares of a fixed row meet in LDS, one a lane, in a fixed tree (one thread a row: the
// five calls on the 512-token layer 43.2 us, 41.7 like this, and twice the rms error of alpha: 9.9e-8 against 4.3e-8).
//
// Measured, fp32 512 tokens x 4 heads, head_dim 64: 57 -> 18 us for both sweeps (before: one wave per row on the vector
// units, element by element).  Meant for small layers; nothing is staged or shared between workgroups.
#include "f32_tiles.h"

#include <math.h>

namespace kvs {
namespace {

constexpr int kCfWaves = 8;
constexpr int kCfThreads = kCfWaves * 64;
constexpr int kCfRows = 16;

// SWEEP 1: stats[g][row] = (maximum, 1 / sum of exp(score - maximum)); SWEEP 2: alpha[g][key].  Rows of a KV head's queries:
// row = token * grp + head-in-group.  (The pair and not its log-sum-exp: rounding that to 32 bits moves a whole row's weights
// by up to 3e-7, the largest single error of alpha.  512 tokens, rms error against 64 bits: 1.6e-7 with it, 1.0e-7 with the pair, at the same time.)
template <int SWEEP, int DTYPE, int D>
__global__ __launch_bounds__(kCfThreads) void colsum_f32_kernel(int n, int n_q_heads, int n_kv_heads, const void *__restrict__ q,
                                                                const void *__restrict__ k, float scale,
                                                                const float2 *__restrict__ row_stats, float2 *__restrict__ stats, float *__restrict__ alpha)
{
    __shared__ float m_s[kCfWaves * 4][kCfRows + 1], z_s[kCfWaves * 4][kCfRows + 1];
    const int tid = threadIdx.x, lane = tid & 63, m16 = lane & 15, kk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = n_q_heads / n_kv_heads;
    const int g = blockIdx.x % n_kv_heads, blk = blockIdx.x / n_kv_heads;
    const int n_qrows = n * grp, n_fixed = SWEEP == 1 ? n_qrows : n;
    // heaviest first: the last query rows see the most keys, the first keys are seen by the most rows
    const int fb = (SWEEP == 1 ? (n_fixed - 1) / kCfRows - blk : blk) * kCfRows;
    auto q_row = [&](int r) { return ((int64_t)(r / grp) * n_q_heads + g * grp + r % grp) * D; };
    auto k_row = [&](int i) { return ((int64_t)i * n_kv_heads + g) * D; };
    const int fr = min(fb + m16, n_fixed - 1);
    float fx[D / 4];
    load_quarter<DTYPE, D>(SWEEP == 1 ? q : k, SWEEP == 1 ? q_row(fr) : k_row(fr), kk, fx);
    const int fpos = SWEEP == 1 ? fr / grp : fr;       // position of the fixed row
    const int last = min(fb + kCfRows, n_fixed) - 1;
    const int t_begin = SWEEP == 1 ? 0 : fb * grp / kCfRows, t_end = SWEEP == 1 ? last / grp / kCfRows + 1 : (n_qrows + kCfRows - 1) / kCfRows;
    const int n_stream = SWEEP == 1 ? n : n_qrows;
    float m = kLowest, z = 0.f;
    // the next tile's rows are on their way while a tile is worked on (past the last tile the last row again, never used)
    float x_next[D / 4];
    float2 st_next[4];
    auto fetch = [&](int t) {
        const int sr = min(t * kCfRows + m16, n_stream - 1);
        load_quarter<DTYPE, D>(SWEEP == 1 ? k : q, SWEEP == 1 ? k_row(sr) : q_row(sr), kk, x_next);
        if (SWEEP == 2) {
#pragma unroll
            for (int r = 0; r < 4; ++r) st_next[r] = row_stats[(int64_t)g * n_qrows + min(t * kCfRows + 4 * kk + r, n_stream - 1)];
        }
    };
    fetch(t_begin + wave);
    for (int t = t_begin + wave; t < t_end; t += kCfWaves) {
        float x[D / 4];
        float2 st4[4];
#pragma unroll
        for (int c = 0; c < D / 4; ++c) x[c] = x_next[c];
#pragma unroll
        for (int r = 0; SWEEP == 2 && r < 4; ++r) st4[r] = st_next[r];
        fetch(t + kCfWaves);
        const f32x4 s = dots<D>(x, fx);
        float y[4];
        bool sees[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int row = t * kCfRows + 4 * kk + r;
            sees[r] = SWEEP == 1 ? row <= fpos : row < n_stream && row / grp >= fpos;
            y[r] = sees[r] ? s[r] * scale : -INFINITY;
        }
        if (SWEEP == 1) {
            const float mn = fmaxf(m, fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])));
            z *= expf(m - mn);
            m = mn;
#pragma unroll
            for (int r = 0; r < 4; ++r) z += expf(y[r] - m);
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const float zr = fmaf(expf(y[r] - st4[r].x), st4[r].y, z);
                z = sees[r] ? zr : z;              // a row that does not see the key adds nothing, whatever its statistics are
            }
        }
    }
    m_s[wave * 4 + kk][m16] = m;
    z_s[wave * 4 + kk][m16] = z;
    __syncthreads();
    // 32 lanes a row, their shares added in a fixed tree
    static_assert(kCfWaves * 4 == 32 && kCfThreads == 32 * kCfRows, "one share a lane");
    const int share = tid & 31, row = tid >> 5;
    float zt = z_s[share][row], mt = m_s[share][row];
    if (SWEEP == 1) {
        const float mine = mt;
#pragma unroll
        for (int o = 16; o >= 1; o >>= 1) mt = fmaxf(mt, __shfl_xor(mt, o));
        zt *= expf(mine - mt);
    }
#pragma unroll
    for (int o = 16; o >= 1; o >>= 1) zt += __shfl_xor(zt, o);
    if (share == 0 && fb + row < n_fixed) {
        if (SWEEP == 1) stats[(int64_t)g * n_qrows + fb + row] = make_float2(mt, 1.0f / zt);
        else alpha[(int64_t)g * n + fb + row] = zt;
    }
}

template <int DTYPE, int D>
kvs_status launch_both(int n, int hq, int hk, const void *q, const void *k, float scale, float2 *stats, float *alpha, hipStream_t st)
{
    const int64_t rows = (int64_t)n * (hq / hk);
    const dim3 block(kCfThreads), g1((unsigned)((rows + kCfRows - 1) / kCfRows * hk)), g2((unsigned)(((int64_t)n + kCfRows - 1) / kCfRows * hk));
    hipLaunchKernelGGL((colsum_f32_kernel<1, DTYPE, D>), g1, block, 0, st, n, hq, hk, q, k, scale, (const float2 *)nullptr, stats,
                       (float *)nullptr);
    hipLaunchKernelGGL((colsum_f32_kernel<2, DTYPE, D>), g2, block, 0, st, n, hq, hk, q, k, scale, (const float2 *)stats,
                       (float2 *)nullptr, alpha);
    return check_launch("kvs_attn_colsum(f32)");
}

} // namespace

kvs_status launch_colsum_f32(const kvs_shape *shape, int64_t n, const void *q, const void *k, float scale,
                             void *row_stats, float *alpha, hipStream_t st)
{
    const int d = shape->head_dim, hq = shape->n_q_heads, hk = shape->n_kv_heads;
    // quadratic work at a few percent of the bf16 matrix-core rate: refuse what would run for minutes
    if (n > 65536) return fail(KVS_EUNSUPPORTED, "kvs_attn_colsum: %lld tokens are too many for the vector path (this shape has no matrix-core kernel)", (long long)n);
    if (n * (int64_t)(hq / hk) > 0x7ffffff0) return fail(KVS_EUNSUPPORTED, "kvs_attn_colsum: %lld tokens x %d query heads", (long long)n, hq);
    float2 *const stats = (float2 *)row_stats;          // 8 bytes per query row
    if (shape->dtype == KVS_F32) return d == 64 ? launch_both<KVS_F32, 64>((int)n, hq, hk, q, k, scale, stats, alpha, st) : launch_both<KVS_F32, 128>((int)n, hq, hk, q, k, scale, stats, alpha, st);
    return d == 64 ? launch_both<KVS_BF16, 64>((int)n, hq, hk, q, k, scale, stats, alpha, st) : launch_both<KVS_BF16, 128>((int)n, hq, hk, q, k, scale, stats, alpha, st);
}

} // namespace kvs
