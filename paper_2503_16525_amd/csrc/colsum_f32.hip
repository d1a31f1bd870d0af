// kvs_attn_colsum in fp32 for the shapes the bf16 matrix-core kernel does not cover (fp32, head_dim 64, a scale that is not
// positive): one sweep for short layers (colsum_f32_rows_kernel), else the same two sweeps (row statistics, then column sums of
// the weights; Alg. 1 steps 1-2) on the fp32 matrix instruction.  In the two sweeps a workgroup owns 16 fixed rows of a KV head (query rows, flattened (token, head-in-group), in sweep
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
// Up to here one sweep, where its shares have room in the workspace: 16 rows' scores over 2048 tokens are 64 registers a lane.  It
// is the faster one at all of these lengths (from 300 tokens on; level below).
constexpr int64_t kCfOneSweepTokens = 2048;
constexpr size_t kCfOneSweepBytes = (size_t)32 << 20;

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

// Short layers in one sweep: the scores of 16 query rows over their whole context stay in the registers of a workgroup, MAXT
// tiles of 16 keys a wave, until the rows' maxima and sums are known (two barriers), and the weights' sums over the 16 rows go to
// part[g][row tile][key]; colsum_f32_join adds the row tiles.  Half of the two sweeps' products and exponentials, and no second
// launch that reads K and Q again.  Here the query rows are the instruction's rows and the keys its columns: a lane has four rows of
// one key, whose sum is its own and its three neighbours'.
// Measured, fp32 layers of 4 heads, head_dim 64, the five calls of a layer with this one among them: 512 tokens 38.6 -> 34.3 us, 1024
// 58.5 -> 50.7, 2048 95.6 -> 70.0; below 300 tokens the host is what they wait for.
// The keys come through LDS (Rows16): 512 tokens 34.7 -> 32.7 us, the kernel 9.1 -> 6.9; 2048 tokens 70.0 -> 65.4.
// A wave's tiles that are on their way together: all four of a short layer where they have room, else two, for two workgroups a unit.
template <int DTYPE, int D>
constexpr int tiles_in_flight(int max_tiles) { return max_tiles <= 4 && Rows16<DTYPE, D>::BYTES <= 4096 ? 4 : 2; }
template <int DTYPE, int D, int MAXT>
__global__ __launch_bounds__(kCfThreads, 2) void colsum_f32_rows_kernel(int n, int n_q_heads, int n_kv_heads, const void *__restrict__ q,
                                                                        const void *__restrict__ k, float scale, float *__restrict__ part)
{
    using Rows = Rows16<DTYPE, D>;
    constexpr int FETCH = tiles_in_flight<DTYPE, D>(MAXT);
    extern __shared__ __attribute__((aligned(16))) char rows_s[];  // the query rows, then FETCH tiles of keys a wave
    __shared__ __attribute__((aligned(16))) float m_s[kCfWaves][kCfRows], z_s[kCfWaves][kCfRows];
    const int tid = threadIdx.x, lane = tid & 63, m16 = lane & 15, kk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int grp = n_q_heads / n_kv_heads;
    const int g = blockIdx.x % n_kv_heads, blk = blockIdx.x / n_kv_heads;
    const int n_qrows = n * grp, row_tiles = (n_qrows + kCfRows - 1) / kCfRows, tile = row_tiles - 1 - blk;   // most keys first
    const int fb = tile * kCfRows;
    const int last = (min(fb + kCfRows, n_qrows) - 1) / grp;       // position of the last row
    char *const mine = rows_s + Rows::BYTES * (1 + FETCH * wave);
    // (past the last row's position keys are clamped and not used)
    auto fetch = [&](int i0) {
#pragma unroll
        for (int i = 0; i < FETCH; ++i) {
            const int k0 = (wave + (i0 + i) * kCfWaves) * kCfRows;
            if (k0 > last) continue;                               // uniform
#pragma unroll
            for (int l = 0; l < Rows::LOADS; ++l)
                Rows::load(k, [&](int r) { return ((int64_t)min(k0 + r, last) * n_kv_heads + g) * D; }, mine + i * Rows::BYTES, l, lane);
        }
    };
    if (wave < Rows::LOADS)
        Rows::load(q, [&](int r) { const int fr = min(fb + r, n_qrows - 1); return ((int64_t)(fr / grp) * n_q_heads + g * grp + fr % grp) * D; },
                   rows_s, wave, lane);
    fetch(0);
    int pos[4];                                                    // of this lane's rows (-1: no row)
#pragma unroll
    for (int r = 0; r < 4; ++r) pos[r] = fb + 4 * kk + r < n_qrows ? (fb + 4 * kk + r) / grp : -1;
    float s[MAXT][4], m[4], z[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) { m[r] = kLowest; z[r] = 0.f; }
    Rows::landed();
    __syncthreads();
    float fx[D / 4];
    Rows::read(rows_s, m16, kk, fx);
#pragma unroll
    for (int i0 = 0; i0 < MAXT; i0 += FETCH) {
        if ((wave + i0 * kCfWaves) * kCfRows > last) continue;     // uniform
        if (i0 > 0) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // what lay there has been read
            fetch(i0);
            Rows::landed();
        }
#pragma unroll
        for (int i = 0; i < FETCH; ++i) {
            const int key = (wave + (i0 + i) * kCfWaves) * kCfRows + m16;
            if (key - m16 > last) continue;
            float x[D / 4];
            Rows::read(mine + i * Rows::BYTES, m16, kk, x);
            const f32x4 y = dots<D>(fx, x);
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                s[i0 + i][r] = key <= pos[r] ? y[r] * scale : -INFINITY;
                m[r] = fmaxf(m[r], s[i0 + i][r]);
            }
        }
    }
    // the rows' maxima: over the 16 lanes of a row, then over the waves
#pragma unroll
    for (int r = 0; r < 4; ++r) m[r] = row16_max(m[r]);
    if (m16 == 0) *reinterpret_cast<f32x4 *>(&m_s[wave][4 * kk]) = f32x4{m[0], m[1], m[2], m[3]};
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kCfWaves; ++w) {
        const f32x4 o = *reinterpret_cast<const f32x4 *>(&m_s[w][4 * kk]);
#pragma unroll
        for (int r = 0; r < 4; ++r) m[r] = fmaxf(m[r], o[r]);
    }
#pragma unroll
    for (int i = 0; i < MAXT; ++i)
        if ((wave + i * kCfWaves) * kCfRows <= last) {
#pragma unroll
            for (int r = 0; r < 4; ++r) { s[i][r] = expf(s[i][r] - m[r]); z[r] += s[i][r]; }
        }
#pragma unroll
    for (int r = 0; r < 4; ++r) z[r] = row16_sum(z[r]);
    if (m16 == 0) *reinterpret_cast<f32x4 *>(&z_s[wave][4 * kk]) = f32x4{z[0], z[1], z[2], z[3]};
    __syncthreads();
    f32x4 o[kCfWaves];
#pragma unroll
    for (int w = 0; w < kCfWaves; ++w) o[w] = *reinterpret_cast<const f32x4 *>(&z_s[w][4 * kk]);
#pragma unroll
    for (int half = kCfWaves / 2; half >= 1; half /= 2)
#pragma unroll
        for (int w = 0; w < half; ++w) o[w] += o[w + half];
    float inv[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) inv[r] = 1.0f / o[0][r];
    float *const dst = part + ((int64_t)g * row_tiles + tile) * n;
#pragma unroll
    for (int i = 0; i < MAXT; ++i) {
        const int key = (wave + i * kCfWaves) * kCfRows + m16;
        if (key - m16 <= last) {
            float sum = 0.f;
#pragma unroll
            for (int r = 3; r >= 0; --r) sum = key <= pos[r] ? fmaf(s[i][r], inv[r], sum) : sum;   // a row that does not see the key adds nothing
            sum += __shfl_xor(sum, 16);
            sum += __shfl_xor(sum, 32);
            if (kk == 0 && key <= last) dst[key] = sum;
        }
    }
}

// alpha[g][key] = the row tiles' shares: 32 keys a workgroup, eight chains each.  In 64 bits, which costs nothing here and leaves the
// roundings of the shares only (rms error of alpha against 64 bits, 129 tokens, 60 layers: 5.0e-8 in 32 bits, two sweeps 4.8e-8, 4.1e-8 like this).
constexpr int kCjKeys = 32, kCjChains = 8;
__global__ __launch_bounds__(kCjKeys * kCjChains) void colsum_f32_join(int n, int grp, int row_tiles, const float *__restrict__ part, float *__restrict__ alpha)
{
    __shared__ double sums[kCjChains][kCjKeys];
    const int g = blockIdx.y, lane = threadIdx.x % kCjKeys, chain = threadIdx.x / kCjKeys, key = blockIdx.x * kCjKeys + lane;
    double sum = 0.0;
    if (key < n)
#pragma unroll 4
        for (int t = key * grp / kCfRows + chain; t < row_tiles; t += kCjChains) sum += part[((int64_t)g * row_tiles + t) * n + key];
    sums[chain][lane] = sum;
    __syncthreads();
    if (chain != 0 || key >= n) return;
#pragma unroll
    for (int c = 1; c < kCjChains; ++c) sum += sums[c][lane];
    alpha[(int64_t)g * n + key] = (float)sum;
}

template <int DTYPE, int D, int MAXT>
kvs_status launch_rows(dim3 grid, int n, int hq, int hk, const void *q, const void *k, float scale, float *part, hipStream_t st)
{
    using Rows = Rows16<DTYPE, D>;
    constexpr int lds_bytes = Rows::BYTES * (1 + tiles_in_flight<DTYPE, D>(MAXT) * kCfWaves);
    static_assert(Rows::LOADS <= kCfWaves, "a wave loads one share of the query rows");
    static DeviceOnce attr_once;
    const kvs_status ast = once_per_device(attr_once, [] {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&colsum_f32_rows_kernel<DTYPE, D, MAXT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        return e == hipSuccess ? KVS_OK : fail(KVS_EHIP, "kvs_attn_colsum: hipFuncSetAttribute: %s", hipGetErrorString(e));
    });
    if (ast != KVS_OK) return ast;
    hipLaunchKernelGGL((colsum_f32_rows_kernel<DTYPE, D, MAXT>), grid, dim3(kCfThreads), lds_bytes, st, n, hq, hk, q, k, scale, part);
    return check_launch("kvs_attn_colsum(f32 rows)");
}

template <int DTYPE, int D>
kvs_status launch_one_sweep(int n, int hq, int hk, const void *q, const void *k, float scale, float *part, float *alpha, hipStream_t st)
{
    const int grp = hq / hk, row_tiles = (n * grp + kCfRows - 1) / kCfRows;
    const dim3 grid((unsigned)(row_tiles * hk));
    constexpr int kFew = 4, kMost = kCfOneSweepTokens / (kCfRows * kCfWaves);
    kvs_status stt = n <= kFew * kCfRows * kCfWaves ? launch_rows<DTYPE, D, kFew>(grid, n, hq, hk, q, k, scale, part, st)
                                                    : launch_rows<DTYPE, D, kMost>(grid, n, hq, hk, q, k, scale, part, st);
    if (stt != KVS_OK) return stt;
    hipLaunchKernelGGL(colsum_f32_join, dim3((unsigned)((n + kCjKeys - 1) / kCjKeys), (unsigned)hk), dim3(kCjKeys * kCjChains), 0, st, n, grp, row_tiles,
                       (const float *)part, alpha);
    return check_launch("kvs_attn_colsum(f32)");
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

// what the row tiles' shares of the one sweep take (0: two sweeps)
static size_t one_sweep_bytes(const kvs_shape *shape, int64_t n)
{
    const int64_t row_tiles = (n * (shape->n_q_heads / shape->n_kv_heads) + kCfRows - 1) / kCfRows;
    const size_t bytes = (size_t)(row_tiles * n * shape->n_kv_heads) * sizeof(float);
    return bytes <= kCfOneSweepBytes ? bytes : 0;
}

size_t colsum_f32_workspace_bytes(const kvs_shape *shape, int64_t n)
{
    // (longer layers ask for no less: a workspace for the longest prompt serves the shorter ones)
    int64_t m = n < kCfOneSweepTokens ? n : kCfOneSweepTokens;
    while (m > 0 && one_sweep_bytes(shape, m) == 0) --m;
    return m > 0 ? one_sweep_bytes(shape, m) : 0;
}

kvs_status launch_colsum_f32(const kvs_shape *shape, int64_t n, const void *q, const void *k, float scale,
                             void *workspace, size_t workspace_bytes, float *alpha, hipStream_t st)
{
    const int d = shape->head_dim, hq = shape->n_q_heads, hk = shape->n_kv_heads;
    // quadratic work at a few percent of the bf16 matrix-core rate: refuse what would run for minutes
    if (n > 65536) return fail(KVS_EUNSUPPORTED, "kvs_attn_colsum: %lld tokens are too many for the vector path (this shape has no matrix-core kernel)", (long long)n);
    if (n * (int64_t)(hq / hk) > 0x7ffffff0) return fail(KVS_EUNSUPPORTED, "kvs_attn_colsum: %lld tokens x %d query heads", (long long)n, hq);
    const size_t shares = n <= kCfOneSweepTokens ? one_sweep_bytes(shape, n) : 0;
    const bool one = shares > 0 && shares <= workspace_bytes;
#define KVS_CF_CASE(DT, DD) (one ? launch_one_sweep<DT, DD>((int)n, hq, hk, q, k, scale, (float *)workspace, alpha, st) \
                                 : launch_both<DT, DD>((int)n, hq, hk, q, k, scale, (float2 *)workspace /* 8 bytes per query row */, alpha, st))
    if (shape->dtype == KVS_F32) return d == 64 ? KVS_CF_CASE(KVS_F32, 64) : KVS_CF_CASE(KVS_F32, 128);
    return d == 64 ? KVS_CF_CASE(KVS_BF16, 64) : KVS_CF_CASE(KVS_BF16, 128);
#undef KVS_CF_CASE
}

} // namespace kvs
