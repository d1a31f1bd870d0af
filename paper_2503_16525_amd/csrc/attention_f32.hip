// Partial-recompute attention in fp32 (Eq. (1) restricted to the selected rows): fp32 inputs, and the bf16 shapes that the
// bf16 matrix-core kernels do not cover (head_dim 64, a scale that is not positive), widened exactly.
//
// Rows are flattened (selected token, head-in-group) as in the other kernels; a workgroup owns 16 rows of one KV head and
// its eight waves deal the keys among themselves, 16 or 64 at a time, each with its own running maximum; their results meet in
// LDS at the end.  Both products run on v_mfma_f32_16x16x4_f32 (fp32 in, fp32 out): S^T = K Q^T leaves a lane with four
// keys of one query, which is the layout the second product, O^T += V^T P^T, wants its P in, so P stays in registers.
// Operands come straight from global memory: the layers that come here are small, and what they are bound by is the
// latency of one chain of loads and products, so the keys are spread over as many waves as there are.
//
// Measured: 47 rows of 4 heads over 512 fp32 tokens, head_dim 64: 39 -> 12.4 us (before: one token per workgroup, its
// keys in turn, dot products on the vector units).
#include "attention.h"
#include "f32_tiles.h"

#include <math.h>

#include <type_traits>

namespace kvs {
namespace {

constexpr int kF32Waves = 8;
constexpr int kF32Threads = kF32Waves * 64;
constexpr int kF32Rows = 16;

template <int DTYPE>
__device__ __forceinline__ float load_elem(const void *p, int64_t i)
{
    if (DTYPE == KVS_F32) return ((const float *)p)[i];
    return __uint_as_float((uint32_t)((const uint16_t *)p)[i] << 16);
}

template <int DTYPE, int D>
__global__ __launch_bounds__(kF32Threads, 2) void attn_f32_kernel(
    const AttnTiles td, int n_q_heads, int n_kv_heads, int total_tiles,
    const void *__restrict__ q_sel, const int32_t *__restrict__ sel_pos,
    const void *__restrict__ k_cache, const void *__restrict__ v_cache, float scale,
    void *__restrict__ out, float *__restrict__ lse_out)
{
    constexpr int DB = D / 16;                         // 16-channel blocks of the output
    __shared__ float m_s[kF32Waves][kF32Rows], l_s[kF32Waves][kF32Rows];
    constexpr int OC = 64;                             // channels that meet in LDS at a time
    __shared__ float o_s[kF32Waves][kF32Rows][OC + 4];
    const int tid = threadIdx.x, lane = tid & 63, m16 = lane & 15, kk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x % n_kv_heads;
    const int tile_lin = total_tiles - 1 - (int)(blockIdx.x / n_kv_heads);         // longest contexts, last rows first
    int b = 0;
    while (b + 1 < td.n_req && tile_lin >= td.tile_begin[b + 1]) ++b;
    const int grp = n_q_heads / n_kv_heads;
    const int n_rows = td.n_sel[b] * grp, ctx_len = td.ctx_len[b];
    const int64_t sel0 = td.sel_lo[b], ctx_off = td.ctx_off[b];
    const int row0 = (tile_lin - td.tile_begin[b]) * kF32Rows;

    // this lane's query (the four lanes of a column share it)
    const int rq = min(row0 + m16, n_rows - 1);
    const int64_t s_glob = sel0 + rq / grp;
    const int head = g * grp + rq % grp;
    const int pos = min(max(sel_pos[s_glob], 0), ctx_len - 1);       // memory safety; the caller guarantees the range
    float qv[D / 4];
    load_quarter<DTYPE, D>(q_sel, (s_glob * n_q_heads + head) * (int64_t)D, kk, qv);
    int pmin = pos, pmax = pos;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) { pmin = min(pmin, __shfl_xor(pmin, o)); pmax = max(pmax, __shfl_xor(pmax, o)); }
    pmin = __builtin_amdgcn_readfirstlane(pmin);
    pmax = __builtin_amdgcn_readfirstlane(pmax);

    f32x4 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = kLowest, l_run = 0.f;               // l_run: this lane's keys only
    // the wave's keys, TILES tiles of 16 at a time: one where that leaves no wave without (64 fp32 tokens of 8 heads of 128: 13.2 -> 9.8 us)
    auto sweep = [&](auto tiles) {
        constexpr int TILES = decltype(tiles)::value;
        for (int k0 = wave * 16 * TILES; k0 <= pmax; k0 += kF32Waves * 16 * TILES) {
            f32x4 s[TILES];
            float mx = -INFINITY;
            // tile t's Inf and NaN values, which its products leave out: to the rows that see their keys (rare and slow)
            auto add_odd_values = [&](int t) {
#pragma unroll 1
                for (int kq = 0; kq < 4; ++kq) {
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int key = k0 + 16 * t + 4 * kq + r;
                        const float p = __shfl(s[t][r], 16 * kq + m16);
                        const int64_t vrow = ((ctx_off + min(key, pmax)) * n_kv_heads + g) * (int64_t)D + 4 * kk;
#pragma unroll
                        for (int c = 0; c < D / 4; ++c) {              // acc[c / 4][c % 4] is channel 16 (c / 4) + 4 kk + c % 4
                            const float v = load_elem<DTYPE>(v_cache, vrow + 16 * (c >> 2) + (c & 3));
                            if (key <= pos && !(fabsf(v) < INFINITY)) acc[c >> 2][c & 3] += p * v;
                        }
                    }
                }
            };
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
                float kv[D / 4];
                const int key = min(k0 + 16 * t + m16, pmax);          // (nothing past the last row's position is read)
                load_quarter<DTYPE, D>(k_cache, ((ctx_off + key) * n_kv_heads + g) * (int64_t)D, kk, kv);
                s[t] = dots<D>(kv, qv);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    s[t][r] = k0 + 16 * t + 4 * kk + r <= pos ? s[t][r] * scale : -INFINITY;
                    mx = fmaxf(mx, s[t][r]);
                }
            }
            mx = fmaxf(mx, __shfl_xor(mx, 16));
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            const float m_new = fmaxf(m_run, mx);          // finite: a column that sees no key here keeps its own
            const float corr = expf(m_run - m_new);
            m_run = m_new;
            l_run *= corr;
#pragma unroll
            for (int db = 0; db < DB; ++db) acc[db] *= corr;
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
#pragma unroll
                for (int r = 0; r < 4; ++r) { s[t][r] = expf(s[t][r] - m_new); l_run += s[t][r]; }
                // instruction r contracts over keys 4 kk + r of the tile, kk = 0 .. 3
                const bool all_seen = k0 + 16 * t + 15 <= pmin;        // uniform: every row sees every key of the tile
                float v[4][DB];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int key = min(k0 + 16 * t + 4 * kk + r, pmax);
                    const int64_t vrow = ((ctx_off + key) * n_kv_heads + g) * (int64_t)D + m16;
#pragma unroll
                    for (int db = 0; db < DB; ++db) v[r][db] = load_elem<DTYPE>(v_cache, vrow + 16 * db);
                }
                bool odd = false;
                if (!all_seen) {
                    // a weight of 0 does not hide an Inf or NaN from a row that does not see the key
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int db = 0; db < DB; ++db) odd |= !(fabsf(v[r][db]) < INFINITY);
                    if (__any(odd)) {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
#pragma unroll
                            for (int db = 0; db < DB; ++db) v[r][db] = fabsf(v[r][db]) < INFINITY ? v[r][db] : 0.f;
                    }
                }
#pragma unroll
                for (int r = 0; r < 4; ++r)
#pragma unroll
                    for (int db = 0; db < DB; ++db) acc[db] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[r][db], s[t][r], acc[db], 0, 0, 0);
                if (!all_seen && __any(odd)) add_odd_values(t);
            }
        }
    };
    if (pmax < kF32Waves * 16) sweep(std::integral_constant<int, 1>{});
    else sweep(std::integral_constant<int, 4>{});
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    if (kk == 0) { m_s[wave][m16] = m_run; l_s[wave][m16] = l_run; }
    // the waves' shares in wave order
#pragma unroll
    for (int c0 = 0; c0 < D; c0 += OC) {
        if (c0 > 0) __syncthreads();
#pragma unroll
        for (int db = 0; db < OC / 16; ++db) *reinterpret_cast<f32x4 *>(&o_s[wave][m16][16 * db + 4 * kk]) = acc[c0 / 16 + db];
        __syncthreads();
        for (int e = tid; e < kF32Rows * OC; e += kF32Threads) {
            const int r = e / OC, c = e % OC;
            if (row0 + r >= n_rows) continue;
            float mt = m_s[0][r];
#pragma unroll
            for (int w = 1; w < kF32Waves; ++w) mt = fmaxf(mt, m_s[w][r]);
            float l = 0.f, o = 0.f;
#pragma unroll
            for (int w = 0; w < kF32Waves; ++w) {
                const float x = expf(m_s[w][r] - mt);
                l += x * l_s[w][r];
                o += x * o_s[w][r][c];
            }
            const int64_t orow = (sel0 + (row0 + r) / grp) * n_q_heads + g * grp + (row0 + r) % grp;
            if (DTYPE == KVS_F32) ((float *)out)[orow * D + c0 + c] = o / l;
            else ((uint16_t *)out)[orow * D + c0 + c] = (uint16_t)f32_to_bf16_bits(o / l);
            if (lse_out && c0 + c == 0) lse_out[orow] = mt + logf(l);
        }
    }
}

} // namespace

kvs_status launch_attention_f32(const kvs_shape *shape, const AttnBatch &bd, int64_t n_sel,
                                const void *q_sel, const int32_t *sel_pos, const void *k_cache,
                                const void *v_cache, float scale, void *out, float *lse_out,
                                hipStream_t st)
{
    if (n_sel == 0) return KVS_OK;
    AttnTiles td;
    const int64_t tiles = build_attn_tiles(shape, bd, kF32Rows, td);
    if (tiles < 0) return fail(KVS_EINVAL, "kvs_partial_attention: too many row tiles");
    if (tiles == 0) return KVS_OK;
    const dim3 grid((unsigned)(tiles * shape->n_kv_heads)), block(kF32Threads);
#define KVS_ATT_CASE(DT, DD)                                                                              \
    hipLaunchKernelGGL((attn_f32_kernel<DT, DD>), grid, block, 0, st, td, shape->n_q_heads,                \
                       shape->n_kv_heads, (int)tiles, q_sel, sel_pos, k_cache, v_cache, scale, out, lse_out)
    if (shape->dtype == KVS_F32 && shape->head_dim == 64) KVS_ATT_CASE(KVS_F32, 64);
    else if (shape->dtype == KVS_F32 && shape->head_dim == 128) KVS_ATT_CASE(KVS_F32, 128);
    else if (shape->dtype == KVS_BF16 && shape->head_dim == 64) KVS_ATT_CASE(KVS_BF16, 64);
    else if (shape->dtype == KVS_BF16 && shape->head_dim == 128) KVS_ATT_CASE(KVS_BF16, 128);
    else return fail(KVS_EUNSUPPORTED, "kvs_partial_attention: head_dim %d", shape->head_dim);
#undef KVS_ATT_CASE
    return check_launch("kvs_partial_attention(f32)");
}

} // namespace kvs
