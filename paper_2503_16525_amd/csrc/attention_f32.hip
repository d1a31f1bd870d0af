// Partial-recompute attention in fp32 (Eq. (1) restricted to the selected rows): fp32 inputs, and the bf16 shapes that the
// bf16 matrix-core kernels do not cover (head_dim 64, a scale that is not positive), widened exactly.
//
// Rows are flattened (selected token, head-in-group) as in the other kernels; a workgroup owns 16 rows of one KV head and
// its eight waves deal the keys among themselves, 16 or 64 at a time, each with its own running maximum; their results meet in
// LDS at the end.  Both products run on v_mfma_f32_16x16x4_f32 (fp32 in, fp32 out): S^T = K Q^T leaves a lane with four
// keys of one query, which is the layout the second product, O^T += V^T P^T, wants its P in, so P stays in registers.
// The layers that come here are small, and what they are bound by is one chain of loads and products on a few compute units (12
// workgroups for 47 rows of 4 heads), so the keys are spread over as many waves as there are, K and Q go through LDS as
// consecutive bytes (Rows16) before their positions are known, and a lane's V values are consecutive channels: any order of the
// output's channels over the matrix rows is as good, so lane m16 has the four channels 4 m16 .. of each 64, one load for all.
//
// Measured: 47 rows of 4 heads over 512 fp32 tokens, head_dim 64: 12.3 -> 11.1 us with K and Q through LDS, V in wide loads and the
// waves' weights made once a row; 50 rows of 32:8 heads of 128, 512 tokens, 21.6 -> 17.5, 300 of 64, 3000 tokens, 273 -> 224.  (V asked for
// before the scores: the same, and 12 % slower on 1200 bf16 rows of head_dim 64.)
// (one token per workgroup, its keys in turn, dot products on the vector units: 39 us).
#include "attention.h"
#include "f32_tiles.h"

#include <math.h>

#include <type_traits>

namespace kvs {
namespace {

constexpr int kF32Waves = 8;
constexpr int kF32Threads = kF32Waves * 64;
constexpr int kF32Rows = 16;
constexpr int kF32Tiles = 4;                           // tiles of 16 keys that a wave takes at a time (one in contexts where that leaves waves without)
// Of them, in LDS together: as many as fit beside the query rows.  Of fp32 rows of 64 that leaves a compute unit one workgroup (the other kinds'
// registers do so in any case, or two have room): with two tiles together it has two, which is the faster way for launches of many workgroups,
// and of short contexts, where start and end are most of a workgroup's time.  us with four and two tiles together: 64:8 heads, 300 of 3000 tokens
// (1200 workgroups) 114 and 96, 8:8 heads, 3000 tokens, 1400, 1100 and 760 of them (704, 552, 384) 74.2 and 65.8, 57.9 and 60.8, 44.3 and
// 51.9; 4:4, 6000 tokens, 3000 and 2200 (752, 552) 143 and 126, 104 and 115; 8:8, 760 of 1250 (384) 25.1 and 26.1, 900 and 700 of 1000 (456, 352) 25.1
// and 23.2, 21.5 and 23.1, 520 of 700 (264) 15.9 and 14.6; 16:16, 300 of 500 (304) 16.2 and 12.3.
template <int DTYPE, int D>
constexpr int kF32Flight = Rows16<DTYPE, D>::BYTES <= 4096 ? 4 : 2;
template <int DTYPE, int D>
constexpr int kF32FlightShared = DTYPE == KVS_F32 && D == 64 ? 2 : kF32Flight<DTYPE, D>;
// workgroups from which on two share a unit, by the longest context
inline int64_t shared_from(int64_t max_ctx) { return max_ctx <= 768 ? 257 : max_ctx <= 1536 ? 451 : 641; }

template <int DTYPE>
__device__ __forceinline__ float load_elem(const void *p, int64_t i)
{
    if (DTYPE == KVS_F32) return ((const float *)p)[i];
    return __uint_as_float((uint32_t)((const uint16_t *)p)[i] << 16);
}

// four consecutive elements, widened
template <int DTYPE>
__device__ __forceinline__ void load_four(const void *p, int64_t i, float *x)
{
    if (DTYPE == KVS_F32) {
        const float4 v = *reinterpret_cast<const float4 *>((const float *)p + i);
        x[0] = v.x; x[1] = v.y; x[2] = v.z; x[3] = v.w;
    } else {
        const uint2 v = *reinterpret_cast<const uint2 *>((const uint16_t *)p + i);
        x[0] = bf16_lo(v.x); x[1] = bf16_hi(v.x); x[2] = bf16_lo(v.y); x[3] = bf16_hi(v.y);
    }
}

template <int DTYPE, int D, int IN_FLIGHT>
__global__ __launch_bounds__(kF32Threads, 2) void attn_f32_kernel(
    const AttnTiles td, int n_q_heads, int n_kv_heads, int total_tiles,
    const void *__restrict__ q_sel, const int32_t *__restrict__ sel_pos,
    const void *__restrict__ k_cache, const void *__restrict__ v_cache, float scale,
    void *__restrict__ out, float *__restrict__ lse_out)
{
    constexpr int DB = D / 16;                         // matrix tiles of the output: tile db, row i is channel 64 (db / 4) + 4 i + db % 4
    using Rows = Rows16<DTYPE, D>;
    extern __shared__ __attribute__((aligned(16))) char rows_s[];  // the query rows, then IN_FLIGHT tiles of keys a wave; the results afterwards
    __shared__ float m_s[kF32Waves][kF32Rows], l_s[kF32Waves][kF32Rows], x_s[kF32Waves][kF32Rows];
    const int tid = threadIdx.x, lane = tid & 63, m16 = lane & 15, kk = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.x % n_kv_heads;
    const int tile_lin = total_tiles - 1 - (int)(blockIdx.x / n_kv_heads);         // longest contexts, last rows first
    const int b = request_of(td.tile_begin, td.n_req, tile_lin);
    const int grp = n_q_heads / n_kv_heads;
    const int n_rows = td.n_sel[b] * grp, ctx_len = td.ctx_len[b];
    const int64_t sel0 = td.sel_lo[b], ctx_off = td.ctx_off[b];
    const int row0 = (tile_lin - td.tile_begin[b]) * kF32Rows;

    // this lane's query (the four lanes of a column share it)
    auto q_row = [&](int r) {
        const int rq = min(row0 + r, n_rows - 1);
        return ((sel0 + rq / grp) * n_q_heads + g * grp + rq % grp) * (int64_t)D;
    };
    const int pos = min(max(sel_pos[sel0 + min(row0 + m16, n_rows - 1) / grp], 0), ctx_len - 1);       // memory safety; the caller guarantees the range
    if (wave < Rows::LOADS) Rows::load(q_sel, q_row, rows_s, wave, lane);
    char *const mine = rows_s + Rows::BYTES * (1 + IN_FLIGHT * wave);
    // tile i of the wave's keys from k0 on (keys past `last` are clamped and not used)
    auto fetch = [&](int k0, int i, int last) {
#pragma unroll
        for (int l = 0; l < Rows::LOADS; ++l)
            Rows::load(k_cache, [&](int r) { return ((ctx_off + min(k0 + 16 * i + r, last)) * n_kv_heads + g) * (int64_t)D; }, mine + i * Rows::BYTES, l, lane);
    };
    // the first keys do not wait for the positions
    const bool small = ctx_len <= kF32Waves * 16;
    const int first_k0 = wave * 16 * (small ? 1 : kF32Tiles);
#pragma unroll
    for (int i = 0; i < IN_FLIGHT; ++i)
        if ((i == 0 || !small) && first_k0 + 16 * i < ctx_len) fetch(first_k0, i, ctx_len - 1);
    int pmin = pos, pmax = pos;
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) { pmin = min(pmin, __shfl_xor(pmin, o)); pmax = max(pmax, __shfl_xor(pmax, o)); }
    pmin = __builtin_amdgcn_readfirstlane(pmin);
    pmax = __builtin_amdgcn_readfirstlane(pmax);
    Rows::landed();                                    // (also in waves whose first keys lie past pmax: results go over them)
    __syncthreads();
    float qv[D / 4];
    Rows::read(rows_s, m16, kk, qv);

    f32x4 acc[DB];
#pragma unroll
    for (int db = 0; db < DB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_run = kLowest, l_run = 0.f;               // l_run: this lane's keys only
    // the wave's keys, TILES tiles of 16 at a time: one where that leaves no wave without (64 fp32 tokens of 8 heads of 128: 13.2 -> 9.8 us)
    auto sweep = [&](auto tiles) {
        constexpr int TILES = decltype(tiles)::value, FLIGHT = TILES < IN_FLIGHT ? TILES : IN_FLIGHT;
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
                        const int64_t vrow = ((ctx_off + min(key, pmax)) * n_kv_heads + g) * (int64_t)D + 16 * kk;
#pragma unroll
                        for (int c = 0; c < D / 4; ++c) {              // acc[c / 4][c % 4] is channel 64 (c / 16) + 16 kk + 4 (c % 4) + c / 4 % 4
                            const float v = load_elem<DTYPE>(v_cache, vrow + 64 * (c >> 4) + 4 * (c & 3) + (c >> 2 & 3));
                            if (key <= pos && !(fabsf(v) < INFINITY)) acc[c >> 2][c & 3] += p * v;
                        }
                    }
                }
            };
#pragma unroll
            for (int t0 = 0; t0 < TILES; t0 += FLIGHT) {
                if (k0 != first_k0 || t0 > 0) {
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // what lay there has been read
#pragma unroll
                    for (int i = 0; i < FLIGHT; ++i) fetch(k0 + 16 * t0, i, pmax);
                    Rows::landed();
                }
#pragma unroll
                for (int i = 0; i < FLIGHT; ++i) {
                    float kv[D / 4];
                    Rows::read(mine + i * Rows::BYTES, m16, kk, kv);
                    s[t0 + i] = dots<D>(kv, qv);
                }
            }
#pragma unroll
            for (int t = 0; t < TILES; ++t) {
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
                    const int key = min(k0 + 16 * t + 4 * kk + r, pmax);       // (nothing past the last row's position is read)
                    const int64_t vrow = ((ctx_off + key) * n_kv_heads + g) * (int64_t)D + 4 * m16;
#pragma unroll
                    for (int db = 0; db < DB; db += 4) load_four<DTYPE>(v_cache, vrow + 16 * db, &v[r][db]);
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
    if (pmax < kF32Waves * 16) sweep(std::integral_constant<int, 1>{});      // (by the rows' reach: all but wave 0 ask again in a long context)
    else sweep(std::integral_constant<int, kF32Tiles>{});
    l_run += __shfl_xor(l_run, 16);
    l_run += __shfl_xor(l_run, 32);
    if (kk == 0) { m_s[wave][m16] = m_run; l_s[wave][m16] = l_run; }
    // the waves' shares in wave order: their weights, one a thread, then four channels of a row a thread
    float *const o_s = reinterpret_cast<float *>(rows_s);          // [waves][rows][64 + 4], over the keys
    constexpr int OC = 64, OP = OC + 4;                            // channels that meet in LDS at a time, and a row's pitch
#pragma unroll
    for (int c0 = 0; c0 < D; c0 += OC) {
        __syncthreads();                                           // the keys, or the channels before, have been read
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *reinterpret_cast<f32x4 *>(o_s + (wave * kF32Rows + m16) * OP + 16 * kk + 4 * r) =
                f32x4{acc[c0 / 16][r], acc[c0 / 16 + 1][r], acc[c0 / 16 + 2][r], acc[c0 / 16 + 3][r]};
        if (c0 == 0 && tid < kF32Waves * kF32Rows) {
            const int w = tid / kF32Rows, r = tid % kF32Rows;
            float mt = m_s[0][r];
#pragma unroll
            for (int v = 1; v < kF32Waves; ++v) mt = fmaxf(mt, m_s[v][r]);
            x_s[w][r] = expf(m_s[w][r] - mt);
        }
        __syncthreads();
        const int r = tid / (OC / 4), c = tid % (OC / 4) * 4;
        if (r >= kF32Rows || row0 + r >= n_rows) continue;
        float l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kF32Waves; ++w) {
            const float x = x_s[w][r];
            const f32x4 ow = *reinterpret_cast<const f32x4 *>(o_s + (w * kF32Rows + r) * OP + c);
            l += x * l_s[w][r];
#pragma unroll
            for (int u = 0; u < 4; ++u) o[u] += x * ow[u];
        }
        const int64_t orow = (sel0 + (row0 + r) / grp) * n_q_heads + g * grp + (row0 + r) % grp, at = orow * D + c0 + c;
        if (DTYPE == KVS_F32) {
            *reinterpret_cast<f32x4 *>((float *)out + at) = f32x4{o[0] / l, o[1] / l, o[2] / l, o[3] / l};
        } else {
            uint2 w2;
            w2.x = f32_to_bf16_bits(o[0] / l) | f32_to_bf16_bits(o[1] / l) << 16;
            w2.y = f32_to_bf16_bits(o[2] / l) | f32_to_bf16_bits(o[3] / l) << 16;
            *reinterpret_cast<uint2 *>((uint16_t *)out + at) = w2;
        }
        if (lse_out && c0 + c == 0) {
            float mt = m_s[0][r];
#pragma unroll
            for (int w = 1; w < kF32Waves; ++w) mt = fmaxf(mt, m_s[w][r]);
            lse_out[orow] = mt + logf(l);
        }
    }
}

template <int DTYPE, int D, int IN_FLIGHT>
kvs_status launch_f32(dim3 grid, const AttnTiles &td, const kvs_shape *shape, int tiles, const void *q_sel, const int32_t *sel_pos,
                      const void *k_cache, const void *v_cache, float scale, void *out, float *lse_out, hipStream_t st)
{
    using Rows = Rows16<DTYPE, D>;
    static_assert(Rows::LOADS <= kF32Waves, "a wave loads one share of the query rows");
    constexpr int keys = Rows::BYTES * (1 + IN_FLIGHT * kF32Waves), results = kF32Waves * kF32Rows * (64 + 4) * (int)sizeof(float);
    constexpr int lds_bytes = keys > results ? keys : results;
    static DeviceOnce attr_once;
    const kvs_status ast = once_per_device(attr_once, [] {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&attn_f32_kernel<DTYPE, D, IN_FLIGHT>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes);
        return e == hipSuccess ? KVS_OK : fail(KVS_EHIP, "kvs_partial_attention: hipFuncSetAttribute: %s", hipGetErrorString(e));
    });
    if (ast != KVS_OK) return ast;
    hipLaunchKernelGGL((attn_f32_kernel<DTYPE, D, IN_FLIGHT>), grid, dim3(kF32Threads), lds_bytes, st, td, shape->n_q_heads, shape->n_kv_heads, tiles,
                       q_sel, sel_pos, k_cache, v_cache, scale, out, lse_out);
    return check_launch("kvs_partial_attention(f32)");
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
    const dim3 grid((unsigned)(tiles * shape->n_kv_heads));
    int64_t max_ctx = 0;
    for (int i = 0; i < bd.n_req; ++i) max_ctx = bd.ctx_len[i] > max_ctx ? bd.ctx_len[i] : max_ctx;
    const bool shared = (int64_t)grid.x >= shared_from(max_ctx);
#define KVS_ATT_CASE_(DT, DD, FL) launch_f32<DT, DD, FL>(grid, td, shape, (int)tiles, q_sel, sel_pos, k_cache, v_cache, scale, out, lse_out, st)
#define KVS_ATT_CASE(DT, DD) return shared ? KVS_ATT_CASE_(DT, DD, (kF32FlightShared<DT, DD>)) : KVS_ATT_CASE_(DT, DD, (kF32Flight<DT, DD>))
    if (shape->dtype == KVS_F32 && shape->head_dim == 64) KVS_ATT_CASE(KVS_F32, 64);
    if (shape->dtype == KVS_F32 && shape->head_dim == 128) KVS_ATT_CASE(KVS_F32, 128);
    if (shape->dtype == KVS_BF16 && shape->head_dim == 64) KVS_ATT_CASE(KVS_BF16, 64);
    if (shape->dtype == KVS_BF16 && shape->head_dim == 128) KVS_ATT_CASE(KVS_BF16, 128);
#undef KVS_ATT_CASE
#undef KVS_ATT_CASE_
    return fail(KVS_EUNSUPPORTED, "kvs_partial_attention: head_dim %d", shape->head_dim);
}

} // namespace kvs
