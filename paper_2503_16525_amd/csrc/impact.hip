// kvs_first_order_impact: the first-order expansion of the attention output's deviation (Sec. 4.1,
// Eq. (2)), token by token.  Reusing token i's cache entry moves output row j of query head h by
//     A[h,j,i] * dV[g,i]                                             value direction (dH/dV = A)
//   + A[h,j,i] * scale * (q[j,h] . dK[g,i]) * (V[g,i] - H[h,j])      key direction (softmax Jacobian)
// and the token's impact is the L1 norm of that movement over all rows j >= i, heads and channels,
// for the value term alone (which is Eq. (3): column mass times |dV|_1), the key term alone, and
// both together.  The paper drops the key term "to reduce computational overhead": unlike the value
// term it does not separate into (something of i) x (something of j) -- every (row, token) pair
// needs its own L1 norm over the channels -- so this is N^2/2 * H_q * d work on the vector units; only the
// two dot products per pair and, for bf16, the differences inside the norm are contractions for the matrix
// cores.  It is a diagnostic for check layers, not a step of the hot path.
//
// bf16 (impact_tiles_kernel).  Per (row, token, channel) there are a subtraction, v - h, its absolute sum, fma(t, v - h, dv)
// and its absolute sum, with a = A[h,j,i] and t = scale * (q . dK) entering once per pair.  The subtraction is a product: over a
// tile of rows x tokens v - h = [-h, 1] . [1, v], a contraction of two that bf16 operands enter exactly.  So the matrix cores make
// it beside the vector units, which are left with three instructions per term and bound the kernel:
//   * only reused tokens are rated: a list of them is made first, and a workgroup takes 32 consecutive entries, whose K, V and dV
//     it keeps in LDS;
//   * a wave takes 32 flattened (row, head) pairs at a time, alone (no barrier in the sweep): q . K_fresh and q . K_cache (exact bf16
//     operands; their difference is q . dK) on the matrix cores, then channel by channel one 32x32x8 MFMA for the differences
//     and 48 vector instructions on its 16 results a lane.  The row's H is an operand as it lies in memory, four channels at
//     a time; the other operand picks one of them (-1 in its slot, zeros beside it).  The fp32 instruction of the same
//     shape takes twice the matrix time and gained nothing (9.9 ms: vector work does not run beside all of it);
//   * the rows are cut into pieces so that the triangle of (row, token) pairs spreads evenly over the chip.
// Measured against four vector instructions a term (lanes are tokens, a wave 32 channels, H through LDS, barriers): Qwen-shaped 8192
// tokens (80 % reused) 10.2 -> 7.5 ms, 7300 Llama-shaped 8.8 -> 7.2, 1963 0.77 -> 0.68, 526 Qwen-shaped 68 -> 58 us, 256 Yi-shaped 41 -> 33.
//
// fp32 (impact_kernel): one workgroup owns 32 tokens (columns) of one KV head: their K, dK, V, dV rows sit in LDS,
// channel-major so that the 32 column lanes of a wave hit 32 banks.  Rows stream past in blocks of 64 flattened (query
// row, head-in-group) pairs, staged in LDS with their output rows H; thread (column c, row lane r) handles four pairs at
// a time: first the two dot products per pair, then the channel loop of the L1 norms.
//
// Sums are kept per thread in a fixed order and added in a fixed order at the end: bit-reproducible.  Per-head partial
// sums go to the workspace; a second kernel adds them and applies the mask.
#include "kvs_internal.h"

#include <math.h>

namespace kvs {
namespace {

constexpr int kImpCols = 32;                 // tokens per workgroup
constexpr int kImpRowLanes = 16;
constexpr int kImpThreads = kImpCols * kImpRowLanes;    // 512
constexpr int kImpPairs = 4;                 // (row, head) pairs a thread handles at a time: a column value read from LDS serves all of them
constexpr int kImpBlock = kImpRowLanes * kImpPairs;      // 64 pairs staged per block

// grid: (column tiles, heaviest first) x kv heads
template <int D>
__global__ __launch_bounds__(kImpThreads) void impact_kernel(
    int n, int n_q_heads, int n_kv_heads,
    const float *__restrict__ q, const float *__restrict__ k_fresh, const float *__restrict__ v_fresh,
    const float *__restrict__ k_cache, const float *__restrict__ v_cache,
    const float *__restrict__ h_fresh, const float *__restrict__ lse, float scale,
    float *__restrict__ part /* [3][n_kv_heads][n]: value, key, both */)
{
    extern __shared__ float lds[];
    float *colV = lds;                        // [D][kImpCols]
    float *colDV = colV + D * kImpCols;
    float *colK = colDV + D * kImpCols;
    float *colDK = colK + D * kImpCols;
    float *rowH = colDK + D * kImpCols;       // [kImpBlock][D]
    float *rowQ = rowH + kImpBlock * D;
    float *rowL = rowQ + kImpBlock * D;       // [kImpBlock] lse; [kImpBlock] row index follows
    int *rowJ = reinterpret_cast<int *>(rowL + kImpBlock);
    float *red = reinterpret_cast<float *>(rowJ + kImpBlock);   // [3][kImpRowLanes][kImpCols]

    const int tid = threadIdx.x, col = tid % kImpCols, rl = tid / kImpCols;
    const int g = blockIdx.y;
    const int grp = n_q_heads / n_kv_heads;
    const int i0 = blockIdx.x * kImpCols;                  // first token of this workgroup (low tiles have the most rows)
    const int i = i0 + col;
    // ---- the tile's columns into LDS ----
    for (int e = tid; e < kImpCols * D; e += kImpThreads) {
        const int c = e % D, t = e / D;                    // consecutive threads read consecutive channels of a token
        const int tok = min(i0 + t, n - 1);
        const int64_t at = ((int64_t)tok * n_kv_heads + g) * D + c;
        const float kf = k_fresh[at], vf = v_fresh[at];
        colK[c * kImpCols + t] = kf;
        colDK[c * kImpCols + t] = k_cache[at] - kf;
        colV[c * kImpCols + t] = vf;
        colDV[c * kImpCols + t] = v_cache[at] - vf;
    }
    __syncthreads();
    float dv_l1 = 0.f;                                     // |dV_i|_1, fixed order
    for (int c = 0; c < D; ++c) dv_l1 += fabsf(colDV[c * kImpCols + col]);

    float acc_a = 0.f, acc_k = 0.f, acc_kv = 0.f;          // sum of A, key-term norm, combined norm for (column, row lane)
    const int64_t n_pairs = (int64_t)(n - i0) * grp;       // flattened (row j >= i0, head in group)
    for (int64_t p0 = 0; p0 < n_pairs; p0 += kImpBlock) {
        __syncthreads();                                    // the block before has been consumed
        for (int e = tid; e < kImpBlock * D; e += kImpThreads) {
            const int c = e % D, r = e / D;
            const int64_t p = min(p0 + r, n_pairs - 1);
            const int j = i0 + (int)(p / grp), h = g * grp + (int)(p % grp);
            const int64_t at = ((int64_t)j * n_q_heads + h) * D + c;
            rowQ[r * D + c] = q[at];
            rowH[r * D + c] = h_fresh[at];
        }
        if (tid < kImpBlock) {
            const int64_t p = p0 + tid;
            const int64_t pc = min(p, n_pairs - 1);
            const int j = i0 + (int)(pc / grp), h = g * grp + (int)(pc % grp);
            rowL[tid] = lse[(int64_t)j * n_q_heads + h];
            rowJ[tid] = p < n_pairs ? j : -1;              // -1: past the end, contributes nothing
        }
        __syncthreads();
        float s[kImpPairs], ds[kImpPairs];
#pragma unroll
        for (int u = 0; u < kImpPairs; ++u) { s[u] = 0.f; ds[u] = 0.f; }
#pragma unroll 4
        for (int c = 0; c < D; c += 4) {
            float4 qv[kImpPairs];
#pragma unroll
            for (int u = 0; u < kImpPairs; ++u) qv[u] = *reinterpret_cast<const float4 *>(&rowQ[(rl * kImpPairs + u) * D + c]);
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const float kk = colK[(c + cc) * kImpCols + col], dk = colDK[(c + cc) * kImpCols + col];
#pragma unroll
                for (int u = 0; u < kImpPairs; ++u) {
                    const float qe = cc == 0 ? qv[u].x : cc == 1 ? qv[u].y : cc == 2 ? qv[u].z : qv[u].w;
                    s[u] = fmaf(qe, kk, s[u]);
                    ds[u] = fmaf(qe, dk, ds[u]);
                }
            }
        }
        // With a = A[h,j,i] and t = scale * (q . dK), the pair moves output row (j, h) by a * (dV + t * (V - H)):
        // |key term|_1 = a |t| * sum_c |V_c - H_c| and |both|_1 = a * sum_c |dV_c + t (V_c - H_c)|, so the channel
        // loop needs a subtraction, an fma and two |.|-adds per channel and the pair's weights enter once at the end.
        float a[kImpPairs], t[kImpPairs];
#pragma unroll
        for (int u = 0; u < kImpPairs; ++u) {
            const int r = rl * kImpPairs + u;
            const int j = rowJ[r];
            const bool live = j >= i && i < n;             // causal: row j sees token i; rows past the end carry -1
            a[u] = live ? __expf(scale * s[u] - rowL[r]) : 0.f;
            t[u] = scale * ds[u];
            acc_a += a[u];
        }
        float nk[kImpPairs], nkv[kImpPairs];
#pragma unroll
        for (int u = 0; u < kImpPairs; ++u) { nk[u] = 0.f; nkv[u] = 0.f; }
#pragma unroll 4
        for (int c = 0; c < D; c += 4) {
            float4 hv[kImpPairs];
#pragma unroll
            for (int u = 0; u < kImpPairs; ++u) hv[u] = *reinterpret_cast<const float4 *>(&rowH[(rl * kImpPairs + u) * D + c]);
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const float vv = colV[(c + cc) * kImpCols + col], dv = colDV[(c + cc) * kImpCols + col];
#pragma unroll
                for (int u = 0; u < kImpPairs; ++u) {
                    const float he = cc == 0 ? hv[u].x : cc == 1 ? hv[u].y : cc == 2 ? hv[u].z : hv[u].w;
                    const float dd = vv - he;
                    nk[u] += fabsf(dd);
                    nkv[u] += fabsf(fmaf(t[u], dd, dv));
                }
            }
        }
#pragma unroll
        for (int u = 0; u < kImpPairs; ++u) { acc_k += a[u] * fabsf(t[u]) * nk[u]; acc_kv += a[u] * nkv[u]; }
    }
    // ---- the 16 row lanes of each column, added in lane order ----
    red[(0 * kImpRowLanes + rl) * kImpCols + col] = acc_a;
    red[(1 * kImpRowLanes + rl) * kImpCols + col] = acc_k;
    red[(2 * kImpRowLanes + rl) * kImpCols + col] = acc_kv;
    __syncthreads();
    if (rl == 0 && i < n) {
        float sa = 0.f, sk = 0.f, skv = 0.f;
        for (int r = 0; r < kImpRowLanes; ++r) {
            sa += red[(0 * kImpRowLanes + r) * kImpCols + col];
            sk += red[(1 * kImpRowLanes + r) * kImpCols + col];
            skv += red[(2 * kImpRowLanes + r) * kImpCols + col];
        }
        const int64_t o = (int64_t)g * n + i, stride = (int64_t)n_kv_heads * n;
        part[o] = sa * dv_l1;             // value direction: (sum of A over rows and heads of the group) * |dV|_1
        part[stride + o] = sk;
        part[2 * stride + o] = skv;
    }
}

// ---- bf16: the reused tokens' list -------------------------------------------------------------------------------
// list[0 .. count) = positions with reused != 0, ascending; one workgroup, every thread a contiguous share
constexpr int kListThreads = 1024;
__global__ __launch_bounds__(kListThreads) void impact_list_kernel(int n, const uint8_t *__restrict__ reused, int32_t *__restrict__ list,
                                                                   int32_t *__restrict__ count)
{
    __shared__ int tot[kListThreads / kWave];
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int per = (n + kListThreads - 1) / kListThreads, a = min(n, tid * per), e = min(n, a + per);
    int mine = 0;
    for (int i = a; i < e; ++i) mine += reused[i] != 0;
    int incl = mine;
    for (int o = 1; o < kWave; o <<= 1) {
        const int up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    if (lane == kWave - 1) tot[wave] = incl;
    __syncthreads();
    int at = incl - mine;
    for (int w = 0; w < wave; ++w) at += tot[w];
    for (int i = a; i < e; ++i)
        if (reused[i] != 0) list[at++] = i;
    if (tid == kListThreads - 1) *count = at;
}

// ---- bf16: 32 tokens of the list x one piece of the rows ----------------------------------------------------------
typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 imp_bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float imp_floatx16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short imp_s16x4;
constexpr int kTileCols = 32, kTileRows = 32, kTileThreads = 256, kTileWaves = kTileThreads / kWave;

// a token's row in LDS is an odd number of 16-byte pieces: the reads of eight lanes meet no bank twice
template <int D>
constexpr int tile_ld_v() { return D + 2; }
template <int D>
constexpr int tile_ld_dv() { return D + 4; }
template <int D>
constexpr int tile_lds_bytes() { return 2 * kTileCols * D * 2 + kTileCols * (tile_ld_v<D>() * 8 + tile_ld_dv<D>() * 4) + D * 8; }

// sum += x, the rounding error carried along (a lane adds tens of thousands of rows); an infinite sum stays infinite
__device__ __forceinline__ void add_carried(float &sum, float &carry, float x)
{
    const float y = x - carry, t = sum + y;
    carry = fabsf(t) < INFINITY ? (t - sum) - y : 0.f;
    sum = t;
}

template <int D>
__global__ __launch_bounds__(kTileThreads, 2) void impact_tiles_kernel(
    int n, int n_q_heads, int n_kv_heads, int rows_per_piece,
    const uint16_t *__restrict__ q, const uint16_t *__restrict__ k_fresh, const uint16_t *__restrict__ v_fresh,
    const uint16_t *__restrict__ k_cache, const uint16_t *__restrict__ v_cache,
    const uint16_t *__restrict__ h_fresh, const float *__restrict__ lse, float scale,
    const int32_t *__restrict__ list /* NULL: every token */, const int32_t *__restrict__ count,
    float *__restrict__ part /* [pieces][3][n_kv_heads][n]: value, key, both */)
{
    constexpr int PIECES = D / 8;                            // 16-byte pieces of a bf16 row
    constexpr int LDV = tile_ld_v<D>(), LDD = tile_ld_dv<D>();
    extern __shared__ __attribute__((aligned(16))) char ilds[];
    uint64_t *colV = reinterpret_cast<uint64_t *>(ilds);     // [32][LDV]: channel c in 16-bit slot c & 3, zeros beside it
    uint64_t *minus = colV + kTileCols * LDV;                // [D]: -1 likewise
    float *colDV = reinterpret_cast<float *>(minus + D);     // [32][LDD]
    uint16_t *colKf = reinterpret_cast<uint16_t *>(colDV + kTileCols * LDD);            // [32][D], pieces XOR-swizzled by the row
    uint16_t *colKc = colKf + kTileCols * D;

    const int tid = threadIdx.x, lane = tid & 63, ln = tid & 31, hf = (tid >> 5) & 1;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g = blockIdx.y, piece = blockIdx.z;
    const int grp = n_q_heads / n_kv_heads;
    const int n_cols = list ? *count : n;
    const int l0 = blockIdx.x * kTileCols;
    if (l0 >= n_cols) return;                                // uniform; these columns are nobody's
    auto token = [&](int c) { const int l = min(l0 + c, n_cols - 1); return list ? list[l] : l; };
    const int i = token(ln);
    const bool col_ok = l0 + ln < n_cols;
    const int i0 = __builtin_amdgcn_readfirstlane(i), i_last = __builtin_amdgcn_readlane(i, min(kTileCols, n_cols - l0) - 1);
    // rows j of this piece that the first (lowest) token can be seen by
    const int j0 = max(i0, piece * rows_per_piece), j1 = min(n, (piece + 1) * rows_per_piece);
    const int64_t stride = (int64_t)n_kv_heads * n, o = 3 * stride * piece + (int64_t)g * n + i;
    if (j0 >= j1) {
        if (tid < kTileCols && col_ok) { part[o] = 0.f; part[o + stride] = 0.f; part[o + 2 * stride] = 0.f; }
        return;
    }
    for (int e = tid; e < kTileCols * PIECES; e += kTileThreads) {
        const int pc = e % PIECES, t = e / PIECES;
        const int64_t from = ((int64_t)token(t) * n_kv_heads + g) * D + 8 * pc;
        const int dst = t * D + 8 * (pc ^ (t & (PIECES - 1)));
        *reinterpret_cast<uint4 *>(colKf + dst) = *reinterpret_cast<const uint4 *>(k_fresh + from);
        *reinterpret_cast<uint4 *>(colKc + dst) = *reinterpret_cast<const uint4 *>(k_cache + from);
        const uint4 f = *reinterpret_cast<const uint4 *>(v_fresh + from), x = *reinterpret_cast<const uint4 *>(v_cache + from);
        const uint32_t fw[4] = {f.x, f.y, f.z, f.w}, xw[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float v0 = bf16_lo(fw[u]), v1 = bf16_hi(fw[u]);
            *reinterpret_cast<ulonglong2 *>(colV + t * LDV + 8 * pc + 2 * u) = make_ulonglong2((uint64_t)(fw[u] & 0xffffu) << (u & 1 ? 32 : 0),
                                                                                            (uint64_t)(fw[u] & 0xffff0000u) << (u & 1 ? 32 : 0));
            *reinterpret_cast<float2 *>(colDV + t * LDD + 8 * pc + 2 * u) = make_float2(bf16_lo(xw[u]) - v0, bf16_hi(xw[u]) - v1);
        }
    }
    for (int e = tid; e < D; e += kTileThreads) minus[e] = (uint64_t)0xbf80u << (16 * (e & 3));
    __syncthreads();

    // v - h of one channel, 32 rows x 32 tokens, is a product over the lower half-wave's four slots of the contraction (four channels
    // of the row's H with -1 in one of them) and the upper one's (ones with the token's V in the same slot)
    const uint64_t *b_from = hf ? colV + ln * LDV : minus;
    const float *dv_from = colDV + ln * LDD;
    const uint32_t n_pairs = (uint32_t)(j1 - j0) * (uint32_t)grp;          // flattened (row, head in group)
    const int my_token = col_ok ? i : 0x7fffffff;            // out of reach if the column has none
    float sum_a = 0.f, sum_k = 0.f, sum_kv = 0.f, carry_a = 0.f, carry_k = 0.f, carry_kv = 0.f;
    for (uint32_t p0 = (uint32_t)(wave * kTileRows); p0 < n_pairs; p0 += kTileWaves * kTileRows) {
        const uint32_t p = min(p0 + (uint32_t)ln, n_pairs - 1), jr = p / (uint32_t)grp;
        const int64_t row = (int64_t)(j0 + (int)jr) * n_q_heads + g * grp + (int)(p - jr * (uint32_t)grp);
        const float row_lse = lse[row];
        const int row_j = p0 + (uint32_t)ln < n_pairs ? j0 + (int)jr : -1;                // -1: past the end, contributes nothing
        const uint4 *q_from = reinterpret_cast<const uint4 *>(q + row * D) + hf, *h_from = reinterpret_cast<const uint4 *>(h_fresh + row * D);
        uint4 qa[D / 16], h[PIECES];
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qa[ks] = q_from[2 * ks];
#pragma unroll
        for (int c8 = 0; c8 < PIECES; ++c8) {
            h[c8] = make_uint4(0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u);
            if (hf == 0) h[c8] = h_from[c8];
        }
        // 32 rows x 32 tokens; entry e of a lane is row 8 (e >> 2) + 4 hf + (e & 3), token ln
        imp_floatx16 sf, sc;
#pragma unroll
        for (int e = 0; e < 16; ++e) { sf[e] = 0.f; sc[e] = 0.f; }
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            const int at = ln * D + 8 * ((2 * ks + hf) ^ (ln & (PIECES - 1)));
            const imp_bf16x8 qv = __builtin_bit_cast(imp_bf16x8, qa[ks]);
            sf = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qv, *reinterpret_cast<const imp_bf16x8 *>(colKf + at), sf, 0, 0, 0);
            sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qv, *reinterpret_cast<const imp_bf16x8 *>(colKc + at), sc, 0, 0, 0);
        }
        float a[16], t[16];
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int r = 8 * (e >> 2) + 4 * hf + (e & 3);
            a[e] = __expf(scale * sf[e] - __shfl(row_lse, r));
            a[e] = __shfl(row_j, r) >= my_token ? a[e] : 0.f;      // causal: row j sees token i
            t[e] = scale * (sc[e] - sf[e]);
        }
        // |key term|_1 = a |t| sum_c |v_c - h_c| and |both|_1 = a sum_c |dv_c + t (v_c - h_c)|, each one fp32 chain over the channels
        imp_floatx16 nk, nkv;
#pragma unroll
        for (int e = 0; e < 16; ++e) { nk[e] = 0.f; nkv[e] = 0.f; }
        const imp_floatx16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        auto row_h = [&](int c) -> imp_s16x4 {               // the A operand: channels c & ~3 .. + 3
            const uint4 w = h[c >> 3];
            return __builtin_bit_cast(imp_s16x4, c & 4 ? (uint64_t)w.w << 32 | w.z : (uint64_t)w.y << 32 | w.x);
        };
        ulonglong2 b01 = *reinterpret_cast<const ulonglong2 *>(b_from), b23 = *reinterpret_cast<const ulonglong2 *>(b_from + 2);
        float4 dv = *reinterpret_cast<const float4 *>(dv_from);
        imp_floatx16 x = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(row_h(0), __builtin_bit_cast(imp_s16x4, (uint64_t)b01.x), zero, 0, 0, 0);
#pragma unroll
        for (int c4 = 0; c4 < D / 4; ++c4) {
            const int next = c4 + 1 < D / 4 ? c4 + 1 : c4;
            const ulonglong2 b01_next = *reinterpret_cast<const ulonglong2 *>(b_from + 4 * next), b23_next = *reinterpret_cast<const ulonglong2 *>(b_from + 4 * next + 2);
            const float4 dv_next = *reinterpret_cast<const float4 *>(dv_from + 4 * next);
            const uint64_t be[4] = {b01.y, b23.x, b23.y, b01_next.x};
            const float dve[4] = {dv.x, dv.y, dv.z, dv.w};
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                // the next channel's differences run beside this channel's vector work; nk and nkv pass through the empty statement,
                // which keeps the compiler from drawing the MFMAs of all channels together
                imp_floatx16 x_next = x;
                if (4 * c4 + u + 1 < D) {
                    x_next = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(row_h(4 * c4 + u + 1), __builtin_bit_cast(imp_s16x4, be[u]), zero, 0, 0, 0);
                    asm volatile("" : "+v"(nk), "+v"(nkv));
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    nk[e] += fabsf(x[e]);
                    nkv[e] += fabsf(fmaf(t[e], x[e], dve[u]));
                }
                x = x_next;
            }
            b01 = b01_next;
            b23 = b23_next;
            dv = dv_next;
        }
        // a slot's zero times an infinite or NaN H is a NaN in its three neighbours: then channel by channel
        float any = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) any += nk[e];
        if (__builtin_amdgcn_ballot_w64(any != any) != 0) {
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const uint16_t *h_row = h_fresh + __shfl((long long)row, 8 * (e >> 2) + 4 * hf + (e & 3)) * D;
                float k1 = 0.f, kv1 = 0.f;
#pragma unroll 1
                for (int c = 0; c < D; ++c) {
                    const float d = __uint_as_float((uint32_t)(colV[ln * LDV + c] >> (16 * (c & 3))) << 16) - __uint_as_float((uint32_t)h_row[c] << 16);
                    k1 += fabsf(d);
                    kv1 += fabsf(fmaf(t[e], d, colDV[ln * LDD + c]));
                }
                nk[e] = k1;
                nkv[e] = kv1;
            }
        }
        // (a pair that is none, a row before its token or past the end, adds nothing even where its norm is Inf or NaN)
        const bool all_pairs = j0 + (int)(p0 / (uint32_t)grp) >= i_last && p0 + kTileRows <= n_pairs;     // uniform
        float blk_a[4] = {0.f, 0.f, 0.f, 0.f}, blk_k[4] = {0.f, 0.f, 0.f, 0.f}, blk_kv[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const bool pair = all_pairs || __shfl(row_j, 8 * (e >> 2) + 4 * hf + (e & 3)) >= my_token;
            blk_a[e & 3] += a[e];
            const float to_k = fmaf(a[e] * fabsf(t[e]), nk[e], blk_k[e & 3]), to_kv = fmaf(a[e], nkv[e], blk_kv[e & 3]);
            blk_k[e & 3] = pair ? to_k : blk_k[e & 3];
            blk_kv[e & 3] = pair ? to_kv : blk_kv[e & 3];
        }
        add_carried(sum_a, carry_a, (blk_a[0] + blk_a[1]) + (blk_a[2] + blk_a[3]));
        add_carried(sum_k, carry_k, (blk_k[0] + blk_k[1]) + (blk_k[2] + blk_k[3]));
        add_carried(sum_kv, carry_kv, (blk_kv[0] + blk_kv[1]) + (blk_kv[2] + blk_kv[3]));
    }
    // ---- the shares of the waves and half-waves, added in their order ----
    __syncthreads();
    float *red = reinterpret_cast<float *>(colKf);           // [3][4][64]
    static_assert(3 * kTileWaves * 64 * 4 <= 2 * kTileCols * 64 * 2, "fits the smaller K tiles");
    red[(0 * kTileWaves + wave) * 64 + lane] = sum_a;
    red[(1 * kTileWaves + wave) * 64 + lane] = sum_k;
    red[(2 * kTileWaves + wave) * 64 + lane] = sum_kv;
    __syncthreads();
    if (tid < kTileCols && col_ok) {
        double sa = 0., sk = 0., skv = 0., l1 = 0.;          // (a few additions: rounded once, where the share is stored)
        for (int w = 0; w < 2 * kTileWaves; ++w) {
            sa += red[0 * kTileWaves * 64 + 32 * w + ln];
            sk += red[1 * kTileWaves * 64 + 32 * w + ln];
            skv += red[2 * kTileWaves * 64 + 32 * w + ln];
        }
        for (int c = 0; c < D; ++c) l1 += fabsf(colDV[ln * LDD + c]);
        // value direction: (sum of A over rows and heads of the group) * |dV|_1, nothing from a piece that does not see the token
        part[o] = sa == 0. ? 0.f : (float)(sa * l1);
        part[o + stride] = (float)sk;
        part[o + 2 * stride] = (float)skv;
    }
}

// adds the pieces and the KV heads; what is not rated is -inf (and was never written).  A workgroup takes one of the three
// results for 64 tokens, its eight waves the pieces in turn: a thread that adds all 3 x 32 x 4 shares of a token by itself is a
// chain of loads (8192 tokens: 124 us, 5 like this; the whole call at 526 tokens: 167 -> 78).
constexpr int kReduceWaves = 8;
__global__ __launch_bounds__(kReduceWaves * 64) void impact_reduce_kernel(
    int n, int n_kv_heads, int pieces, const float *__restrict__ part, const uint8_t *__restrict__ reused,
    float *__restrict__ impact_v, float *__restrict__ impact_k, float *__restrict__ impact_kv)
{
    __shared__ double share[kReduceWaves][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, t = blockIdx.y;
    float *out = t == 0 ? impact_v : t == 1 ? impact_k : impact_kv;
    if (!out) return;                                        // uniform
    const int i = blockIdx.x * 64 + lane;
    const bool cand = i < n && (reused ? reused[i] != 0 : true);
    double s = 0.;
    if (cand)
        for (int p = wave; p < pieces; p += kReduceWaves) {
            const float *from = part + (int64_t)(3 * p + t) * n_kv_heads * n + i;
#pragma unroll 4
            for (int g = 0; g < n_kv_heads; ++g) s += from[(int64_t)g * n];
        }
    share[wave][lane] = s;
    __syncthreads();
    if (wave == 0 && i < n) {
        for (int w = 1; w < kReduceWaves; ++w) s += share[w][lane];
        out[i] = cand ? (float)s : -INFINITY;
    }
}

template <int D>
constexpr size_t impact_lds_bytes()
{
    return sizeof(float) * (4 * D * kImpCols + 2 * kImpBlock * D + 2 * kImpBlock + 3 * kImpRowLanes * kImpCols);
}

// Pieces of the rows (bf16): 32 tokens of a KV head see up to n rows, and the launch is a triangle of such strips;
// some 16384 workgroups, half of them with rows, even it out over 512 resident ones (8192 Qwen-shaped tokens 7.54 ms, with 8192
// workgroups 7.62, 4096 8.00).  A piece is a whole number of rounds of the four waves, 128 (row, head in group) pairs, as nearly as its
// rows allow: a round costs the same however few of its pairs there are (256 Yi-shaped tokens, pieces of 64 pairs: 52 us, 33 like this).
constexpr int kImpUnits = 16384, kImpMaxPieces = 32, kImpRound = kTileRows * kTileWaves;
struct ImpactPieces {
    int n, rows;            // pieces, rows of each
};
int64_t impact_most_pieces(const kvs_shape *shape, int64_t n)
{
    const int64_t blocks = (n * (shape->n_q_heads / shape->n_kv_heads) + kTileRows - 1) / kTileRows;
    return blocks < 1 ? 1 : blocks < kImpMaxPieces ? blocks : kImpMaxPieces;
}
ImpactPieces impact_pieces(const kvs_shape *shape, int64_t n)
{
    const int64_t strips = (n + kTileCols - 1) / kTileCols * shape->n_kv_heads, grp = shape->n_q_heads / shape->n_kv_heads;
    int64_t p = kImpUnits / strips;
    if (p > impact_most_pieces(shape, n)) p = impact_most_pieces(shape, n);
    if (p < 1) p = 1;
    int64_t rows = (n + p - 1) / p;
    rows = (rows * grp + kImpRound - 1) / kImpRound * kImpRound / grp;
    return {(int)((n + rows - 1) / rows), (int)rows};
}
size_t impact_part_bytes(const kvs_shape *shape, int64_t n, int pieces) { return sizeof(float) * 3 * (size_t)pieces * (size_t)shape->n_kv_heads * (size_t)n; }

} // namespace

size_t impact_workspace_bytes(const kvs_shape *shape, int64_t n_tokens)
{
    if (n_tokens <= 0 || shape->n_kv_heads <= 0 || shape->dtype != KVS_BF16) return impact_part_bytes(shape, n_tokens, 1) + 256;
    // The pieces' sums, then the list of reused tokens and its length.  The pieces are counted by a bound that grows with the
    // tokens, so that a workspace for the longest prompt serves the shorter ones: no more than their limits allow, and no
    // more than kImpUnits strips' worth of sums, unless it is one.
    const int64_t most = impact_most_pieces(shape, n_tokens);
    size_t part = impact_part_bytes(shape, n_tokens, (int)most);
    const size_t one = impact_part_bytes(shape, n_tokens, 1), strips = sizeof(float) * 3 * (size_t)kImpUnits * kTileCols;
    if (part > strips) part = strips > one ? strips : one;
    return part + sizeof(int32_t) * ((size_t)n_tokens + 1) + 256;
}

} // namespace kvs

extern "C" kvs_status kvs_first_order_impact(const kvs_shape *shape, int64_t n_tokens, const void *q,
                                             const void *k_fresh, const void *v_fresh,
                                             const void *k_cache, const void *v_cache,
                                             const void *h_fresh, const float *lse,
                                             const uint8_t *reused, float scale,
                                             float *impact_v, float *impact_k, float *impact_kv,
                                             void *workspace, size_t workspace_bytes, void *stream)
{
    using namespace kvs;
    kvs_status st = check_shape(shape);
    if (st != KVS_OK) return st;
    if (n_tokens < 0) return fail(KVS_EINVAL, "kvs_first_order_impact: n_tokens < 0");
    if (n_tokens == 0) return KVS_OK;
    if (n_tokens > (1 << 20)) return fail(KVS_EUNSUPPORTED, "kvs_first_order_impact: more than 2^20 tokens");
    if (!q || !k_fresh || !v_fresh || !k_cache || !v_cache || !h_fresh || !lse) return fail(KVS_EINVAL, "kvs_first_order_impact: NULL tensor pointer");
    if (!(isfinite(scale))) return fail(KVS_EINVAL, "kvs_first_order_impact: scale is not finite");
    if (shape->n_kv_heads > 65535) return fail(KVS_EUNSUPPORTED, "kvs_first_order_impact: too many kv heads");
    const size_t need = impact_workspace_bytes(shape, n_tokens);
    if (!workspace || workspace_bytes < need) return fail(KVS_EWORKSPACE, "kvs_first_order_impact: workspace %zu < %zu bytes", workspace_bytes, need);
    if (reinterpret_cast<uintptr_t>(workspace) & 255u) return fail(KVS_EINVAL, "kvs_first_order_impact: workspace must be 256-byte aligned");
    hipStream_t hs = (hipStream_t)stream;
    const int n = (int)n_tokens, hk = shape->n_kv_heads;
    float *part = (float *)workspace;
    int pieces = 1;
    if (shape->dtype == KVS_BF16) {
        const ImpactPieces cut = impact_pieces(shape, n_tokens);
        pieces = cut.n;
        // (up to two strips of tokens are computed whole, and those not reused dropped at the end: the launch that makes the list
        // costs more than a strip; 33 to 64 tokens of 28:4, 32:8 and 8:8 heads, 20 to 80 % reused: 24 us, with a list 27)
        int32_t *list = reused && n > 2 * kTileCols ? (int32_t *)((char *)workspace + impact_part_bytes(shape, n_tokens, pieces)) : nullptr;
        int32_t *count = list ? list + n : nullptr;
        if (list) {
            hipLaunchKernelGGL(impact_list_kernel, dim3(1), dim3(kListThreads), 0, hs, n, reused, list, count);
            if ((st = check_launch("kvs_first_order_impact(list)")) != KVS_OK) return st;
        }
        const dim3 grid((unsigned)((n + kTileCols - 1) / kTileCols), (unsigned)hk, (unsigned)pieces);
#define KVS_IMP(DD)                                                                                                       \
    do {                                                                                                                  \
        static DeviceOnce once;                                                                                           \
        st = once_per_device(once, [] {                                                                                   \
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&impact_tiles_kernel<DD>),            \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, tile_lds_bytes<DD>());   \
            return e == hipSuccess ? KVS_OK : fail(KVS_EHIP, "kvs_first_order_impact: hipFuncSetAttribute: %s", hipGetErrorString(e)); \
        });                                                                                                               \
        if (st != KVS_OK) return st;                                                                                      \
        hipLaunchKernelGGL(impact_tiles_kernel<DD>, grid, dim3(kTileThreads), tile_lds_bytes<DD>(), hs, n, shape->n_q_heads, hk, cut.rows, \
                           (const uint16_t *)q, (const uint16_t *)k_fresh, (const uint16_t *)v_fresh, (const uint16_t *)k_cache, \
                           (const uint16_t *)v_cache, (const uint16_t *)h_fresh, lse, scale, list, count, part);          \
    } while (0)
        if (shape->head_dim == 128) KVS_IMP(128);
        else KVS_IMP(64);
#undef KVS_IMP
    } else {
        const dim3 grid((unsigned)((n + kImpCols - 1) / kImpCols), (unsigned)hk);
#define KVS_IMP(DD)                                                                                                       \
    do {                                                                                                                  \
        static DeviceOnce once;                                                                                           \
        st = once_per_device(once, [] {                                                                                   \
            const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&impact_kernel<DD>),                  \
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)impact_lds_bytes<DD>()); \
            return e == hipSuccess ? KVS_OK : fail(KVS_EHIP, "kvs_first_order_impact: hipFuncSetAttribute: %s", hipGetErrorString(e)); \
        });                                                                                                               \
        if (st != KVS_OK) return st;                                                                                      \
        hipLaunchKernelGGL(impact_kernel<DD>, grid, dim3(kImpThreads), (impact_lds_bytes<DD>()), hs, n, shape->n_q_heads, hk, \
                           (const float *)q, (const float *)k_fresh, (const float *)v_fresh, (const float *)k_cache,      \
                           (const float *)v_cache, (const float *)h_fresh, lse, scale, part);                             \
    } while (0)
        if (shape->head_dim == 128) KVS_IMP(128);
        else KVS_IMP(64);
#undef KVS_IMP
    }
    if ((st = check_launch("kvs_first_order_impact")) != KVS_OK) return st;
    hipLaunchKernelGGL(impact_reduce_kernel, dim3((unsigned)((n + 63) / 64), 3), dim3(kReduceWaves * 64), 0, hs, n, hk, pieces, part, reused,
                       impact_v, impact_k, impact_kv);
    return check_launch("kvs_first_order_impact(reduce)");
}
