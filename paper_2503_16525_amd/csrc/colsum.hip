// kvs_attn_colsum: the attention column mass of a whole prefill (Alg. 1 steps 1-2),
//     alpha[g, i] = sum over the query heads h of KV head g and over the rows j >= i of A_h[j, i],
//     A_h = causal row softmax of scale * Q_h K_g^T,
// in two sweeps over the score matrix, neither of which stores it:
//   sweep 1 (per query row): the log-sum-exp of the row, kept in a scratch array;
//   sweep 2 (per key):       the sum over the rows of exp(score - row's log-sum-exp).
//
// Both sweeps are the same kernel.  A workgroup owns 256 "fixed" rows of one KV head (sweep 1:
// query rows, flattened (token, head-in-group) like the attention kernels; sweep 2: keys), held
// in registers as the B operand of v_mfma_f32_32x32x16_bf16, 64 per wave; the other side streams
// past in tiles of 32 rows that go from global memory straight into an LDS ring (buffer loads
// with the LDS flag) and are read as the A operand, each read feeding two MFMAs.  In the result
// tile a lane's column is one fixed row, so the running sum of a fixed row is one scalar per lane
// (two half-waves, added at the end) and the loop has no cross-lane traffic: per score one fma,
// one exp2 and one add.  State is small (about 128 registers, 33 KiB of LDS), so several
// workgroups share a compute unit and the hardware overlaps one wave's MFMAs with another's
// vector work.
//
// Sweep 1 uses a fixed exponent reference per row, taken from the row's first key tile (plus a
// shift that centres the fp32 exponent range); if a sum
// ends above 2^100 the workgroup finds the exact row maxima in a score-only sweep and repeats.
// Sweep 2 needs none: exp(score - lse) <= 1.  No atomics: the result is identical from run to run.
//
// A sweep whose blocks of fixed rows are few, or of very different length (the first keys are seen by every
// query row, the last by a handful), leaves most of the chip waiting for its longest block.  Such a sweep is
// cut along the streamed side into pieces of `chunk` tiles, the same absolute ranges for every block; the
// pieces leave their log-sum-exps / column sums in the workspace and a small kernel combines them in order.
#include "kvs_internal.h"

#include <math.h>

namespace kvs {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int D = 128;                  // head_dim
constexpr int TS = 32;                  // streamed rows per tile
constexpr int NB = 2;                   // 32-row blocks of fixed rows per wave
constexpr int NWAVES = 4;
constexpr int NT = NWAVES * 64;
constexpr int FIXED = NWAVES * NB * 32; // fixed rows per workgroup
constexpr int ROW_B = D * 2;            // bytes of one row of one head
constexpr int TILE_B = TS * ROW_B;
constexpr int SLOT_B = TILE_B + 256;    // a tile and the 32 log-sum-exps of its rows (sweep 2)
constexpr int RING = 4;                 // slots; tiles are requested RING - 1 steps ahead
constexpr int LDS_BYTES = RING * SLOT_B;
// How a sweep is cut (plan_cut).  Three workgroups are resident per compute unit, 768 on the chip.  Measured, whole
// call, uncut -> cut: Qwen-shaped 8192 tokens 1685 -> 522 us (sweep 2 was 128 workgroups of 1 to 1792 tiles: 1450 us),
// 4296 tokens 876 -> 180, 600 tokens 150 -> 27; Llama-shaped 20000 tokens 3790 -> 3000; Yi-shaped 24000 7140 -> 4300.
constexpr int kCutResident = 768;
constexpr int kCutUnits = 3072;         // a large sweep aims at this many pieces, four rounds: the last one is then short
                                        // (8192 tokens: 528 us with two rounds, 522 with four, 535 with eight)
constexpr int kCutSmallUnits = 512;     // a small one at less than one round, of pieces of
constexpr int kCutMinChunk = 4;         // this many tiles (1500 tokens: 45 us with pieces of 8, 56 with 5; 600 tokens: 27 with 4, 31 with 8)
constexpr int kCutRoundChunk = 16;      // to this many (3001 tokens: 112 us with 16, 123 with 24, 133 with 8)
// base-2 offset of sweep 1's fixed reference above the first tile's maximum: the row sums are then
// taken around 2^-60, where fp32 is as precise as around 1, and only overflow for a logit 160 above
constexpr float kRefShift = 60.0f;
constexpr float kNoKey = -1.0e30f;      // stands for the maximum of a row that sees no key of a piece

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4_t v) { return __builtin_bit_cast(bf16x8, v); }

// row of the 32x32 result tile that element r of a lane in half-wave hf holds
__device__ __forceinline__ int tile_row(int r, int hf) { return 8 * (r >> 2) + 4 * hf + (r & 3); }

// `in_flight` = staging instructions of younger tiles that may still be outstanding
#define KVS_CS_BARRIER_(in_flight) asm volatile("s_waitcnt vmcnt(" #in_flight ")\n\ts_barrier" ::: "memory")
#define KVS_CS_BARRIER(in_flight) KVS_CS_BARRIER_(in_flight)

// Blocks of fixed rows that have streamed tiles in piece p of a cut sweep, 0 past the last piece.
// Sweep 1: block b reaches tile p * chunk if its last query row's token is at least 32 p chunk, i.e. from
// b = p * chunk * grp / 8 on.  Sweep 2: block b streams the last tiles(b) = n_tiles - 8 grp b tiles.
template <int SWEEP>
__host__ __device__ __forceinline__ int blocks_in_piece(int n, int grp, int n_blocks, int chunk, int p)
{
    static_assert(FIXED / TS == 8, "the arithmetic below");
    if (SWEEP == 1) {
        const int tiles = (n + TS - 1) / TS;
        const int64_t first = (int64_t)p * chunk * grp / 8;
        return (int64_t)p * chunk < tiles && first < n_blocks ? n_blocks - (int)first : 0;
    }
    const int64_t left = ((int64_t)n * grp + TS - 1) / TS - (int64_t)p * chunk;
    if (left <= 0) return 0;
    const int64_t b = (left + 8 * grp - 1) / (8 * grp);
    return b < n_blocks ? (int)b : n_blocks;
}

// SWEEP 1: fixed = query rows, streamed = keys, writes lse2[g][row] (base-2, scale included).
// SWEEP 2: fixed = keys, streamed = query rows, reads lse2, writes alpha[g][key].
// Rows of a KV head's queries are flattened as row = token * grp + head-in-group.
// chunk > 0: the streamed side is cut into pieces of that many tiles; piece p of the results goes to
// part[p * n_kv_heads * (rows of `lse2` / columns of `alpha` per head)].
template <int SWEEP>
__global__ __launch_bounds__(NT, 2) void colsum_kernel(int n, int n_q_heads, int n_kv_heads,
                                                       const uint16_t *__restrict__ q,
                                                       const uint16_t *__restrict__ k, float scale_log2,
                                                       const float *__restrict__ lse2, float *__restrict__ result,
                                                       int chunk)
{
    extern __shared__ __attribute__((aligned(16))) char lds_b[];
    __shared__ int redo_flag;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int hf = lane >> 5, ln = lane & 31;
    const int grp = n_q_heads / n_kv_heads;
    // x / grp for x < 2^24 without a division in the loops (grp 1 has no 32-bit multiplier)
    const uint32_t grp_magic = 0xffffffffu / (uint32_t)grp + 1u;
    auto div_grp = [&](uint32_t x) -> uint32_t { return grp == 1 ? x : __umulhi(x, grp_magic); };
    const int g = blockIdx.x % n_kv_heads;
    int blk = blockIdx.x / n_kv_heads;
    const int n_qrows = n * grp;
    const int n_fixed = SWEEP == 1 ? n_qrows : n;
    const int n_stream = SWEEP == 1 ? n : n_qrows;
    const int n_blocks = (n_fixed + FIXED - 1) / FIXED;
    // which piece: the blocks that reach a piece are a run at the heavy end of the order below
    int piece = 0;
    if (chunk > 0) {
        for (int c = blocks_in_piece<SWEEP>(n, grp, n_blocks, chunk, 0); blk >= c; c = blocks_in_piece<SWEEP>(n, grp, n_blocks, chunk, piece)) {
            blk -= c;
            ++piece;
        }
    }
    // heaviest first: the last query rows see the most keys, the first keys are seen by the most rows
    const int fb = (SWEEP == 1 ? n_blocks - 1 - blk : blk) * FIXED;

    // ---- fixed rows: operands and positions ------------------------------------------------------
    bf16x8 bfix[NB][D / 16];
    int fpos[NB];          // token position of the lane's fixed row (query token / key index)
    int frow[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
        frow[nb] = fb + wave * (NB * 32) + nb * 32 + ln;
        const int fr = min(frow[nb], n_fixed - 1);
        const uint16_t *src;
        if (SWEEP == 1) {
            const int tok = (int)div_grp((uint32_t)fr), hh = fr - tok * grp;
            fpos[nb] = tok;
            src = q + ((int64_t)tok * n_q_heads + g * grp + hh) * D;
        } else {
            fpos[nb] = fr;
            src = k + ((int64_t)fr * n_kv_heads + g) * D;
        }
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks)
            bfix[nb][ks] = as_bf16x8(*reinterpret_cast<const u32x4_t *>(src + 16 * ks + 8 * hf));
    }
    int pmin = min(fpos[0], fpos[1]), pmax = max(fpos[0], fpos[1]);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        pmin = min(pmin, __shfl_xor(pmin, o));
        pmax = max(pmax, __shfl_xor(pmax, o));
    }

    // ---- streamed tiles ---------------------------------------------------------------------------
    // sweep 1: key tiles 0 .. (last token of the workgroup) / 32; sweep 2: query-row tiles from the
    // workgroup's first key on
    const int last_fixed = min(fb + FIXED, n_fixed) - 1;
    int t_begin = SWEEP == 1 ? 0 : (int)(((int64_t)fb * grp) / TS);
    int t_end = SWEEP == 1 ? (int)div_grp((uint32_t)last_fixed) / TS + 1 : (n_stream + TS - 1) / TS;
    if (chunk > 0) {
        // pieces count from the end of the streamed tensor at which a sweep starts (see tile_of)
        if (SWEEP == 1) { t_begin = piece * chunk; t_end = min(t_end, t_begin + chunk); }
        else { t_end -= piece * chunk; t_begin = max(t_begin, t_end - chunk); }
    }
    const int n_tiles = t_end - t_begin;
    // Step k of a sweep takes tile t_begin + k in sweep 1 and tile t_end - 1 - k in sweep 2: every
    // workgroup of a KV head then starts at the same end of the streamed tensor (key 0 / the last
    // query row) whatever its own range, so the workgroups that run together read the same tiles
    // at the same time and share them through L2.  (Sweep 2 run forwards, each workgroup from its
    // own first key, fetched 13 GB from HBM per call at 32k instead of well under 1 GB.)
    auto tile_of = [&](int k) { k = min(k, n_tiles - 1); return SWEEP == 1 ? t_begin + k : t_end - 1 - k; };

    auto make_rsrc = [&](const void *base, uint32_t bytes) -> u32x4_t {
        const uint64_t a = reinterpret_cast<uint64_t>(base);
        u32x4_t r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, bytes, 0x00020000u};
        r.x = __builtin_amdgcn_readfirstlane(r.x);
        r.y = __builtin_amdgcn_readfirstlane(r.y);
        r.z = __builtin_amdgcn_readfirstlane(r.z);
        return r;
    };
    // the streamed tensor seen from this KV head's first row (byte offsets below fit 32 bits: the
    // host checks the tensor size)
    const uint32_t k_row_bytes = (uint32_t)n_kv_heads * ROW_B, q_row_bytes = (uint32_t)n_q_heads * ROW_B;
    const u32x4_t srs = SWEEP == 1 ? make_rsrc(k + (int64_t)g * D, (uint32_t)n * k_row_bytes - (uint32_t)g * ROW_B)
                                   : make_rsrc(q + (int64_t)g * grp * D, (uint32_t)n * q_row_bytes - (uint32_t)(g * grp) * ROW_B);
    const u32x4_t lrs = make_rsrc(lse2 + (int64_t)g * n_qrows, (uint32_t)n_qrows * 4u);
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane(
        (uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)lds_b);
    // One staging instruction moves 64 x 16 bytes to 1 KiB of consecutive LDS: four rows.  A wave
    // stages rows 4w .. 4w+3 of each half of the tile.  The 16-byte piece p of row r sits at
    // position p ^ (r & 15), which makes the operand reads below conflict-free; the load realises
    // it by letting lane (row, position) fetch piece position ^ (row & 15).
    const int st_row = 4 * wave + (lane >> 4);
    const uint32_t st_piece = (uint32_t)((lane & 15) ^ st_row) * 16u;
    auto stage_16 = [&](uint32_t lds_dst, uint32_t voff) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                     :: "s"(lds_dst), "v"(voff), "s"(srs));
    };
    auto stage_4 = [&](uint32_t lds_dst, uint32_t voff) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dword %1, %2, 0 offen lds"
                     :: "s"(lds_dst), "v"(voff), "s"(lrs));
    };
    // Any step index is accepted and clamped to the sweep's last step, rows past the tensor to its
    // last row: the sweep requests tiles past its end (into slots nothing reads) so that every step
    // issues the same number of loads and the waits can count them.
    // Offsets of the lane's two rows inside tile 0, with the swizzled piece: a tile wholly inside the
    // tensor then only adds its own offset (sweep 2: when the group size divides 32, so that every
    // tile starts at a token boundary; otherwise the row index is split per tile).
    uint32_t st_off[2];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
        const uint32_t r = (uint32_t)(16 * half + st_row);
        if (SWEEP == 1) {
            st_off[half] = r * k_row_bytes + st_piece;
        } else {
            const uint32_t tok = div_grp(r), hh = r - tok * (uint32_t)grp;
            st_off[half] = tok * q_row_bytes + hh * ROW_B + st_piece;
        }
    }
    const bool even_tiles = SWEEP == 1 || TS % grp == 0;
    const uint32_t tile_bytes = SWEEP == 1 ? TS * k_row_bytes : (uint32_t)(TS / grp) * q_row_bytes;
    auto stage_tile = [&](int k) {                  // step k's tile into slot k % RING
        const uint32_t slot = lds_base + (uint32_t)((k & (RING - 1)) * SLOT_B);
        const int t = tile_of(k);
        const bool inside = even_tiles && (t + 1) * TS <= n_stream;      // uniform
#pragma unroll
        for (int half = 0; half < 2; ++half) {
            uint32_t off;
            if (inside) {
                off = st_off[half] + (uint32_t)t * tile_bytes;
            } else {
                const int sr = min(t * TS + 16 * half + st_row, n_stream - 1);
                if (SWEEP == 1) {
                    off = (uint32_t)sr * k_row_bytes + st_piece;
                } else {
                    const uint32_t tok = div_grp((uint32_t)sr), hh = (uint32_t)sr - tok * (uint32_t)grp;
                    off = tok * q_row_bytes + hh * ROW_B + st_piece;
                }
            }
            stage_16(__builtin_amdgcn_readfirstlane(slot + (uint32_t)(16 * half + 4 * wave) * ROW_B), off);
        }
        if (SWEEP == 2 && wave == 0) {
            if (lane < TS) stage_4(__builtin_amdgcn_readfirstlane(slot + TILE_B), (uint32_t)min(t * TS + lane, n_stream - 1) * 4u);
        }
    };
    // the lane reads piece 2*ks + hf of row ln, at position (2*ks + hf) ^ (ln & 15)
    const uint32_t a_read_off = (uint32_t)(ln * ROW_B + ((hf ^ (ln & 15)) * 16));
    auto read_a = [&](uint32_t slot_off, int ks) -> u32x4_t {
        return *reinterpret_cast<const u32x4_t *>(lds_b + ((a_read_off ^ (uint32_t)(32 * ks)) + slot_off));
    };

    const floatx16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    auto scores = [&](int k, floatx16 (&s)[NB]) {
        const uint32_t slot_off = (uint32_t)((k & (RING - 1)) * SLOT_B);
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) {
            const u32x4_t a = read_a(slot_off, ks);
#pragma unroll
            for (int nb = 0; nb < NB; ++nb)
                s[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(a), bfix[nb][ks], ks == 0 ? zero : s[nb], 0, 0, 0);
        }
    };
    // causal mask where the tile can hold a (key, query) pair with key > query for this wave, and
    // streamed rows past the tensor; s -> -inf there
    auto mask_tile = [&](int t, floatx16 (&s)[NB]) {
        const int r0 = t * TS;
        if (SWEEP == 1) {
            if (r0 + TS - 1 > pmin) {
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        if (r0 + tile_row(r, hf) > fpos[nb]) s[nb][r] = -INFINITY;
            }
        } else {
            const int tok0 = (int)div_grp((uint32_t)r0);
            if (tok0 < pmax || r0 + TS > n_stream) {
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int sr = r0 + tile_row(r, hf);
                    const int tok = (int)div_grp((uint32_t)sr);
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        if (tok < fpos[nb] || sr >= n_stream) s[nb][r] = -INFINITY;
                }
            }
        }
    };
    // wave 0 issues one more load per tile in sweep 2 (the log-sum-exps)
    auto step_barrier = [&]() {
        if (SWEEP == 2 && wave == 0) KVS_CS_BARRIER(6);
        else KVS_CS_BARRIER(4);
    };
    // One sweep over the streamed tiles; f(k, t, s) consumes the masked scores of step k = tile t.
    // At the top of step k the loads of steps k .. k+2 have been sent; the barrier makes step k's
    // tile visible to every wave and tells that every wave is done with step k-1, whose slot step
    // k+3 then takes.
    auto sweep = [&](auto f) {
#pragma unroll
        for (int i = 0; i < RING - 1; ++i) stage_tile(i);
        for (int k = 0; k < n_tiles; ++k) {
            step_barrier();
            stage_tile(k + RING - 1);
            const int t = tile_of(k);
            floatx16 s[NB];
            scores(k, s);
            mask_tile(t, s);
            f(k, t, s);
        }
        // nothing may still be on its way into LDS when the ring is reused or the workgroup ends
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };

    float acc[NB];
    if (SWEEP == 1) {
        float ref[NB] = {0.f, 0.f};
        for (int pass = 0; pass < 2; ++pass) {
            if (pass == 1) {
                // exact row maxima
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) ref[nb] = -INFINITY;
                sweep([&](int, int, floatx16 (&s)[NB]) {
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                        for (int r = 0; r < 16; ++r) ref[nb] = fmaxf(ref[nb], s[nb][r]);
                });
#pragma unroll
                for (int nb = 0; nb < NB; ++nb) ref[nb] = fmaxf(fmaxf(ref[nb], __shfl_xor(ref[nb], 32)) * scale_log2, kNoKey);
            }
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) acc[nb] = 0.f;
            sweep([&](int k, int, floatx16 (&s)[NB]) {
                if (pass == 0 && k == 0) {
                    // the reference: the largest score of the row's first tile, whose first key a row sees if it
                    // sees any of the piece (a row that sees none keeps a finite reference and a sum of 0)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb) {
                        float mx = s[nb][0];
#pragma unroll
                        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, s[nb][r]);
                        ref[nb] = fmaxf(fmaxf(mx, __shfl_xor(mx, 32)) * scale_log2, kNoKey) + kRefShift;
                    }
                }
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
                        acc[nb] += __builtin_amdgcn_exp2f(fmaf(s[nb][r], scale_log2, -ref[nb]));
            });
            bool bad = false;
#pragma unroll
            for (int nb = 0; nb < NB; ++nb) {
                acc[nb] += __shfl_xor(acc[nb], 32);
                bad |= !(acc[nb] < 1.2676506e30f);          // 2^100; also true for inf and nan
            }
            if (pass == 1) break;
            if (tid == 0) redo_flag = 0;
            __syncthreads();
            if (bad) redo_flag = 1;
            __syncthreads();
            if (redo_flag == 0) break;
        }
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
            // the sum is taken around 2^-kRefShift: scaled back first (exactly), its logarithm is small and so is that
            // logarithm's last place (with log2(acc) near -50 the column sums of 8192 tokens were 1.7e-6 off)
            if (hf == 0 && frow[nb] < n_fixed) {
                const bool low = acc[nb] < 1.0f;
                const float l = (low ? ref[nb] - kRefShift : ref[nb]) + __builtin_amdgcn_logf(low ? acc[nb] * 0x1p60f : acc[nb]);
                result[((int64_t)piece * n_kv_heads + g) * n_qrows + frow[nb]] = l;    // -inf for a sum of 0
            }
    } else {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) acc[nb] = 0.f;
        sweep([&](int k, int, floatx16 (&s)[NB]) {
            const char *lp = lds_b + (k & (RING - 1)) * SLOT_B + TILE_B + 16 * hf;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float4 l4 = *reinterpret_cast<const float4 *>(lp + 32 * i);   // rows 8i + 4hf .. +3
                const float lv[4] = {l4.x, l4.y, l4.z, l4.w};
#pragma unroll
                for (int c = 0; c < 4; ++c)
#pragma unroll
                    for (int nb = 0; nb < NB; ++nb)
                        acc[nb] += __builtin_amdgcn_exp2f(fmaf(s[nb][4 * i + c], scale_log2, -lv[c]));
            }
        });
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) {
            acc[nb] += __shfl_xor(acc[nb], 32);
            if (hf == 0 && frow[nb] < n_fixed) result[((int64_t)piece * n_kv_heads + g) * n + frow[nb]] = acc[nb];
        }
    }
}

// lse2[g][row] of the pieces' log-sum-exps: m + log2(sum_p 2^(l_p - m)), pieces in order
__global__ __launch_bounds__(256) void colsum_join_rows(int n_qrows, int n_kv_heads, int grp, int chunk, const float *__restrict__ part,
                                                        float *__restrict__ lse2)
{
    const int row = blockIdx.x * 256 + threadIdx.x, g = blockIdx.y;
    if (row >= n_qrows) return;
    const int64_t at = (int64_t)g * n_qrows + row, stride = (int64_t)n_kv_heads * n_qrows;
    const int pieces = row / grp / TS / chunk + 1;              // up to the row's own token
    float m = -INFINITY, sum = 0.f;
    for (int p = 0; p < pieces; ++p) m = fmaxf(m, part[p * stride + at]);
    for (int p = 0; p < pieces; ++p) sum += __builtin_amdgcn_exp2f(part[p * stride + at] - m);
    lse2[at] = m + __builtin_amdgcn_logf(sum);
}

// alpha[g][key] of the pieces' column sums, in order
__global__ __launch_bounds__(256) void colsum_join_cols(int n, int n_kv_heads, int grp, int chunk, const float *__restrict__ part,
                                                        float *__restrict__ alpha)
{
    const int i = blockIdx.x * 256 + threadIdx.x, g = blockIdx.y;   // a workgroup is a block of fixed keys
    static_assert(FIXED == 256, "one block of keys per workgroup");
    if (i >= n) return;
    const int64_t at = (int64_t)g * n + i, stride = (int64_t)n_kv_heads * n;
    const int tiles = (int)(((int64_t)n * grp + TS - 1) / TS) - (int)blockIdx.x * 8 * grp;
    const int pieces = (tiles + chunk - 1) / chunk;
    float sum = 0.f;
#pragma unroll 8
    for (int p = 0; p < pieces; ++p) sum += part[p * stride + at];
    alpha[at] = sum;
}

// How a sweep is cut: tiles per piece (0: not at all), pieces, workgroups per KV head.
struct Cut {
    int chunk, pieces, units;
};
template <int SWEEP>
Cut plan_cut(const kvs_shape *shape, int64_t n)
{
    const int grp = shape->n_q_heads / shape->n_kv_heads;
    const int64_t n_fixed = SWEEP == 1 ? n * grp : n, n_stream = SWEEP == 1 ? n : n * grp;
    const int64_t blocks = (n_fixed + FIXED - 1) / FIXED, tiles = (n_stream + TS - 1) / TS;
    const Cut whole = {0, 1, (int)blocks};
    if (SWEEP == 1 && blocks * shape->n_kv_heads >= kCutResident) return whole;   // its blocks are many (every query head's rows) and fill the chip
    // (causal: a block has half the tiles on average)
    const int64_t work = blocks * tiles / 2 * shape->n_kv_heads;
    int64_t chunk = work / kCutSmallUnits;
    if (chunk > kCutRoundChunk) chunk = kCutRoundChunk;
    if (chunk < work / kCutUnits) chunk = work / kCutUnits;
    if (chunk < kCutMinChunk) chunk = kCutMinChunk;
    if (chunk >= tiles) return whole;
    Cut c = {(int)chunk, 0, 0};
    for (int b; (b = blocks_in_piece<SWEEP>((int)n, grp, (int)blocks, (int)chunk, c.pieces)) > 0; ++c.pieces) c.units += b;
    return c;
}

template <int SWEEP>
kvs_status launch_sweep(const kvs_shape *shape, int64_t n, const void *q, const void *k, float scale_log2,
                        const float *lse2, float *result, float *part, const Cut &cut, hipStream_t st)
{
    static DeviceOnce attr_once;
    const kvs_status ast = once_per_device(attr_once, [] {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&colsum_kernel<SWEEP>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, LDS_BYTES);
        return e == hipSuccess ? KVS_OK : fail(KVS_EHIP, "kvs_attn_colsum: hipFuncSetAttribute: %s", hipGetErrorString(e));
    });
    if (ast != KVS_OK) return ast;
    const int grp = shape->n_q_heads / shape->n_kv_heads, hk = shape->n_kv_heads;
    hipLaunchKernelGGL(colsum_kernel<SWEEP>, dim3((unsigned)(cut.units * (int64_t)hk)), dim3(NT), LDS_BYTES, st,
                       (int)n, shape->n_q_heads, hk, (const uint16_t *)q, (const uint16_t *)k, scale_log2,
                       lse2, cut.chunk > 0 ? part : result, cut.chunk);
    const kvs_status stt = check_launch(SWEEP == 1 ? "kvs_attn_colsum(row sums)" : "kvs_attn_colsum(column sums)");
    if (stt != KVS_OK || cut.chunk == 0) return stt;
    const dim3 grid((unsigned)(((SWEEP == 1 ? n * grp : n) + 255) / 256), (unsigned)hk);
    if (SWEEP == 1) hipLaunchKernelGGL(colsum_join_rows, grid, dim3(256), 0, st, (int)(n * grp), hk, grp, cut.chunk, part, result);
    else hipLaunchKernelGGL(colsum_join_cols, grid, dim3(256), 0, st, (int)n, hk, grp, cut.chunk, part, result);
    return check_launch("kvs_attn_colsum(join)");
}

bool on_matrix_cores(const kvs_shape *shape, int64_t n_tokens)
{
    // rows are addressed with 32-bit byte offsets and divided by the group size with a 24-bit trick
    return shape->dtype == KVS_BF16 && shape->head_dim == D && n_tokens * shape->n_q_heads * (int64_t)ROW_B < ((int64_t)1 << 32) &&
           n_tokens * (shape->n_q_heads / shape->n_kv_heads) < (1 << 24);
}

size_t row_bytes(const kvs_shape *shape, int64_t n_tokens) { return ((size_t)n_tokens * shape->n_q_heads * sizeof(float) + 255) / 256 * 256; }

// The most that the pieces of one sweep take at a time, in a form that grows with n_tokens (the pieces themselves do not:
// their number jumps where plan_cut rounds, and a large sweep 1 is not cut), so that a workspace for the longest prompt serves
// the shorter ones.  With e = n_tokens * n_q_heads results per piece of sweep 1 (sweep 2: no more pieces times results), t
// its tiles and w = plan_cut's work, w >= t * e / 512: a chunk c gives at most t / c + 1 pieces, and c is at least 4, at
// least 4/5 of w / 3072, and at least 4/5 of w / 512 unless it is 16.
size_t piece_bytes(const kvs_shape *shape, int64_t n_tokens)
{
    static_assert(kCutMinChunk == 4 && kCutRoundChunk == 16 && kCutSmallUnits == 512 && kCutUnits == 3072, "the bounds below");
    const int64_t e = n_tokens * shape->n_q_heads, steps = (n_tokens < (1 << 20) ? n_tokens : 1 << 20) * e;   // (from there on by_units is the least)
    const int64_t by_least = steps / 128 + 2 * e;
    const int64_t sixteen = steps / 512, by_small = (sixteen > 640 * 512 ? sixteen : 640 * 512) + 2 * e;
    const int64_t by_units = 3840 * 512 + 2 * e;
    const int64_t most = by_least < by_small ? by_least : by_small;
    return sizeof(float) * (size_t)(most < by_units ? most : by_units);
}

} // namespace

// what every call needs; fp32 layers take more if they are given it (one sweep instead of two)
static size_t colsum_least_bytes(const kvs_shape *shape, int64_t n_tokens)
{
    const size_t rows = row_bytes(shape, n_tokens);
    // (fp32 kernels: two floats a row; they also take a scale that is not positive)
    const size_t pieces = shape->dtype == KVS_BF16 && shape->head_dim == D ? piece_bytes(shape, n_tokens) : 0;
    return rows + (pieces > rows ? pieces : rows) + 256;
}

size_t colsum_workspace_bytes(const kvs_shape *shape, int64_t n_tokens)
{
    if (n_tokens <= 0) return 256;
    const size_t least = colsum_least_bytes(shape, n_tokens);
    const size_t one_sweep = shape->dtype == KVS_BF16 && shape->head_dim == D ? 0 : colsum_f32_workspace_bytes(shape, n_tokens);
    return one_sweep > least ? one_sweep : least;
}

} // namespace kvs

extern "C" kvs_status kvs_attn_colsum(const kvs_shape *shape, int64_t n_tokens, const void *q, const void *k,
                                      float scale, float *alpha, void *workspace, size_t workspace_bytes,
                                      void *stream)
{
    using namespace kvs;
    kvs_status st = check_shape(shape);
    if (st != KVS_OK) return st;
    if (n_tokens < 0) return fail(KVS_EINVAL, "kvs_attn_colsum: n_tokens < 0");
    if (n_tokens == 0) return KVS_OK;
    if (!isfinite(scale)) return fail(KVS_EINVAL, "kvs_attn_colsum: scale is not finite");
    if (!q || !k || !alpha) return fail(KVS_EINVAL, "kvs_attn_colsum: NULL tensor pointer");
    if (!aligned16(q) || !aligned16(k)) return fail(KVS_EINVAL, "kvs_attn_colsum: Q/K pointers must be 16-byte aligned");
    if (!workspace || (reinterpret_cast<uintptr_t>(workspace) & 255u)) return fail(KVS_EINVAL, "kvs_attn_colsum: workspace must be given, 256-byte aligned");
    if (workspace_bytes < colsum_least_bytes(shape, n_tokens))
        return fail(KVS_EWORKSPACE, "kvs_attn_colsum: workspace of %zu bytes, %zu needed", workspace_bytes, colsum_least_bytes(shape, n_tokens));
    // the matrix-core kernel: bf16, head_dim 128, a positive scale (it folds the scale into an exp2
    // argument after taking maxima).  Everything else takes the fp32 kernels.
    const bool mfma = shape->dtype == KVS_BF16 && shape->head_dim == D && scale > 0.f;
    if (!mfma) return launch_colsum_f32(shape, n_tokens, q, k, scale, workspace, workspace_bytes, alpha, (hipStream_t)stream);
    if (!on_matrix_cores(shape, n_tokens))
        return fail(KVS_EUNSUPPORTED, "kvs_attn_colsum: %lld tokens x %d heads exceed the 4 GiB the kernel addresses", (long long)n_tokens, shape->n_q_heads);
    float *lse2 = (float *)workspace;
    const float scale_log2 = scale * 1.4426950408889634f;
    hipStream_t hs = (hipStream_t)stream;
    const Cut c1 = plan_cut<1>(shape, n_tokens), c2 = plan_cut<2>(shape, n_tokens);
    float *part = (float *)((char *)workspace + row_bytes(shape, n_tokens));
    st = launch_sweep<1>(shape, n_tokens, q, k, scale_log2, nullptr, lse2, part, c1, hs);
    if (st != KVS_OK) return st;
    return launch_sweep<2>(shape, n_tokens, q, k, scale_log2, lse2, alpha, part, c2, hs);
}
