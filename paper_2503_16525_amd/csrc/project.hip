// kvs_project_qkv: a later layer's Q, K and V of the selected tokens (App. D.1: the tokens picked in an
// early layer are the ones recomputed in the layers after it).  Recomputing a token's Q/K/V in a layer is
// that layer's projection of its hidden state; the models the paper evaluates turn Q and K by rotary
// position factors, which are applied here from a caller-supplied table while the results are still in
// registers.  One launch: gather of the selected hidden rows, the bf16 matrix product on the matrix
// cores, the rotation, the split into the Q / K / V tensors.
//
// Shape of the product: out[token, feature] = sum_c x[rows[token], c] * w[feature, c].  Both operands
// are contiguous along c, the contraction index, which is what the matrix core wants from both sides
// (8 consecutive c per lane): neither needs a transposing read.
//
// Tiling.  A workgroup owns 256 features x 256 tokens; its four waves 128 x 128 each (one wave per
// SIMD, the 16 accumulator tiles of 32 x 32 fill the accumulation registers), so every 16-byte
// operand fetched from LDS feeds four MFMAs.  The contraction runs in steps of 32; a step's two
// tiles (256 rows x 64 bytes each) are staged from global memory straight into LDS by buffer loads
// with the LDS flag -- the gather costs nothing, every lane supplies the address of its own row --
// into a ring of five stages, two to four steps ahead of their use, one barrier per step.  Rows are 64
// bytes in LDS; the 16-byte pieces of a row are permuted per row (row_swizzle) so that the lanes an operand
// read serves together never share a bank (the plain layout and a swizzle by (r >> 1) & 3 both measured
// one conflict cycle per active LDS cycle).
//
// The features are the MFMA's rows and the tokens its columns: a lane then ends up with four
// consecutive features of one token per accumulator quad, so the rotation pairs (c, c + 64) sit in
// the same lane (feature blocks fb and fb + 2 of the wave's head).  The rotary table rows come in and
// the results go out through LDS, as whole rows.
//
// Launch order.  Workgroup b runs on XCD b % 8.  The grid of tiles (feature tiles x token tiles) is cut
// into eight blocks, fx along the features and 8 / fx along the tokens, one block per XCD: what an XCD
// pulls through its L2 is then its block's rows of weights plus its block's hidden rows, and the cut is
// chosen for the smallest block first (the launch is as long as the fullest XCD) and the smallest sum of
// the two after that.
//
// Launches too small for that tile take a second kernel, project_few_kernel, below.
#include "kvs_internal.h"

#include <type_traits>

namespace kvs {
namespace {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float floatx16;

constexpr int PD = 128;                 // head_dim
constexpr int PBM = 256;                // tokens per workgroup tile
constexpr int PBN = 256;                // features per workgroup tile (two heads)
constexpr int PBK = 32;                 // contraction step
constexpr int PSTAGES = 5;              // ring slots of 32 KiB: 5 fill the 160 KiB of a compute unit
constexpr int PNT = 256;
constexpr int PROW_B = PBK * 2;         // bytes of a tile row in LDS
constexpr int PTILE_B = 256 * PROW_B;   // one operand tile: 16 KiB
constexpr int PSTAGE_B = 2 * PTILE_B;   // weights, then tokens
constexpr int PLDS_BYTES = PSTAGES * PSTAGE_B;
constexpr int PXCDS = 8;

// position of the 16-byte piece p of tile row r inside the row's 64 bytes: p ^ row_swizzle(r).  Rows are 64
// bytes apart, so rows r, r+4, r+8, r+12 meet in the same quarter of a 256-byte bank line and rows r, r+2,
// r+4, r+6 in the same half of a 128-byte one: the two bits below are a one-to-one image of (r3, r2) and of
// (r2, r1) alike, so lanes reading the same piece of neighbouring rows never share a bank either way.
__device__ __forceinline__ int row_swizzle(int r) { return ((r >> 2) & 1) | ((((r >> 3) ^ (r >> 1)) & 1) << 1); }

__device__ __forceinline__ bf16x8 as_frag(u32x4_t v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi)
{
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    f32x2 f = {lo, hi};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));
}

__global__ __launch_bounds__(PNT, 1) void project_qkv_kernel(
    int n_q_heads, int n_kv_heads, int hidden, const uint16_t *__restrict__ x, int64_t n_tokens,
    const int32_t *__restrict__ x_rows, const int32_t *__restrict__ sel_pos, int n_sel,
    const uint16_t *__restrict__ w, const float *__restrict__ rope, int rope_positions,
    uint16_t *__restrict__ q_out, uint16_t *__restrict__ k_out, uint16_t *__restrict__ v_out,
    int tiles_m, int tiles_n, int xcd_fx, int block_n, int block_m)
{
    extern __shared__ __attribute__((aligned(16))) char plds[];
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wf = wave & 1, wt = wave >> 1;      // which 128 features / 128 tokens of the tile
    // the XCD's block of the tile grid, walked with the feature tile running fastest
    const int xcd = (int)(blockIdx.x % PXCDS), in_block = (int)(blockIdx.x / PXCDS);
    const int tile_n = (xcd % xcd_fx) * block_n + in_block % block_n, tile_m = (xcd / xcd_fx) * block_m + in_block / block_n;
    if (tile_n >= tiles_n || tile_m >= tiles_m) return;      // uniform: blocks at the edges of the grid are not full
    const int m0 = tile_m * PBM, n0 = tile_n * PBN;
    const int nk = hidden / PBK;

    // ---- staging: one instruction moves 64 x 16 bytes = 16 tile rows; a wave stages rows
    // 64 w .. 64 w + 63 of the weight tile and of the token tile, 8 instructions per step
    const uint32_t row_bytes = (uint32_t)hidden * 2u;
    const int st_row = lane >> 2, st_pos = lane & 3;
    uint32_t voff_w[4], voff_x[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = 64 * wave + 16 * i + st_row;                   // row of the tile
        const uint32_t piece = (uint32_t)(st_pos ^ row_swizzle(r)) * 16u;
        voff_w[i] = (uint32_t)(n0 + r) * row_bytes + piece;
        const int t = min(m0 + r, n_sel - 1);                         // rows past the end repeat the last token (never stored)
        int64_t xr = x_rows ? (int64_t)x_rows[t] : (int64_t)t;
        xr = min(max(xr, (int64_t)0), n_tokens - 1);                  // memory safety; the caller guarantees the range
        voff_x[i] = (uint32_t)xr * row_bytes + piece;
    }
    const int n_features = (n_q_heads + 2 * n_kv_heads) * PD;
    auto make_rsrc = [&](const uint16_t *base, uint64_t bytes) -> u32x4_t {
        const uint64_t a = reinterpret_cast<uint64_t>(base);
        u32x4_t r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, (uint32_t)bytes, 0x00020000u};
        r.x = __builtin_amdgcn_readfirstlane(r.x);
        r.y = __builtin_amdgcn_readfirstlane(r.y);
        r.z = __builtin_amdgcn_readfirstlane(r.z);
        return r;
    };
    const u32x4_t wrs = make_rsrc(w, (uint64_t)n_features * row_bytes);
    const u32x4_t xrs = make_rsrc(x, (uint64_t)n_tokens * row_bytes);
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)plds);
    // the offsets above came through ordinary loads: none may be outstanding when the counted waits begin
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    auto stage_1k = [&](const u32x4_t &rs, uint32_t lds_dst, uint32_t voff, uint32_t soff) {
        asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                     :: "s"(lds_dst), "v"(voff), "s"(rs), "s"(soff));
    };
    // Contraction steps 2t and 2t+1 are the two halves of the same 128-byte lines of global memory and are
    // requested as a pair, a row group's first half right before its second.  Load k of a pair (0..15): row
    // group k / 4; weights for k % 4 < 2, tokens otherwise; first step of the pair for even k.  Steps
    // past the end repeat the last one (their slots are never read).
    auto stage_one = [&](int first_step, int slot_a, int slot_b, int k) {
        const int i = k >> 2, second = k & 1, tokens = (k >> 1) & 1;
        const int ks = min(first_step + second, nk - 1);
        const uint32_t soff = __builtin_amdgcn_readfirstlane((uint32_t)ks * (uint32_t)(PBK * 2));
        const uint32_t dst = lds_base + (uint32_t)((second ? slot_b : slot_a) * PSTAGE_B) + (uint32_t)(64 * wave + 16 * i) * PROW_B
                             + (uint32_t)(tokens ? PTILE_B : 0);
        stage_1k(tokens ? xrs : wrs, __builtin_amdgcn_readfirstlane(dst), tokens ? voff_x[i] : voff_w[i], soff);
    };

    // ---- operand reads: lane (ln, hf) reads piece 2 ks + hf of row (block base + ln)
    const uint32_t rd_off = (uint32_t)(ln * PROW_B + ((hf ^ row_swizzle(ln)) * 16));
    auto read_frag = [&](uint32_t tile_off, int block, int ks) -> u32x4_t {      // tile_off: byte offset of the operand tile
        return *reinterpret_cast<const u32x4_t *>(plds + tile_off + (uint32_t)(block * 32 * PROW_B) + (rd_off ^ (uint32_t)(32 * ks)));
    };

    floatx16 acc[4][4];     // [feature block][token block]
#pragma unroll
    for (int fb = 0; fb < 4; ++fb)
#pragma unroll
        for (int tb = 0; tb < 4; ++tb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fb][tb][r] = 0.f;

    // Software pipeline.  Step j multiplies with the first half of its operands (read from LDS during step
    // j-1) while it fetches the second half, passes the step's one barrier, fetches the first half of
    // step j+1 and multiplies with the second half: the matrix pipe has work on both sides of the barrier.
    // Everything is issued in order, so what must overlap is interleaved in program order and pinned there
    // with scheduling fences: per 4 MFMAs two LDS fetches and one global -> LDS load.  (LDS takes one 16-byte
    // fetch per ~9 clocks from the four waves together and the texture path one 1 KiB load per ~23: issued in
    // bursts they hold up the MFMAs behind them -- fetches in a block cost 1760 clocks per step against 1024 of
    // matrix work, a step's loads in a block another 40 %.)
    //
    // Slots and waits.  The slot of step s is read from the barrier of step s-1 to the barrier of step s.
    // The pair (e+4, e+5), e even, takes the slots of steps e-1 and e and goes out in four quarters
    // after the barrier of step e: second half of e, both halves of e+1, first half of e+2; it is needed at
    // the barriers of e+3 (first step) and e+4 (second), a full step after its last load.  So at an even
    // step's barrier the youngest pair (16 loads) is complete behind the one needed, and at an odd step's
    // barrier 8 loads of the next pair plus the last load of the needed pair (which belongs to its second
    // step) may be in flight.  Each wave waits for its own loads and LDS fetches, the barrier covers the
    // others'.
    static_assert(PSTAGES == 5, "the waits below are counted for five slots");
#pragma unroll
    for (int k = 0; k < 16; ++k) stage_one(0, 0, 1, k);
#pragma unroll
    for (int k = 0; k < 12; ++k) stage_one(2, 2, 3, k);                 // (its last quarter goes out in step 0, as in every even step)
    asm volatile("s_waitcnt vmcnt(13)\n\ts_barrier" ::: "memory");      // step 0 has landed
    u32x4_t a0[4], b0[4];
    {
        const uint32_t w_tile = (uint32_t)(wf * 128 * PROW_B), x_tile = (uint32_t)(PTILE_B + wt * 128 * PROW_B);
#pragma unroll
        for (int i = 0; i < 4; ++i) { a0[i] = read_frag(w_tile, i, 0); b0[i] = read_frag(x_tile, i, 0); }
    }
    // one half of a step: 16 MFMAs with (a_use, b_use); the fetches of (a_get, b_get) from the given tiles, ks;
    // loads quarter*4 .. quarter*4+3 of the pair that starts at `pair_step`
    auto half = [&](const u32x4_t (&a_use)[4], const u32x4_t (&b_use)[4], u32x4_t (&a_get)[4], u32x4_t (&b_get)[4],
                    uint32_t w_from, uint32_t x_from, int ks, int pair_step, int slot_a, int slot_b, int quarter) {
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            const int fb = g >> 1, tb0 = 2 * (g & 1);
            acc[fb][tb0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(a_use[fb]), as_frag(b_use[tb0]), acc[fb][tb0], 0, 0, 0);
            acc[fb][tb0 + 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(a_use[fb]), as_frag(b_use[tb0 + 1]), acc[fb][tb0 + 1], 0, 0, 0);
            if (g < 4) b_get[g] = read_frag(x_from, g, ks);      // the token operands first: the next half's first MFMAs
            else a_get[g - 4] = read_frag(w_from, g - 4, ks);    // need all four of them and one weight operand
            if (g & 1) stage_one(pair_step, slot_a, slot_b, 4 * quarter + (g >> 1));
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto wrap = [](int s) { return s >= PSTAGES ? s - PSTAGES : s; };
    int slot = 0;           // ring slot of step e
    for (int e = 0; e < nk; e += 2) {      // nk is even
        const int s1 = wrap(slot + 1), s2 = wrap(slot + 2), s3 = wrap(slot + 3), s4 = wrap(slot + 4);
        auto w_of = [&](int sl) { return (uint32_t)(sl * PSTAGE_B) + (uint32_t)(wf * 128 * PROW_B); };
        auto x_of = [&](int sl) { return (uint32_t)(sl * PSTAGE_B) + (uint32_t)(PTILE_B + wt * 128 * PROW_B); };
        u32x4_t a1[4], b1[4];
        // even step e: pair (e+2, e+3) sits in slots s2, s3; pair (e+4, e+5) goes to slots s4 and `slot`
        half(a0, b0, a1, b1, w_of(slot), x_of(slot), 1, e + 2, s2, s3, 3);
        asm volatile("s_waitcnt vmcnt(16) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        half(a1, b1, a0, b0, w_of(s1), x_of(s1), 0, e + 4, s4, slot, 0);
        // odd step e+1
        half(a0, b0, a1, b1, w_of(s1), x_of(s1), 1, e + 4, s4, slot, 1);
        asm volatile("s_waitcnt vmcnt(9) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        half(a1, b1, a0, b0, w_of(s2), x_of(s2), 0, e + 4, s4, slot, 2);
        slot = s2;
    }
    // nothing may still be on its way into LDS when the workgroup ends
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // ---- epilogue: rotate, convert, store -----------------------------------------------------------
    // entry r of acc[fb][tb]: feature 32 fb + 8 (r >> 2) + 4 hf + (r & 3) of the wave's head, token 32 tb + ln.
    // A lane's results are 8-byte pieces of 128 different rows and the rotary factors it needs are 32-byte
    // pieces of its tokens' table rows: written and read that way, a tile spent as long in its epilogue as
    // in 50 contraction steps.  Both go through LDS instead (the ring is free now): the table rows of the
    // tile's 256 tokens come in as whole rows, the results leave as whole rows.
    const int head = n0 / PD + wf;
    uint16_t *dst;
    int heads_of_dst, h_local;
    if (head < n_q_heads) { dst = q_out; heads_of_dst = n_q_heads; h_local = head; }
    else if (head < n_q_heads + n_kv_heads) { dst = k_out; heads_of_dst = n_kv_heads; h_local = head - n_q_heads; }
    else { dst = v_out; heads_of_dst = n_kv_heads; h_local = head - n_q_heads - n_kv_heads; }
    const bool turned = rope != nullptr && head < n_q_heads + n_kv_heads;
    const bool tile_turned = rope != nullptr && n0 / PD < n_q_heads + n_kv_heads;      // uniform over the workgroup
    __syncthreads();                                   // every wave is done with the ring
    if (tile_turned) {
        // table rows of tokens 64 w .. 64 w + 63 of the tile, two rows (2 x 512 bytes) per instruction, straight
        // into LDS; the 16-byte piece p of token T's row sits at position p ^ (T & 31), so that the 32 lanes of
        // a half-wave, which hold 32 consecutive tokens and want the same piece, read 32 different columns
        const int t_mine = min(m0 + 64 * wave + lane, n_sel - 1);
        int p_mine = sel_pos[t_mine];
        p_mine = min(max(p_mine, 0), rope_positions - 1);          // memory safety; the caller guarantees the range
        const uint64_t ra = reinterpret_cast<uint64_t>(rope);
        u32x4_t rrs = {(uint32_t)ra, (uint32_t)(ra >> 32) & 0xffffu, (uint32_t)rope_positions * (uint32_t)(PD * 4), 0x00020000u};
        rrs.x = __builtin_amdgcn_readfirstlane(rrs.x);
        rrs.y = __builtin_amdgcn_readfirstlane(rrs.y);
        rrs.z = __builtin_amdgcn_readfirstlane(rrs.z);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll 4
        for (int i = 0; i < 32; ++i) {
            const int tok = 2 * i + hf;                             // token of the wave's 64 this lane fetches a piece of
            const int p = __shfl(p_mine, tok);
            const uint32_t voff = (uint32_t)p * (uint32_t)(PD * 4) + (uint32_t)((ln ^ (tok & 31)) * 16);
            stage_1k(rrs, __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)((64 * wave + 2 * i) * (PD * 4))), voff, 0u);
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (turned) {
#pragma unroll
            for (int tb = 0; tb < 4; ++tb) {
                const int T = 128 * wt + 32 * tb + ln;              // token of the tile; T & 31 == ln
                const char *row = plds + T * (PD * 4);
#pragma unroll
                for (int fb = 0; fb < 2; ++fb)
#pragma unroll
                    for (int r4 = 0; r4 < 4; ++r4) {
                        const int piece = (32 * fb + 8 * r4 + 4 * hf) / 2;      // (cos, sin) of channels c0, c0+1; the next piece: c0+2, c0+3
                        const float4 cs01 = *reinterpret_cast<const float4 *>(row + ((piece ^ ln) * 16));
                        const float4 cs23 = *reinterpret_cast<const float4 *>(row + (((piece + 1) ^ ln) * 16));
                        const float cs[4] = {cs01.x, cs01.z, cs23.x, cs23.z}, sn[4] = {cs01.y, cs01.w, cs23.y, cs23.w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float y1 = acc[fb][tb][4 * r4 + i], y2 = acc[fb + 2][tb][4 * r4 + i];
                            acc[fb][tb][4 * r4 + i] = y1 * cs[i] - y2 * sn[i];
                            acc[fb + 2][tb][4 * r4 + i] = y2 * cs[i] + y1 * sn[i];
                        }
                    }
            }
        }
        __syncthreads();                               // the table rows have been read: LDS is free again
    }
    // results -> this wave's LDS region [128 tokens][264 bytes] (the 8 bytes of padding spread a half-wave's
    // 32 rows over all banks) -> whole rows of 256 bytes to global memory, four rows per store instruction
    constexpr int OROW_B = PD * 2 + 8;
    char *region = plds + wave * (128 * OROW_B);
#pragma unroll
    for (int tb = 0; tb < 4; ++tb)
#pragma unroll
        for (int fb = 0; fb < 4; ++fb)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4) {
                const int c0 = 32 * fb + 8 * r4 + 4 * hf;
                *reinterpret_cast<uint2 *>(region + (32 * tb + ln) * OROW_B + 2 * c0) =
                    make_uint2(pack_bf16x2(acc[fb][tb][4 * r4 + 0], acc[fb][tb][4 * r4 + 1]), pack_bf16x2(acc[fb][tb][4 * r4 + 2], acc[fb][tb][4 * r4 + 3]));
            }
    // (same wave wrote and reads: LDS handles a wave's requests in order, no barrier)
    const int sub = lane >> 4, chunk = lane & 15;
#pragma unroll 4
    for (int i = 0; i < 32; ++i) {
        const int tok = 4 * i + sub;
        const int t = m0 + 128 * wt + tok;
        const uint2 lo = *reinterpret_cast<const uint2 *>(region + tok * OROW_B + 16 * chunk);
        const uint2 hi = *reinterpret_cast<const uint2 *>(region + tok * OROW_B + 16 * chunk + 8);
        if (t < n_sel)
            *reinterpret_cast<uint4 *>(dst + ((int64_t)t * heads_of_dst + h_local) * PD + 8 * chunk) = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
}

// ---- few tokens ---------------------------------------------------------------------------------------
// With 256 x 256 tiles a launch of a few hundred tokens leaves most of the chip idle and the others on one long
// tile.  Here a workgroup owns 64 FBW features of one head (rotation pairs together) x 32 TB tokens, the pair chosen per
// launch so that the tiles just fill the chip.  Tiles this small are bound by the global -> LDS path (1 KiB per ~23
// clocks and compute unit) and the LDS port, not by the matrix cores, so what matters is that nothing waits:
//   * eight waves, two per SIMD: wave (kg, half) multiplies the 16-wide slice kg of every contraction step of 64 for
//     one half of the features, so every 16-byte operand feeds FBW or TB MFMAs whatever the tile's shape;
//   * operands of step j+1 are fetched from LDS while step j multiplies; one barrier per step, which says that step
//     j+1 has landed and that everybody has fetched step j, whose slot then takes step j + slots;
//   * the four slices' sums meet in LDS at the end, 32 tokens at a time, where the rotation pairs sit in one thread
//     and rows leave as whole segments.
// What bounds it: one tile on an otherwise idle chip runs at the global -> LDS rate (128 x 160 tile, hidden 4096: 27 us;
// 36 us before fetches and loads were dealt out between the MFMAs).  With all units busy (39 us at 656 tokens, 470 ns a step and 8 us
// besides) no unit is saturated: matrix cores busy 38 % of the launch, L2 at 13 TB/s with 81 % hits, LDS port 18 %; the waves wait 37 % of their
// time.  Starting every tile at its own place in the contraction loses the shared L2 lines: 71 us.
constexpr int FNT = 512;
constexpr int FBK = 64;                        // contraction step; rows of 128 bytes in LDS
constexpr int FROW_B = FBK * 2;
constexpr int FLDS_MAX = 152 * 1024;

// slots of the ring: what fits, at most 12 (a few tokens: the launch streams the weights, and bytes in flight are all)
constexpr int few_slots(int fbw, int tb)
{
    const int stage = (64 * fbw + 32 * tb) * FROW_B, n = FLDS_MAX / stage;
    return n < 12 ? n : 12;
}
constexpr int few_lds_bytes(int fbw, int tb)
{
    const int ring = few_slots(fbw, tb) * (64 * fbw + 32 * tb) * FROW_B, join = (tb > 1 ? 2 : 1) * 4 * 32 * (64 * fbw + 4) * 4;
    return ring > join ? ring : join;
}

template <int FBW, int TB>
__global__ __launch_bounds__(FNT, 2) void project_few_kernel(
    int n_q_heads, int n_kv_heads, int hidden, const uint16_t *__restrict__ x, int64_t n_tokens,
    const int32_t *__restrict__ x_rows, const int32_t *__restrict__ sel_pos, int n_sel,
    const uint16_t *__restrict__ w, const float *__restrict__ rope, int rope_positions,
    uint16_t *__restrict__ q_out, uint16_t *__restrict__ k_out, uint16_t *__restrict__ v_out,
    int tiles_m, int n_tiles, int per_xcd)
{
    constexpr int WROWS = 64 * FBW, TROWS = 32 * TB;
    constexpr int STAGE_B = (WROWS + TROWS) * FROW_B, W_B = WROWS * FROW_B;
    constexpr int SLOTS = few_slots(FBW, TB);
    constexpr int NLOADS = (WROWS + TROWS) / 8;                 // 1 KiB instructions per stage, dealt to the eight waves
    constexpr int PER_WAVE = (NLOADS + 7) / 8, SHORT_FROM = NLOADS % 8 == 0 ? 8 : NLOADS % 8;   // waves from here on issue one fewer
    static_assert(SLOTS >= 3, "ring depth");
    extern __shared__ __attribute__((aligned(16))) char plds[];
    const int tid = threadIdx.x, lane = tid & 63, ln = lane & 31, hf = lane >> 5;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kg = wave & 3, half = wave >> 2;
    // an XCD takes a run of tiles, the token tile fastest: the workgroups that share weight rows share an L2
    const int tile = (int)(blockIdx.x % PXCDS) * per_xcd + (int)(blockIdx.x / PXCDS);
    if (tile >= n_tiles) return;                                // uniform
    const int tile_n = tile / tiles_m, m0 = (tile % tiles_m) * TROWS;
    const int head = FBW == 2 ? tile_n : tile_n >> 1, c0 = FBW == 2 ? 0 : 32 * (tile_n & 1);
    const int nk = hidden / FBK;
    const uint32_t row_bytes = (uint32_t)hidden * 2u;

    // ---- staging: one instruction moves 8 rows of 128 bytes; instruction q of a stage is weight rows 8 q .. for
    // 8 q < WROWS, token rows behind them; wave v issues q = v, v + 8, ...  Piece p of row r sits at position
    // p ^ ((r >> 1) & 7): 16 lanes reading one piece of 16 rows then hit all 64 banks once.
    uint32_t voff[PER_WAVE];
#pragma unroll
    for (int i = 0; i < PER_WAVE; ++i) {
        const int r = 8 * (wave + 8 * i) + (lane >> 3);
        const uint32_t piece = (uint32_t)((lane & 7) ^ ((r >> 1) & 7)) * 16u;
        if (r < WROWS) {
            // feature row r of the tile: FBW 2: channel r; FBW 1: channels c0 .. c0+31, then c0+64 .. c0+95
            const int c = FBW == 2 ? r : c0 + (r & 31) + 64 * (r >> 5);
            voff[i] = (uint32_t)(head * PD + c) * row_bytes + piece;
        } else {
            const int t = min(m0 + r - WROWS, n_sel - 1);       // rows past the end repeat the last token (never stored)
            int64_t xr = x_rows ? (int64_t)x_rows[t] : (int64_t)t;
            xr = min(max(xr, (int64_t)0), n_tokens - 1);        // memory safety; the caller guarantees the range
            voff[i] = (uint32_t)xr * row_bytes + piece;
        }
    }
    auto make_rsrc = [&](const uint16_t *base, uint64_t bytes) -> u32x4_t {
        const uint64_t a = reinterpret_cast<uint64_t>(base);
        u32x4_t r = {(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, (uint32_t)bytes, 0x00020000u};
        r.x = __builtin_amdgcn_readfirstlane(r.x);
        r.y = __builtin_amdgcn_readfirstlane(r.y);
        r.z = __builtin_amdgcn_readfirstlane(r.z);
        return r;
    };
    const u32x4_t wrs = make_rsrc(w, (uint64_t)(n_q_heads + 2 * n_kv_heads) * PD * row_bytes);
    const u32x4_t xrs = make_rsrc(x, (uint64_t)n_tokens * row_bytes);
    const uint32_t lds_base = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) char *)plds);
    // the epilogue's thread: four channels of a token and their partners 64 on, PER_TOK threads per token; its tokens' positions
    constexpr int PER_TOK = 8 * FBW;
    const int my_tok = tid / PER_TOK, my_c = 4 * (tid % PER_TOK);   // channel inside the tile's lower half
    const bool turned = rope != nullptr && head < n_q_heads + n_kv_heads;
    int my_pos[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) my_pos[tb] = turned ? sel_pos[min(m0 + 32 * tb + my_tok, n_sel - 1)] : 0;
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        my_pos[tb] = min(max(my_pos[tb], 0), rope_positions - 1);   // memory safety; the caller guarantees the range
        asm volatile("" : "+v"(my_pos[tb]));
    }
    // the offsets above came through ordinary loads: none may be outstanding when the counted waits begin
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    // load i of the wave's share of a stage; steps past the end repeat the last one (their slots are never read)
    auto stage_one = [&](int step, int slot, int i) {
        const uint32_t soff = __builtin_amdgcn_readfirstlane((uint32_t)min(step, nk - 1) * (uint32_t)FROW_B);
        const int q = wave + 8 * i;
        if (i < PER_WAVE - 1 || wave < SHORT_FROM) {            // uniform
            const uint32_t dst = __builtin_amdgcn_readfirstlane(lds_base + (uint32_t)(slot * STAGE_B + q * 1024));
            const u32x4_t &rs = i < WROWS / 64 ? wrs : xrs;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds" :: "s"(dst), "v"(voff[i]), "s"(rs), "s"(soff));
        }
    };
    auto stage = [&](int step, int slot) {
#pragma unroll
        for (int i = 0; i < PER_WAVE; ++i) stage_one(step, slot, i);
    };
    // waits for this wave's own loads but the youngest `SLOTS - 2` stages', and for its LDS fetches; then the barrier
    auto step_barrier = [&]() {
        if (wave < SHORT_FROM) asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((SLOTS - 2) * PER_WAVE) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" :: "n"((SLOTS - 2) * (PER_WAVE - 1)) : "memory");
    };
    static_assert((SLOTS - 2) * PER_WAVE <= 63, "the wait's counter has 6 bits");

    // ---- operands: lane (ln, hf) reads piece 2 kg + hf of row (block base + ln)
    const uint32_t rd = (uint32_t)(ln * FROW_B + (((2 * kg + hf) ^ ((ln >> 1) & 7)) * 16));
    struct Ops { u32x4_t a[FBW], b[TB]; };
    auto fetch = [&](int slot, Ops &o) {
        const char *base = plds + slot * STAGE_B + rd;
#pragma unroll
        for (int i = 0; i < FBW; ++i) o.a[i] = *reinterpret_cast<const u32x4_t *>(base + (FBW * half + i) * 32 * FROW_B);
#pragma unroll
        for (int i = 0; i < TB; ++i) o.b[i] = *reinterpret_cast<const u32x4_t *>(base + W_B + i * 32 * FROW_B);
    };
    floatx16 acc[FBW][TB];
#pragma unroll
    for (int fb = 0; fb < FBW; ++fb)
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[fb][tb][r] = 0.f;
    auto multiply = [&](const Ops &o) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb)
#pragma unroll
            for (int fb = 0; fb < FBW; ++fb)
                acc[fb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(o.a[fb]), as_frag(o.b[tb]), acc[fb][tb], 0, 0, 0);
    };

    // Stages 0 .. SLOTS-2 go out ahead; stage 0 has landed when the SLOTS-2 younger ones may be in flight.
#pragma unroll
    for (int s = 0; s < SLOTS - 1; ++s) stage(s, s);
    step_barrier();
    Ops o0, o1;
    fetch(0, o0);
    stage(SLOTS - 1, SLOTS - 1);
    int slot = 0;                                   // of step j
    auto next = [](int s) { return s + 1 == SLOTS ? 0 : s + 1; };
    auto step = [&](int j, const Ops &cur, Ops &nxt) {
        step_barrier();                             // step j+1 has landed; everybody has fetched step j
        const int s1 = next(slot);
        const char *base = plds + s1 * STAGE_B + rd;
        // issue is in order: the step's fetches and loads are dealt out between its MFMAs and pinned there
        constexpr int MM = FBW * TB, SIDE = FBW + TB + PER_WAVE;
#pragma unroll
        for (int m = 0; m < MM; ++m) {
            const int tb = m / FBW, fb = m % FBW;
            acc[fb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_frag(cur.a[fb]), as_frag(cur.b[tb]), acc[fb][tb], 0, 0, 0);
#pragma unroll
            for (int o = m * SIDE / MM; o < (m + 1) * SIDE / MM; ++o) {
                const int ld = (o + 1) * PER_WAVE / SIDE, is_ld = ld != o * PER_WAVE / SIDE, f = o - ld;
                if (is_ld) stage_one(j + SLOTS, slot, ld - 1);
                else if (f < FBW) nxt.a[f] = *reinterpret_cast<const u32x4_t *>(base + (FBW * half + f) * 32 * FROW_B);
                else nxt.b[f - FBW] = *reinterpret_cast<const u32x4_t *>(base + W_B + (f - FBW) * 32 * FROW_B);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        slot = s1;
    };
    int j = 0;
    for (; j + 2 <= nk; j += 2) {
        step(j, o0, o1);
        step(j + 1, o1, o0);
    }
    if (j < nk) multiply(o0);                       // odd number of steps
    // nothing may still be on its way into LDS when it changes its use
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");

    // ---- epilogue, 32 tokens at a time: [kg][token][feature] sums in LDS, 16 bytes of padding per row.  The positions were read
    // before the sweep, the rotary rows of all token blocks are asked for before the first one is joined, and the blocks alternate
    // between two places in LDS, one barrier each: block by block, two dependent round trips and two barriers each cost 16 tokens
    // of 4096 11.8 -> 11.3 us, 96 tokens 16.1 -> 15.1, 384 27.5 -> 26.2, 656 41.2 -> 39.4; the rotation is now as good as free (39.0 without).
    constexpr int JROW = WROWS + 4;                 // floats
    const int c = c0 + my_c;                        // channel of the head, its partner is c + 64
    float4 cs[TB][2];
    if (turned) {
#pragma unroll
        for (int tb = 0; tb < TB; ++tb) {
            const float4 *row = reinterpret_cast<const float4 *>(rope + ((int64_t)my_pos[tb] * (PD / 2) + c) * 2);
            cs[tb][0] = row[0];
            cs[tb][1] = row[1];
        }
    }
    uint16_t *dst;
    int heads_of_dst, h_local;
    if (head < n_q_heads) { dst = q_out; heads_of_dst = n_q_heads; h_local = head; }
    else if (head < n_q_heads + n_kv_heads) { dst = k_out; heads_of_dst = n_kv_heads; h_local = head - n_q_heads; }
    else { dst = v_out; heads_of_dst = n_kv_heads; h_local = head - n_q_heads - n_kv_heads; }
    __syncthreads();
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
        float *join = reinterpret_cast<float *>(plds) + (tb & 1) * (4 * 32 * JROW);
#pragma unroll
        for (int fb = 0; fb < FBW; ++fb)
#pragma unroll
            for (int r4 = 0; r4 < 4; ++r4)
                *reinterpret_cast<float4 *>(join + (kg * 32 + ln) * JROW + 32 * (FBW * half + fb) + 8 * r4 + 4 * hf) =
                    make_float4(acc[fb][tb][4 * r4], acc[fb][tb][4 * r4 + 1], acc[fb][tb][4 * r4 + 2], acc[fb][tb][4 * r4 + 3]);
        __syncthreads();
        const int t = m0 + 32 * tb + my_tok;
        if (my_tok < 32 && t < n_sel) {
            float y1[4] = {0.f, 0.f, 0.f, 0.f}, y2[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const float4 a = *reinterpret_cast<const float4 *>(join + (k * 32 + my_tok) * JROW + my_c);
                const float4 b = *reinterpret_cast<const float4 *>(join + (k * 32 + my_tok) * JROW + 32 * FBW + my_c);
                y1[0] += a.x; y1[1] += a.y; y1[2] += a.z; y1[3] += a.w;
                y2[0] += b.x; y2[1] += b.y; y2[2] += b.z; y2[3] += b.w;
            }
            if (turned) {
                const float4 cs01 = cs[tb][0], cs23 = cs[tb][1];
                const float co[4] = {cs01.x, cs01.z, cs23.x, cs23.z}, sn[4] = {cs01.y, cs01.w, cs23.y, cs23.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const float a = y1[i], b = y2[i];
                    y1[i] = a * co[i] - b * sn[i];
                    y2[i] = b * co[i] + a * sn[i];
                }
            }
            uint16_t *row = dst + ((int64_t)t * heads_of_dst + h_local) * PD + c;
            *reinterpret_cast<uint2 *>(row) = make_uint2(pack_bf16x2(y1[0], y1[1]), pack_bf16x2(y1[2], y1[3]));
            *reinterpret_cast<uint2 *>(row + 64) = make_uint2(pack_bf16x2(y2[0], y2[1]), pack_bf16x2(y2[2], y2[3]));
        }
    }
}

} // namespace

namespace {
struct ProjectArgs {
    const kvs_shape *shape;
    int hidden;
    const void *x;
    int64_t n_tokens;
    const int32_t *x_rows, *sel_pos;
    int64_t n_sel;
    const void *w;
    const float *rope;
    int64_t rope_positions;
    void *q, *k, *v;
};

template <int FBW, int TB>
kvs_status launch_few(const ProjectArgs &a, hipStream_t hs)
{
    constexpr int lds = few_lds_bytes(FBW, TB);
    static DeviceOnce attr_once;
    const kvs_status st = once_per_device(attr_once, [] {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&project_few_kernel<FBW, TB>),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, lds);
        return e == hipSuccess ? KVS_OK : fail(KVS_EHIP, "kvs_project_qkv: hipFuncSetAttribute: %s", hipGetErrorString(e));
    });
    if (st != KVS_OK) return st;
    const int64_t tiles_m = (a.n_sel + 32 * TB - 1) / (32 * TB);
    const int64_t tiles = tiles_m * (a.shape->n_q_heads + 2 * a.shape->n_kv_heads) * (2 / FBW);
    const int64_t per_xcd = (tiles + PXCDS - 1) / PXCDS;
    hipLaunchKernelGGL((project_few_kernel<FBW, TB>), dim3((unsigned)(per_xcd * PXCDS)), dim3(FNT), lds, hs, a.shape->n_q_heads,
                       a.shape->n_kv_heads, a.hidden, (const uint16_t *)a.x, a.n_tokens, a.x_rows, a.sel_pos, (int)a.n_sel,
                       (const uint16_t *)a.w, a.rope, (int)a.rope_positions, (uint16_t *)a.q, (uint16_t *)a.k, (uint16_t *)a.v,
                       (int)tiles_m, (int)tiles, (int)per_xcd);
    return check_launch("kvs_project_qkv(few)");
}

// Which tile.  A launch takes rounds of one workgroup per compute unit, 32 units per XCD; a round costs what its tile
// costs, measured in nanoseconds per 64 of the contraction and per tile (rounds that fill the chip).  The cheapest sum
// is taken, against the 256 x 256 tiles with what rounds after the first cost it besides: a workgroup that follows another
// starts cold, and with more rounds than one every XCD streams the selected rows through its L2 again (without the two, 4 to 44 %
// slower than the large tiles at 2300 to 6600 tokens of 8 to 24 heads and at hidden 512).  Llama-shaped layer, hidden 4096, 256 x 256 tiles -> the choice: 16
// tokens 72 -> 12 us, 96 tokens 73 -> 16, 256 tokens 76 -> 22, 384 tokens 74 -> 26, 640 tokens 76 -> 34, 656 tokens 76 -> 39,
// 1280 tokens 78 -> 65; the large tiles from 1281 on, and the small ones once more where the large ones would start a second
// round for a handful: 2561 to 2688 tokens 175 -> 144 us.  The costs are from before the small tiles' epilogue lost 3 to 6 %, and
// the line is early by that: small against large tiles 71 and 78 us at 1281 tokens, 72 and 78.5 at 1400, 76 and 78.6 at 1500, 77 and
// 82 at 1600, 96 and 84 at 1700 (hidden 1024: 28 and 31 at 1281, 30 and 32 at 1600; 3584 on 28:4 heads: 66 and 71 at 1800, 72 and
// 80 at 2100, where the large tiles are taken as well).
struct FewTile {
    int fbw, tb, step_ns, fixed_ns;
    kvs_status (*launch)(const ProjectArgs &, hipStream_t);
};
constexpr int kLargeStepNs = 1100, kLargeFixedNs = 8000;        // the 256 x 256 kernel
constexpr int kFewRoundNs = 2000, kFewBytesPerNs = 5000;        // a round after the first, and the selected rows if there is one
constexpr int kUnitsPerXcd = 32;
const FewTile few_tiles[] = {
    {1, 1, 150, 2500, launch_few<1, 1>}, {1, 2, 210, 2600, launch_few<1, 2>}, {2, 1, 235, 2600, launch_few<2, 1>},
    {1, 3, 270, 2700, launch_few<1, 3>}, {2, 2, 300, 2800, launch_few<2, 2>}, {2, 3, 410, 3000, launch_few<2, 3>},
    {2, 4, 510, 3300, launch_few<2, 4>}, {2, 5, 590, 3500, launch_few<2, 5>},
};

// NULL: the 256 x 256 kernel
const FewTile *choose_few(const ProjectArgs &a)
{
    const int64_t heads = a.shape->n_q_heads + 2 * a.shape->n_kv_heads, steps = a.hidden / FBK;
    auto rounds = [](int64_t tiles) { return ((tiles + PXCDS - 1) / PXCDS + kUnitsPerXcd - 1) / kUnitsPerXcd; };
    const int64_t large = (a.n_sel + PBM - 1) / PBM * (heads * PD / PBN);
    int64_t best = INT64_MAX, n = 0;
    const FewTile *pick = nullptr;
    for (const FewTile &f : few_tiles) {
        const int64_t tiles = (a.n_sel + 32 * f.tb - 1) / (32 * f.tb) * heads * (2 / f.fbw);
        const int64_t cost = rounds(tiles) * (steps * f.step_ns + f.fixed_ns);
        if (cost < best && tiles <= 0x7fffffff) { best = cost; n = rounds(tiles); pick = &f; }
    }
    if (n > 1) best += (n - 1) * kFewRoundNs + a.n_sel * a.hidden * 2 / kFewBytesPerNs;
    return best < rounds(large) * (steps * kLargeStepNs + kLargeFixedNs) ? pick : nullptr;
}
} // namespace
} // namespace kvs

extern "C" kvs_status kvs_project_qkv(const kvs_shape *shape, int32_t hidden, const void *x, int64_t n_tokens,
                                      const int32_t *x_rows, const int32_t *sel_pos, int64_t n_sel,
                                      const void *w_qkv, const float *rope, int64_t rope_positions,
                                      void *q_out, void *k_out, void *v_out, void *stream)
{
    using namespace kvs;
    kvs_status st = check_shape(shape);
    if (st != KVS_OK) return st;
    if (n_tokens < 0 || n_sel < 0) return fail(KVS_EINVAL, "kvs_project_qkv: negative size");
    if (shape->dtype != KVS_BF16 || shape->head_dim != PD)
        return fail(KVS_EUNSUPPORTED, "kvs_project_qkv: bf16 with head_dim 128 is built");
    if ((shape->n_q_heads + 2 * shape->n_kv_heads) % 2 != 0)
        return fail(KVS_EUNSUPPORTED, "kvs_project_qkv: an odd number of heads in all (a workgroup takes two)");
    if (hidden < 2 * PBK || hidden % (2 * PBK) != 0) return fail(KVS_EUNSUPPORTED, "kvs_project_qkv: hidden size %d (multiples of %d)", hidden, 2 * PBK);
    if (n_sel == 0) return KVS_OK;
    if (n_tokens == 0) return fail(KVS_EINVAL, "kvs_project_qkv: tokens selected from an empty x");
    if (!x_rows && n_sel > n_tokens) return fail(KVS_EINVAL, "kvs_project_qkv: n_sel %lld exceeds the rows of x", (long long)n_sel);
    if (!x || !w_qkv || !q_out || !k_out || !v_out) return fail(KVS_EINVAL, "kvs_project_qkv: NULL tensor pointer");
    if (rope && (!sel_pos || rope_positions <= 0)) return fail(KVS_EINVAL, "kvs_project_qkv: a rotary table needs sel_pos and its own length");
    if (!aligned16(x) || !aligned16(w_qkv) || !aligned16(q_out) || !aligned16(k_out) || !aligned16(v_out) || (rope && !aligned16(rope)))
        return fail(KVS_EINVAL, "kvs_project_qkv: tensors must be 16-byte aligned");
    const int64_t features = (int64_t)(shape->n_q_heads + 2 * shape->n_kv_heads) * PD;
    // rows are addressed with 32-bit byte offsets
    if (n_tokens * hidden * 2 >= ((int64_t)1 << 32) || features * hidden * 2 >= ((int64_t)1 << 32))
        return fail(KVS_EUNSUPPORTED, "kvs_project_qkv: x or w of 4 GiB or more");
    if (n_sel > 0x7fffffff) return fail(KVS_EUNSUPPORTED, "kvs_project_qkv: too many tokens");
    if (rope && rope_positions * (int64_t)(PD * 4) >= ((int64_t)1 << 32)) return fail(KVS_EUNSUPPORTED, "kvs_project_qkv: rotary table of 4 GiB or more");
    const ProjectArgs args = {shape, hidden, x, n_tokens, x_rows, sel_pos, n_sel, w_qkv, rope, rope_positions, q_out, k_out, v_out};
    if (const FewTile *few = choose_few(args)) return few->launch(args, (hipStream_t)stream);
    static DeviceOnce attr_once;
    st = once_per_device(attr_once, [] {
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void *>(&project_qkv_kernel),
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, PLDS_BYTES);
        return e == hipSuccess ? KVS_OK : fail(KVS_EHIP, "kvs_project_qkv: hipFuncSetAttribute: %s", hipGetErrorString(e));
    });
    if (st != KVS_OK) return st;
    const int64_t tiles_m = (n_sel + PBM - 1) / PBM, tiles_n = features / PBN;
    int fx = PXCDS;
    int64_t block_n = 0, block_m = 0;
    for (int f = PXCDS; f >= 1; f >>= 1) {
        const int64_t bn = (tiles_n + f - 1) / f, bm = (tiles_m + PXCDS / f - 1) / (PXCDS / f);
        if (block_n == 0 || bn * bm < block_n * block_m || (bn * bm == block_n * block_m && bn + bm < block_n + block_m)) {
            fx = f; block_n = bn; block_m = bm;
        }
    }
    const int64_t per_xcd = block_n * block_m;
    if (per_xcd * PXCDS > 0x7fffffff) return fail(KVS_EUNSUPPORTED, "kvs_project_qkv: too many tiles");
    hipLaunchKernelGGL(project_qkv_kernel, dim3((unsigned)(per_xcd * PXCDS)), dim3(PNT), PLDS_BYTES, (hipStream_t)stream,
                       shape->n_q_heads, shape->n_kv_heads, (int)hidden, (const uint16_t *)x, n_tokens, x_rows, sel_pos, (int)n_sel,
                       (const uint16_t *)w_qkv, rope, (int)rope_positions, (uint16_t *)q_out, (uint16_t *)k_out, (uint16_t *)v_out,
                       (int)tiles_m, (int)tiles_n, fx, (int)block_n, (int)block_m);
    return check_launch("kvs_project_qkv");
}
