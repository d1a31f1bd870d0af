// Internal declarations shared by the attention translation units (not part of the ABI).
#pragma once

#include "kvs_internal.h"

namespace kvs {

constexpr int kAttnMaxReq = 64; // requests described per launch (passed by value as a kernel argument)

// Host-side request table, copied into the kernel's argument block: no device allocation, no
// asynchronous host-to-device copy whose source would have to outlive the call.
struct AttnBatch {
    int64_t ctx_off[kAttnMaxReq];     // first cache row of request b
    int64_t ctx_len[kAttnMaxReq];     // context rows of request b
    int64_t cu_sel[kAttnMaxReq + 1];  // selected tokens of request b: [cu_sel[b], cu_sel[b+1]) (global numbering)
    int64_t sel_begin;                // first selected token covered by this launch (= cu_sel[0])
    int32_t n_req;
};

// Per-launch table for the matrix-core kernels: request geometry plus the first row tile of each
// request in the launch's grid (row tiles never span requests).
// The entries are the launch's requests ordered by context length, longest last: the kernels take
// row tiles from the end of the table, so the workgroups with the longest sweeps start first and
// the short ones fill the end of the launch.
struct AttnTiles {
    int64_t ctx_off[kAttnMaxReq];
    int64_t sel_lo[kAttnMaxReq];      // first selected token of the entry's request (global numbering)
    int32_t n_sel[kAttnMaxReq];       // and how many
    int32_t ctx_len[kAttnMaxReq];
    int32_t tile_begin[kAttnMaxReq + 1];
    int32_t n_req;
};

// The last request that begins at or before tile t (requests without tiles begin where the next one does), for a t that is the same in every lane and
// a table whose entries past n_req begin where the last request ends.  By quarters, three entries at once: one round trip to the argument
// block up to 4 requests, two up to 16, three for all 64, and no entry is asked for that is far from the others unless there are as many requests.
// Against a walk and against six halvings (whose first, of entry 32, the compiler makes for any number of requests), us: decode checks of up
// to 1000 tokens, 8 requests 22.1, 22.2, 21.9; 16: 25.0, 24.6, 24.3; 64: 41.8, 36.9, 36.7; 40 of up to 2000 41.3, 38.8, 39.1; write-back and
// attention, 2 requests 28.7, 28.9, 28.6; 8: 39.8, 40.4, 39.5 to 40.2; 64: 72.5, 61.6, 61.4.
__device__ __forceinline__ int request_of(const int32_t *tile_begin, int n_req, int t)
{
    static_assert(kAttnMaxReq == 64, "three quarterings");
    if (n_req <= 1) return 0;
    auto upto_t = [t](int begin) { return (int)((uint32_t)(begin - (t + 1)) >> 31); };     // begin <= t, without a detour over vector registers
    int b = 0;
#pragma unroll
    for (int s = 16; s > 0; s /= 4)
        if (n_req > s) b += s * (upto_t(tile_begin[b + s]) + upto_t(tile_begin[b + 2 * s]) + upto_t(tile_begin[b + 3 * s]));
    return b;
}

// The same where lanes ask for different tiles, by halving.  (Only as many steps as n_req asks for: no difference for the shares of 2 to 8 requests.)
__device__ __forceinline__ int request_of_lane(const int32_t *tile_begin, int n_req, int t)
{
    static_assert(kAttnMaxReq <= 64, "six halvings");
    int b = 0;
    if (n_req > 1) {
#pragma unroll
        for (int s = 32; s > 0; s >>= 1)
            if (b + s < n_req && tile_begin[b + s] <= t) b += s;
    }
    return b;
}

// fills `td` for row tiles of `rows_per_tile` flattened (token, head-in-group) rows; returns the
// number of row tiles, or -1 if the grid would overflow
int64_t build_attn_tiles(const kvs_shape *shape, const AttnBatch &bd, int rows_per_tile, AttnTiles &td);

// Key-range splitting (both matrix-core kernels): a piece stores its unnormalised fp32 accumulators
// and (exponent reference, sum of the weights as the matrix core saw them, sum of the unrounded
// weights, unused) per row; slot = row * n_splits + piece.
constexpr size_t kAttnPartBytesPerSlot = 128 * sizeof(float) + 4 * sizeof(float);
constexpr int kAttnSplitMax = 16;
constexpr int kAttnSplitCus = 256;         // compute units a round of pieces is spread over
constexpr int kAttnSplitBelowWgs = 384;    // launches with fewer workgroups than this get split
// start-up (6 us), write-out (4 us) and merge share of a piece, in key tiles; between 18 and 40 it does not matter (12 loses 7 % on 590 of
// 32768 tokens)
constexpr double kAttnPieceOverhead = 18.0;
// Pieces of the 256-row kernel, as the merge sees them: piece s is keys [kAttnPieceKeys * y * (x - 1 - s), kAttnPieceKeys * y * (x - s)) with x, y of
// what attn_plan_kernel left, and only pieces that begin at or before a row's position have left anything for it (a position past its request's context: empty
// records above the context's last piece).
struct AttnMergePlan {
    const int4 *plan;          // nullptr: every one of n_splits slots is filled in, without keys with sum 0
    const int32_t *sel_pos;    // of the first row's token
    int n_q_heads, max_ctx;
};
constexpr int kAttnPieceKeys = 32;
// out = sum_s w_s O_s / sum_s w_s l_s with w_s = 2^(m_s - max m); pieces with l = 0 drop out;
// the log-sum-exp comes from the unrounded sums
kvs_status launch_attention_merge(int64_t n_rows, int n_splits, const float *part_o, const float4 *part_ml,
                                  uint16_t *out, float *lse_out, hipStream_t st, const AttnMergePlan &pieces = {nullptr, nullptr, 1, 1});

// What the host fixes for a split launch of the 256-row kernel: piece slots per row tile (1: no
// cutting, nothing else is read) and the longest context.  Launches too small to fill the chip
// are cut: the size of the pieces is chosen on the device, from the positions, so that the
// pieces just fill whole rounds of the compute units.  Pieces are started from the top of the
// context down, range by range.
// recentre: whole key ranges with a reference that moves where a row's sum outgrows it, for launches
// whose K and V no longer fit the last-level cache (kAttnRecentreBytes).  The look at the sums after
// every tile costs 2 to 5 % of the sweep at any length, and spares the workgroups that meet a logit 111 above
// their first tile's two more sweeps: fixed -> moving, ms, plain and with 200 keys of 40 times the size in
// mid-context: 32768 tokens of 32:8 heads, 15 % selected, 1.13 -> 1.16 and 2.83 -> 1.17; 98304 of 32:4, 10 %,
// 6.81 -> 7.08 and 15.7 -> 7.0; 131072 11.9 -> 12.3 and 26.6 -> 11.9; 131072 of 32:8, 5 %, 6.17 -> 6.52 and
// 15.7 -> 6.5.  So the line is no crossing point.  It lies where such launches used to be cut into pieces of 8192
// keys with a merge, which repeated a piece only (131072 tokens 12.9 and 13.2): beyond it large keys never cost
// more sweeps, and shorter contexts, most of whose launches meet none, keep the plain speed.
struct AttnSplitPlan {
    int n_splits;
    int max_ctx;
    bool recentre;
};
constexpr int64_t kAttnRecentreBytes = (int64_t)192 << 20;   // K + V of a launch's largest request
constexpr int kAttnPlanMaxTiles = 2048;    // row tiles a planned launch may have
// the device-side plan and the list of piece ids (16 bits each, kAttnSplitMax per row tile), after
// the pieces in the workspace
constexpr size_t kAttnPlanBytes = 16 + 2 * (size_t)kAttnSplitMax * kAttnPlanMaxTiles;
static_assert(kAttnSplitMax * kAttnPlanMaxTiles <= 65536, "piece ids are 16 bits");
// 64 query rows per wave (two MFMAs per LDS operand), one wave per SIMD, 256-row tiles.  The plan
// comes from attention_mfma2_plan, which needs the workspace size.
AttnSplitPlan attention_mfma2_plan(const kvs_shape *shape, const AttnBatch &bd, size_t workspace_bytes);
kvs_status launch_attention_mfma2(const kvs_shape *shape, const AttnBatch &bd, const void *q_sel,
                                  const int32_t *sel_pos, const void *k_cache, const void *v_cache,
                                  float scale, void *out, float *lse_out, void *workspace, size_t workspace_bytes,
                                  const AttnSplitPlan &plan, hipStream_t st);

kvs_status launch_attention_f32(const kvs_shape *shape, const AttnBatch &bd, int64_t n_sel,
                                 const void *q_sel, const int32_t *sel_pos, const void *k_cache,
                                 const void *v_cache, float scale, void *out, float *lse_out,
                                 hipStream_t st);

// bf16, head_dim 128 matrix-core path; returns KVS_EUNSUPPORTED for shapes it does not cover
kvs_status launch_attention_mfma(const kvs_shape *shape, const AttnBatch &bd, int64_t n_sel,
                                 const void *q_sel, const int32_t *sel_pos, const void *k_cache,
                                 const void *v_cache, float scale, void *out, float *lse_out,
                                 void *workspace, size_t workspace_bytes, hipStream_t st);
// workspace that lets small launches split their key range (0 bytes still works, unsplit)
size_t attention_workspace_bytes(const kvs_shape *shape, int32_t batch, int64_t n_rows_total, int64_t n_sel_total);
bool attention_mfma_supports(const kvs_shape *shape);

} // namespace kvs
