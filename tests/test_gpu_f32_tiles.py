"""The fp32 attention and column-mass kernels (fp32, head_dim 64, scales that are not positive) at the edges of their 16-row
tiles, of a wave's 64 keys and of the eight waves' 512, and the scoring kernel's small tiles, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_16525_amd import binding as B
from paper_2503_16525_amd import synth

pytestmark = pytest.mark.gpu

SHAPES = [("f32", 4, 4, 64), ("f32", 6, 2, 128), ("bf16", 10, 2, 64), ("bf16", 3, 1, 128)]


def layer(dtype, hq, hk, d, n):
    return synth.scaled(synth.TINY, n, dtype=dtype, n_q_heads=hq, n_kv_heads=hk, head_dim=d, n_spans=0, span_mean=16.0, coverage=0.8)


@pytest.mark.parametrize("dtype,hq,hk,d", SHAPES)
@pytest.mark.parametrize("n,k", [(1, 1), (16, 16), (17, 5), (64, 16), (65, 17), (128, 128), (129, 40), (512, 33), (513, 8), (1030, 48)])
def test_attention(dtype, hq, hk, d, n, k):
    print(f"fp32 attention: {dtype} {hq}x{hk} heads, head_dim {d}, {k} of {n} tokens", flush=True)
    w = layer(dtype, hq, hk, d, n)
    lay = synth.make_layer(w)
    pos = np.sort(np.random.default_rng(n).permutation(n)[:k]).astype(np.int32)
    pos[-1] = n - 1
    q = lay["q"][torch.from_numpy(pos.astype(np.int64))].contiguous()
    scale = -0.7 if d == 128 and dtype == "bf16" else 1.0
    kc, vc = oracle._as_np(lay["k_cache"]), oracle._as_np(lay["v_cache"])
    ref, lse_ref = oracle.partial_attention(q, pos, kc, vc, scale)
    guard = 3
    out = torch.full((k + guard, hq, d), 7.0, dtype=w.torch_dtype, device="cuda")
    lse = torch.full((k + guard, hq), 7.0, device="cuda")
    B.kvs_partial_attention(B.shape_of(w), [0], [n], [0, k], q.cuda(), torch.from_numpy(pos).cuda(), lay["k_cache"].cuda(),
                            lay["v_cache"].cuda(), scale, out, lse)
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.all(got[k:] == 7.0) and bool((lse[k:] == 7.0).all()), "rows past the last one were written"
    # fp32 products and sums of up to 1030 weights: 1e-5 of the values' size; a bf16 result adds its own rounding
    tol = 1e-5 * (1.0 + np.abs(ref).max()) + (2.0 ** -8 * np.abs(ref) if dtype == "bf16" else 0.0)
    assert np.all(np.abs(got[:k] - ref) <= tol), np.abs(got[:k] - ref).max()
    np.testing.assert_allclose(lse[:k].cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("dtype,hq,hk,d", SHAPES)
@pytest.mark.parametrize("n,lo,k", [(600, 0, 40), (600, 60, 70), (1100, 100, 60), (2500, 0, 300)])
def test_attention_low_in_a_long_context(dtype, hq, hk, d, n, lo, k):
    """Selected tokens that reach a part of the first keys only: most waves have asked for rows that no query sees."""
    print(f"fp32 attention: {dtype} {hq}x{hk} heads, head_dim {d}, tokens {lo}..{lo + k - 1} of {n}", flush=True)
    w = layer(dtype, hq, hk, d, n)
    lay = synth.make_layer(w)
    pos = np.arange(lo, lo + k, dtype=np.int32)
    q = lay["q"][lo:lo + k].contiguous()
    scale = -0.7 if d == 128 and dtype == "bf16" else 1.0
    ref, lse_ref = oracle.partial_attention(q, pos, oracle._as_np(lay["k_cache"]), oracle._as_np(lay["v_cache"]), scale)
    out, lse = torch.full((k + 3, hq, d), 7.0, dtype=w.torch_dtype, device="cuda"), torch.full((k + 3, hq), 7.0, device="cuda")
    B.kvs_partial_attention(B.shape_of(w), [0], [n], [0, k], q.cuda(), torch.from_numpy(pos).cuda(), lay["k_cache"].cuda(), lay["v_cache"].cuda(), scale, out, lse)
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.all(got[k:] == 7.0) and bool((lse[k:] == 7.0).all()), "rows past the last one were written"
    # as above: fp32 products and sums of up to 300 weights; a bf16 result adds its own rounding
    tol = 1e-5 * (1.0 + np.abs(ref).max()) + (2.0 ** -8 * np.abs(ref) if dtype == "bf16" else 0.0)
    assert np.all(np.abs(got[:k] - ref) <= tol), np.abs(got[:k] - ref).max()
    np.testing.assert_allclose(lse[:k].cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("hq,hk,n,k", [(32, 32, 150, 128), (32, 32, 150, 129), (30, 30, 769, 240), (41, 41, 769, 171), (40, 40, 1537, 256), (40, 40, 1537, 257)])
def test_attention_of_many_workgroups(dtype, d, hq, hk, n, k):
    """On both sides of 256 workgroups with a short context, of 450 and 640 with longer ones: a wave's tiles in flight change."""
    print(f"fp32 attention: {dtype} {hq}x{hk} heads, head_dim {d}, {k} of {n} tokens, {(k + 15) // 16 * hk} workgroups", flush=True)
    w = layer(dtype, hq, hk, d, n)
    lay = synth.make_layer(w)
    pos = np.sort(np.random.default_rng(n + k).permutation(n)[:k]).astype(np.int32)
    q = lay["q"][torch.from_numpy(pos.astype(np.int64))].contiguous()
    ref, lse_ref = oracle.partial_attention(q, pos, oracle._as_np(lay["k_cache"]), oracle._as_np(lay["v_cache"]), 1.0)
    out, lse = torch.full((k + 3, hq, d), 7.0, dtype=w.torch_dtype, device="cuda"), torch.full((k + 3, hq), 7.0, device="cuda")
    B.kvs_partial_attention(B.shape_of(w), [0], [n], [0, k], q.cuda(), torch.from_numpy(pos).cuda(), lay["k_cache"].cuda(), lay["v_cache"].cuda(), 1.0, out, lse)
    got = out.float().cpu().numpy().astype(np.float64)
    assert np.all(got[k:] == 7.0) and bool((lse[k:] == 7.0).all()), "rows past the last one were written"
    # as above: fp32 products and sums of up to 1537 weights; a bf16 result adds its own rounding
    tol = 1e-5 * (1.0 + np.abs(ref).max()) + (2.0 ** -8 * np.abs(ref) if dtype == "bf16" else 0.0)
    assert np.all(np.abs(got[:k] - ref) <= tol), np.abs(got[:k] - ref).max()
    np.testing.assert_allclose(lse[:k].cpu().numpy(), lse_ref, rtol=1e-5, atol=1e-5)


@pytest.mark.parametrize("dtype,hq,hk,d", SHAPES)
@pytest.mark.parametrize("at", [0, 15, 16, 50, 130, 400])
def test_attention_hides_what_a_row_does_not_see(dtype, hq, hk, d, at):
    """An Inf or NaN in K or V reaches the rows whose position is at or past it, and no other: bit for bit."""
    print(f"fp32 attention, Inf and NaN at token {at}: {dtype} {hq}x{hk} heads, head_dim {d}", flush=True)
    n, grp = 600, hq // hk
    pos = np.array([0, 3, 14, 15, 16, 17, 49, 50, 51, 129, 130, 131, 200, 399, 400, 401], np.int32)
    w = layer(dtype, hq, hk, d, n)
    lay = synth.make_layer(w)
    q = lay["q"][torch.from_numpy(pos.astype(np.int64))].contiguous().cuda()
    scale = -0.7 if d == 128 and dtype == "bf16" else 1.0

    def run(k, v):
        out, lse = torch.full((len(pos), hq, d), 7.0, dtype=w.torch_dtype, device="cuda"), torch.full((len(pos), hq), 7.0, device="cuda")
        B.kvs_partial_attention(B.shape_of(w), [0], [n], [0, len(pos)], q, torch.from_numpy(pos).cuda(), k, v, scale, out, lse)
        return out.float().cpu().numpy(), lse.cpu().numpy()
    k, v = lay["k_cache"].cuda(), lay["v_cache"].cuda()
    clean, lse_clean = run(k, v)
    assert np.all(np.isfinite(clean))
    # rows of the cache that nothing selected reaches yet
    k1, v1 = k.clone(), v.clone()
    k1[402:], v1[402:] = float("nan"), float("inf")
    out, lse = run(k1, v1)
    np.testing.assert_array_equal(out, clean)
    np.testing.assert_array_equal(lse, lse_clean)
    # single values of one token: the last KV head's channels 5 and 7
    v1 = v.clone()
    v1[at, hk - 1, 5], v1[at, hk - 1, 7] = float("inf"), float("nan")
    want, sees = clean.copy(), pos >= at
    want[sees, (hk - 1) * grp:, 5], want[sees, (hk - 1) * grp:, 7] = np.inf, np.nan
    np.testing.assert_array_equal(run(k, v1)[0], want)
    k1 = k.clone()
    k1[at, 0, 3] = float("nan")
    want, lse_want = clean.copy(), lse_clean.copy()
    want[sees, :grp], lse_want[sees, :grp] = np.nan, np.nan
    out, lse = run(k1, v)
    np.testing.assert_array_equal(out, want)
    np.testing.assert_array_equal(lse, lse_want)


@pytest.mark.parametrize("dtype,hq,hk,d", SHAPES)
@pytest.mark.parametrize("n", [1, 15, 16, 17, 127, 129, 300])
def test_column_mass(dtype, hq, hk, d, n):
    print(f"fp32 column mass: {dtype} {hq}x{hk} heads, head_dim {d}, {n} tokens", flush=True)
    w = layer(dtype, hq, hk, d, n)
    lay = synth.make_layer(w)
    scale = -0.7 if d == 128 and dtype == "bf16" else 1.0
    _, ref = oracle.alpha_prefill(lay["q"], lay["k_fresh"], scale)
    alpha = torch.full((hk + 1, n), 7.0, device="cuda")
    ws = torch.empty(B.kvs_workspace_size("attn_colsum", B.shape_of(w), 1, n), dtype=torch.uint8, device="cuda")
    B.kvs_attn_colsum(B.shape_of(w), n, lay["q"].cuda(), lay["k_fresh"].cuda(), scale, alpha, ws)
    assert bool((alpha[hk] == 7.0).all())
    np.testing.assert_allclose(alpha[:hk].cpu().numpy(), ref, rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("dtype,hq,hk,d", SHAPES)
def test_attention_of_scores_far_below_zero(dtype, hq, hk, d):
    """All scores below -1e34: a row gives the largest, which only one token has, a weight of 1."""
    print(f"fp32 attention, scores below -1e34: {dtype} {hq}x{hk} heads, head_dim {d}", flush=True)
    n, t = 70, torch.float32 if dtype == "f32" else torch.bfloat16
    pos = np.array([0, 1, 40, 69], np.int32)
    q = torch.full((4, hq, d), 2.0 ** 55, dtype=t)
    k = torch.full((n, hk, d), -2.0 ** 55, dtype=t)
    v = torch.randn((n, hk, d), generator=torch.Generator().manual_seed(d)).to(t)
    k[1] *= 0.5                                   # token 1 is the only one with weight for the rows that see it
    sh = B.make_shape(hq, hk, d, B.F32 if dtype == "f32" else B.BF16)
    out, lse = torch.full((4, hq, d), 7.0, dtype=t, device="cuda"), torch.full((4, hq), 7.0, device="cuda")
    scale = 1.0 if d == 64 or dtype == "f32" else -1.0
    B.kvs_partial_attention(sh, [0], [n], [0, 4], q.cuda(), torch.from_numpy(pos).cuda(), k.cuda() * (1.0 if scale > 0 else -1.0), v.cuda(), scale, out, lse)
    want = v[[0, 1, 1, 1]].repeat_interleave(hq // hk, 1)
    assert torch.equal(out.cpu(), want)
    np.testing.assert_allclose(lse[:, 0].cpu().numpy(), -(2.0 ** 110) * d * np.array([1.0, 0.5, 0.5, 0.5]), rtol=1e-6)


@pytest.mark.parametrize("dtype,hq,hk,d", SHAPES)
def test_column_mass_of_scores_far_below_zero(dtype, hq, hk, d):
    """All scores below -1e34: every row that sees token 1 gives it all of its weight."""
    print(f"fp32 column mass, scores below -1e34: {dtype} {hq}x{hk} heads, head_dim {d}", flush=True)
    n, t = 70, torch.float32 if dtype == "f32" else torch.bfloat16
    scale = 1.0 if d == 64 or dtype == "f32" else -1.0
    q, k = torch.full((n, hq, d), 2.0 ** 55, dtype=t), torch.full((n, hk, d), -scale * 2.0 ** 55, dtype=t)
    k[1] *= 0.5
    sh = B.make_shape(hq, hk, d, B.F32 if dtype == "f32" else B.BF16)
    alpha = torch.full((hk, n), 7.0, device="cuda")
    ws = torch.empty(B.kvs_workspace_size("attn_colsum", sh, 1, n), dtype=torch.uint8, device="cuda")
    B.kvs_attn_colsum(sh, n, q.cuda(), k.cuda(), scale, alpha, ws)
    want = np.zeros((hk, n), np.float32)
    want[:, 0], want[:, 1] = hq // hk, (hq // hk) * (n - 1)
    np.testing.assert_array_equal(alpha.cpu().numpy(), want)


@pytest.mark.parametrize("dtype,hq,hk,d", SHAPES)
@pytest.mark.parametrize("row", [0, 7, 15, 16, 100, 255])
def test_column_mass_hides_rows_that_do_not_see_a_key(dtype, hq, hk, d, row):
    """A query row with a NaN or an Inf spoils the mass of the keys that it sees, and of no other: bit for bit."""
    print(f"fp32 column mass, odd query row {row}: {dtype} {hq}x{hk} heads, head_dim {d}", flush=True)
    n = 256
    w = layer(dtype, hq, hk, d, n)
    lay = synth.make_layer(w)
    scale = -0.7 if d == 128 and dtype == "bf16" else 1.0
    k = lay["k_fresh"].cuda()

    def run(q):
        alpha = torch.full((hk, n), 7.0, device="cuda")
        ws = torch.empty(B.kvs_workspace_size("attn_colsum", B.shape_of(w), 1, n), dtype=torch.uint8, device="cuda")
        B.kvs_attn_colsum(B.shape_of(w), n, q, k, scale, alpha, ws)
        return alpha.cpu().numpy()
    q = lay["q"].cuda()
    clean = run(q)
    assert np.all(np.isfinite(clean))
    for odd in ("nan", "inf"):
        q1 = q.clone()
        q1[row, 0, 2] = float(odd)
        got = run(q1)
        assert np.all(np.isnan(got[0, :row + 1]))          # inf - inf or inf * 0 in its softmax
        np.testing.assert_array_equal(got[0, row + 1:], clean[0, row + 1:])
        np.testing.assert_array_equal(got[1:], clean[1:])


# (thousands of tokens with the smaller head counts only)
@pytest.mark.parametrize("dtype,hk,d,n", [(t, hk, d, n) for t, hk, d in [("f32", 4, 64), ("f32", 64, 128), ("bf16", 5, 128), ("bf16", 33, 64)]
                                          for n in [1, 7, 8, 9, 40, 8191, 8192] if n < 1000 or hk <= 5])
@pytest.mark.parametrize("mode", [B.SCORE_V, B.SCORE_KV])
def test_small_scoring_tiles(dtype, hk, d, n, mode):
    print(f"scoring tiles: {dtype} {hk} heads, head_dim {d}, {n} tokens, mode {mode}", flush=True)
    w = layer(dtype, hk, hk, d, n)
    lay = synth.make_layer(w)
    alpha = torch.rand((hk, n), generator=torch.Generator().manual_seed(n)) + 0.5
    dk_ref, dv_ref, sc_ref = oracle.deviation(lay["v_fresh"], lay["v_cache"], lay["k_fresh"], lay["k_cache"], reused=lay["reused"],
                                              alpha=alpha, mode=mode) if mode == B.SCORE_KV else oracle.deviation(
                                                  lay["v_fresh"], lay["v_cache"], reused=lay["reused"], alpha=alpha)
    g = {x: lay[x].cuda() for x in ("k_fresh", "v_fresh", "k_cache", "v_cache", "reused")}
    dev_v, score = torch.full((hk, n), 7.0, device="cuda"), torch.full((n + 64,), 7.0, device="cuda")
    dev_k = torch.full((hk, n), 7.0, device="cuda") if mode == B.SCORE_KV else None
    B.kvs_deviation(B.shape_of(w), n, g["k_fresh"], g["v_fresh"], g["k_cache"], g["v_cache"], g["reused"], alpha.cuda(), mode, dev_k, dev_v, score)
    sc = score.cpu().numpy()
    assert np.all(sc[n:] == 7.0)
    assert np.array_equal(np.isneginf(sc[:n]), np.isneginf(sc_ref))
    fin = np.isfinite(sc_ref)
    np.testing.assert_allclose(sc[:n][fin], sc_ref[fin], rtol=1e-5)          # fp32 sums of at most 128 terms, by head
    np.testing.assert_allclose(dev_v.cpu().numpy(), dv_ref, rtol=1e-5)
    if dev_k is not None:
        np.testing.assert_allclose(dev_k.cpu().numpy(), dk_ref, rtol=1e-5)
