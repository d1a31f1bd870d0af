"""The one-sweep column mass of short fp32 layers: edges of its key tiles, of its two register sizes and of its range, the kinds of rows that
it is built for, and the two sweeps that a smaller workspace, or a layer whose shares would be too large, gets."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_16525_amd import binding as B
from paper_2503_16525_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hk,n", [(2, 2, 511), (2, 2, 513), (7, 1, 640), (4, 2, 1025), (2, 1, 2047), (1, 1, 2048), (1, 1, 2049)])
def test_one_sweep_against_the_oracle_and_the_two(hq, hk, n):
    print(f"fp32 column mass: {hq}x{hk} heads, {n} tokens", flush=True)
    w = synth.scaled(synth.TINY, n, n_q_heads=hq, n_kv_heads=hk, n_spans=0, span_mean=16.0, coverage=0.8)
    sh = B.shape_of(w)
    lay = synth.make_layer(w)
    _, ref = oracle.alpha_prefill(lay["q"], lay["k_fresh"], 1.0)
    q, k = lay["q"].cuda(), lay["k_fresh"].cuda()
    rows = (4 * n * hq + 255) // 256 * 256
    for size in (B.kvs_workspace_size("attn_colsum", sh, 1, n), 2 * rows + 256):
        alpha = torch.full((hk + 1, n), 7.0, device="cuda")
        ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")       # NaN wherever something unwritten is read
        B.kvs_attn_colsum(sh, n, q, k, 1.0, alpha, ws)
        assert bool((alpha[hk] == 7.0).all())
        # fp32 scores, exponentials and sums of up to 2049 weights: a few 2^-24 each
        np.testing.assert_allclose(alpha[:hk].cpu().numpy(), ref, rtol=4e-6, atol=1e-7)


@pytest.mark.parametrize("dtype,d,scale", [("f32", 128, 1.0), ("bf16", 64, 1.0), ("bf16", 128, -0.7)])
@pytest.mark.parametrize("hq,hk,n", [(2, 2, 512), (2, 1, 513), (3, 1, 1025), (1, 1, 2047), (2, 2, 2048)])
def test_one_sweep_of_other_rows(dtype, d, scale, hq, hk, n):
    """Other row sizes go through LDS in other pieces, two tiles at a time, and their places are used again."""
    print(f"column mass in one sweep: {dtype}, head_dim {d}, {hq}x{hk} heads, {n} tokens", flush=True)
    w = synth.scaled(synth.TINY, n, dtype=dtype, n_q_heads=hq, n_kv_heads=hk, head_dim=d, n_spans=0, span_mean=16.0, coverage=0.8)
    sh = B.shape_of(w)
    lay = synth.make_layer(w)
    _, ref = oracle.alpha_prefill(lay["q"], lay["k_fresh"], scale)
    alpha = torch.full((hk + 1, n), 7.0, device="cuda")
    ws = torch.full((B.kvs_workspace_size("attn_colsum", sh, 1, n),), 255, dtype=torch.uint8, device="cuda")
    B.kvs_attn_colsum(sh, n, lay["q"].cuda(), lay["k_fresh"].cuda(), scale, alpha, ws)
    assert bool((alpha[hk] == 7.0).all())
    # scores are fp32 sums of 64 or 128 exact products: 1e-6 of the largest, of a few units; exponentials and sums a few 2^-24 each
    np.testing.assert_allclose(alpha[:hk].cpu().numpy(), ref, rtol=1e-5, atol=1e-7)


@pytest.mark.parametrize("hq,n", [(31, 2048), (36, 2048), (36, 2000)])
def test_around_the_largest_shares(hq, n):
    """4 bytes a tile of 16 rows and key, 33.5 MB at most: 31 heads of 2048 tokens take 32.5, in one sweep; 36 would take 37.7, of 2000 tokens 36, and run in two."""
    print(f"column mass: {hq} heads of {n} tokens", flush=True)
    w = synth.scaled(synth.TINY, n, n_q_heads=hq, n_kv_heads=1, n_spans=0, span_mean=16.0, coverage=0.8)
    sh = B.shape_of(w)
    lay = synth.make_layer(w)
    q, k = lay["q"].cuda(), lay["k_fresh"].cuda()
    got = []
    for size in (B.kvs_workspace_size("attn_colsum", sh, 1, n), 2 * ((4 * n * hq + 255) // 256 * 256) + 256):
        alpha = torch.full((2, n), 7.0, device="cuda")
        B.kvs_attn_colsum(sh, n, q, k, 1.0, alpha, torch.full((size,), 255, dtype=torch.uint8, device="cuda"))
        assert bool((alpha[1] == 7.0).all())
        got.append(alpha[0].cpu().numpy())
    # column sums over the heads of the oracle's, head by head
    ref = sum(oracle.alpha_prefill(lay["q"][:, h:h + 1].contiguous(), lay["k_fresh"], 1.0)[1][0] for h in range(hq))
    for alpha in got:
        np.testing.assert_allclose(alpha, ref, rtol=4e-6, atol=1e-7)
    if hq > 31:
        np.testing.assert_array_equal(got[0], got[1])
