"""The one-sweep column mass of short fp32 layers: edges of its key tiles, of its two register sizes and of its range, and the
two sweeps that a smaller workspace gets."""
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
