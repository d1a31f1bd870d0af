"""kvs_attn_colsum with its sweeps cut into pieces, against the oracle.  Lengths sit at the edges of tiles (32), blocks (256) and pieces; group sizes that do and do not
divide a tile."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_16525_amd import binding as B
from paper_2503_16525_amd import synth

pytestmark = pytest.mark.gpu


def colsum(w, q, k, ws_bytes):
    sh = B.shape_of(w)
    alpha = torch.full((w.n_kv_heads, w.n_ctx), float("nan"), device="cuda")
    ws = torch.empty(ws_bytes, dtype=torch.uint8, device="cuda")
    B.kvs_attn_colsum(sh, w.n_ctx, q.cuda(), k.cuda(), 1.0, alpha, ws)
    return alpha.cpu().numpy()


@pytest.mark.parametrize("hq,hk", [(28, 4), (32, 8), (8, 1), (3, 3)])
@pytest.mark.parametrize("n", [127, 128, 129, 160, 255, 257, 512, 1031])
def test_pieces_against_the_oracle(hq, hk, n):
    print(f"column mass in pieces: {hq}x{hk} heads, {n} tokens", flush=True)
    w = synth.scaled(synth.LLAMA, n, n_q_heads=hq, n_kv_heads=hk, span_mean=64.0)
    lay = synth.make_layer(w)
    q, k = lay["q"], lay["k_fresh"]
    _, ref = oracle.alpha_prefill(q, k, 1.0)
    full = B.kvs_workspace_size("attn_colsum", B.shape_of(w), 1, n)
    cut = colsum(w, q, k, full)
    # fp32 logits of exact bf16 products (1e-6 of a logit of at most ~8), exp2 and log2 to an ulp: some 1e-6 in all
    np.testing.assert_allclose(cut, ref, rtol=2e-5, atol=1e-7)
    np.testing.assert_array_equal(cut, colsum(w, q, k, full))     # no atomics: the same bits again
    with pytest.raises(B.KvsError):
        colsum(w, q, k, full - 1)


def test_a_late_outlier_in_a_later_piece():
    """A key far above its piece's first tile makes that piece repeat with exact maxima; the other pieces do not."""
    n = 1500
    w = synth.scaled(synth.LLAMA, n, span_mean=64.0)
    lay = synth.make_layer(w)
    q, k = lay["q"].clone(), lay["k_fresh"].clone()
    k[1211] = (q[1300, 0].float() / q[1300, 0].float().norm() * 400.0).to(k.dtype)      # logits up to ~ 400
    _, ref = oracle.alpha_prefill(q, k, 1.0)
    sh = B.shape_of(w)
    cut = colsum(w, q, k, B.kvs_workspace_size("attn_colsum", sh, 1, n))
    # logits of ~400 carry an fp32 rounding of 2e-5, relative in a weight
    np.testing.assert_allclose(cut, ref, rtol=2e-4, atol=1e-6)
