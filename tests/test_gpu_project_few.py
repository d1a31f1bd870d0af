"""kvs_project_qkv at the token counts where its tile changes, against the oracle: both sides of every tile edge, one to
three contraction steps (fewer than the staging ring has slots, odd and even), with and without gather and rotation; and
the 256 x 256 tile with a ragged last tile.  Tolerance as in test_gpu_project.py: one bf16 rounding plus the fp32 sums."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_16525_amd import binding as B
from paper_2503_16525_amd import synth

pytestmark = pytest.mark.gpu


def check(hq, hk, hidden, n_sel, gather, rotary):
    n = n_sel + 57 if gather else n_sel
    w = synth.scaled(synth.LLAMA, n, n_q_heads=hq, n_kv_heads=hk)
    x, wt = synth.make_projection(w, hidden)
    rows = np.random.default_rng(n_sel).permutation(n)[:n_sel].astype(np.int32) if gather else None      # any order
    pos = rows if gather else np.arange(n_sel, dtype=np.int32)
    rope = synth.make_rope_table(n, 128) if rotary else None
    ref = oracle.project_qkv(x, wt, hq, hk, 128, rows=rows, pos=pos if rotary else None, rope=rope)
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    # 64 guard rows behind each output
    outs = [torch.full((n_sel + 64, h, 128), 7.0, dtype=torch.bfloat16, device="cuda") for h in (hq, hk, hk)]
    B.kvs_project_qkv(B.shape_of(w), x.cuda(), dev(rows), dev(pos) if rotary else None, n_sel, wt.cuda(), dev(rope), *outs)
    for name, o, r in zip("qkv", outs, ref):
        got = o.float().cpu().numpy().astype(np.float64)
        assert np.all(got[n_sel:] == 7.0), f"{name}: rows past the last token were written"
        err = np.abs(got[:n_sel] - r)
        assert np.all(err <= 2.0 ** -8 * np.abs(r) + 2e-4), f"{name}: max err {err.max():.3e}"


@pytest.mark.parametrize("hidden", [64, 128, 192])
@pytest.mark.parametrize("n_sel", [1, 31, 33, 64, 65, 96, 97, 129, 161, 255, 257, 384, 385, 513, 640, 641, 700])
def test_tile_edges(n_sel, hidden):
    print(f"project few: {n_sel} tokens, hidden {hidden}", flush=True)
    check(32, 8, hidden, n_sel, gather=n_sel % 2 == 1, rotary=hidden != 128)


@pytest.mark.parametrize("n_sel", [5, 100, 481])
def test_other_heads_and_a_longer_contraction(n_sel):
    print(f"project few: {n_sel} tokens, 28x4 and 6x1 heads", flush=True)
    check(28, 4, 1088, n_sel, True, True)
    check(6, 1, 640, n_sel, True, True)


@pytest.mark.parametrize("hq,hk,hidden,n_sel", [(32, 8, 1024, 1000), (32, 8, 4096, 2561), (32, 8, 4096, 2688), (32, 8, 4096, 2689), (6, 2, 1024, 4096), (6, 2, 1024, 5000)])
def test_around_the_rounds(hq, hk, hidden, n_sel):
    """Small tiles of several rounds, and the large tiles on the other side of the rule."""
    print(f"project: {hq}x{hk} heads, hidden {hidden}, {n_sel} tokens", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(n_sel)
    x = torch.randn((n_sel + 9, hidden), generator=gen, device="cuda").to(torch.bfloat16)
    w = (torch.randn(((hq + 2 * hk) * 128, hidden), generator=gen, device="cuda") / hidden ** 0.5).to(torch.bfloat16)
    rows = torch.randperm(n_sel + 9, generator=gen, device="cuda")[:n_sel].to(torch.int32)
    outs = [torch.full((n_sel + 64, h, 128), 7.0, dtype=torch.bfloat16, device="cuda") for h in (hq, hk, hk)]
    B.kvs_project_qkv(B.make_shape(hq, hk, 128, B.BF16), x, rows, None, n_sel, w, None, *outs)
    ref = (x[rows.long()].double() @ w.double().T).view(n_sel, -1, 128)
    for o, r in zip(outs, torch.split(ref, [hq, hk, hk], 1)):
        assert bool((o[n_sel:] == 7.0).all())
        assert bool(((o[:n_sel].double() - r).abs() <= 2.0 ** -8 * r.abs() + 2e-4).all())


def test_large_tile_with_a_ragged_end():
    print("project: 2817 tokens, hidden 1024", flush=True)
    check(32, 8, 1024, 2817, True, True)
