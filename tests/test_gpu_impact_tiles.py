"""kvs_first_order_impact (bf16) where its list of reused tokens and its pieces of rows have edges, against the formula in
64-bit torch on the same H and log-sum-exp; with a mask (a list of the reused tokens) and without."""
import numpy as np
import pytest
import torch

from paper_2503_16525_amd import binding as B
from paper_2503_16525_amd import synth

pytestmark = pytest.mark.gpu


def reference(lay, h, lse, grp):
    n = lay["q"].shape[0]
    imp, slack = np.zeros((3, n)), np.zeros(n)
    causal = torch.tril(torch.ones((n, n), dtype=torch.bool))
    for head in range(lay["q"].shape[1]):
        g = head // grp
        q, kf, vf = lay["q"][:, head].double(), lay["k_fresh"][:, g].double(), lay["v_fresh"][:, g].double()
        dk, dv = lay["k_cache"][:, g].double() - kf, lay["v_cache"][:, g].double() - vf
        a = torch.where(causal, torch.exp(q @ kf.T - lse[:, head, None].double()), torch.zeros((), dtype=torch.float64))
        t = q @ dk.T
        x = vf[None] - h[:, head, None].double()                       # [row, token, channel]
        imp[0] += (a.sum(0) * dv.abs().sum(-1)).numpy()
        imp[1] += (a * t.abs() * x.abs().sum(-1)).sum(0).numpy()
        imp[2] += (a * (dv[None] + t[..., None] * x).abs().sum(-1)).sum(0).numpy()
        # t is the difference of two fp32 dot products, each 8 steps of 16 channels whose partial sums stay below
        # sum |q| |k|: off by up to 2 * 8 * 2^-24 of that, whatever is left of t
        kc = lay["k_cache"][:, g].double()
        e = 8 * 2.0 ** -24 * (q.abs() @ kf.abs().T + q.abs() @ kc.abs().T)
        slack += (a * e * x.abs().sum(-1)).sum(0).numpy()
    return imp, (0.0 * slack, slack, slack)


@pytest.mark.parametrize("n,reused_tokens,hq,hk,d", [
    (1, 1, 4, 2, 128), (33, 0, 4, 2, 128), (64, 1, 7, 1, 128), (65, 63, 4, 4, 128), (129, 64, 4, 1, 128), (200, 65, 14, 2, 128),
    (257, 257, 4, 2, 128), (300, 190, 3, 3, 64), (160, 128, 8, 2, 64), (9, 5, 40, 1, 128), (64, 30, 3, 3, 64), (65, 40, 7, 1, 64), (481, 200, 2, 2, 64)])
def test_list_and_piece_edges(n, reused_tokens, hq, hk, d):
    print(f"impact tiles: {n} tokens, {reused_tokens} reused, {hq}x{hk} heads, head_dim {d}", flush=True)
    w = synth.scaled(synth.LLAMA, n, n_q_heads=hq, n_kv_heads=hk, head_dim=d, coverage=1.0)
    lay = synth.make_layer(w)
    picked = np.random.default_rng(n).permutation(n)[:reused_tokens]
    mask = torch.zeros(n, dtype=torch.uint8)
    mask[picked] = 1
    q, k, v = lay["q"].double(), lay["k_fresh"].double(), lay["v_fresh"].double()
    grp = hq // hk
    s = torch.einsum("jhd,ihd->hji", q, k.repeat_interleave(grp, 1)).masked_fill(~torch.tril(torch.ones((n, n), dtype=torch.bool)), -np.inf)
    lse = torch.logsumexp(s, -1).T.contiguous()
    h = torch.einsum("hji,ihd->jhd", torch.softmax(s, -1), v.repeat_interleave(grp, 1)).to(torch.bfloat16).contiguous()
    lse = lse.float()
    ref, slack = reference(lay, h, lse, grp)
    sh = B.shape_of(w)
    full = B.kvs_workspace_size("first_order_impact", sh, 1, n)
    dev = {x: lay[x].cuda() for x in ("q", "k_fresh", "v_fresh", "k_cache", "v_cache")}
    for what, m in (("list", mask), ("no mask", None)):
        out = [torch.full((n,), float("nan"), device="cuda") for _ in range(3)]
        ws = torch.full((full,), 255, dtype=torch.uint8, device="cuda")        # NaN patterns: nothing unwritten may be read
        B.kvs_first_order_impact(sh, n, dev["q"], dev["k_fresh"], dev["v_fresh"], dev["k_cache"], dev["v_cache"], h.cuda(), lse.cuda(),
                                 None if m is None else m.cuda(), 1.0, *out, ws)
        cand = np.ones(n, bool) if m is None else m.numpy() != 0
        for name, o, r, sl in zip(("value", "key", "both"), out, ref, slack):
            got = o.cpu().numpy()
            assert np.array_equal(np.isneginf(got), ~cand), (what, name)
            # fp32: dot products of 128 terms (1e-6 of a logit), the hardware's exp, sums of positive terms
            err = np.abs(got[cand] - r[cand])
            assert np.all(err <= 2e-5 * np.abs(r[cand]) + 1e-6 + sl[cand]), f"{what}: {name}: {err.max()}"
    with pytest.raises(B.KvsError):
        B.kvs_first_order_impact(sh, n, dev["q"], dev["k_fresh"], dev["v_fresh"], dev["k_cache"], dev["v_cache"], h.cuda(), lse.cuda(),
                                 mask.cuda(), 1.0, *out, torch.empty(full - 1, dtype=torch.uint8, device="cuda"))


def small_layer(n, hq, hk, d):
    """The inputs of a call on the device, exact H and log-sum-exp among them."""
    lay = synth.make_layer(synth.scaled(synth.LLAMA, n, n_q_heads=hq, n_kv_heads=hk, head_dim=d, coverage=1.0))
    q, k, v = lay["q"].double(), lay["k_fresh"].double().repeat_interleave(hq // hk, 1), lay["v_fresh"].double().repeat_interleave(hq // hk, 1)
    s = torch.einsum("jhd,ihd->hji", q, k).masked_fill(~torch.tril(torch.ones((n, n), dtype=torch.bool)), -np.inf)
    g = {x: lay[x].cuda() for x in ("q", "k_fresh", "v_fresh", "k_cache", "v_cache")}
    g["h"] = torch.einsum("hji,ihd->jhd", torch.softmax(s, -1), v).to(torch.bfloat16).contiguous().cuda()
    g["lse"] = torch.logsumexp(s, -1).T.contiguous().float().cuda()
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.empty(B.kvs_workspace_size("first_order_impact", sh, 1, n), dtype=torch.uint8, device="cuda")

    def impact(reused=None, **changed):
        a = dict(g, **changed)
        out = [torch.full((n,), 7.0, device="cuda") for _ in range(3)]
        B.kvs_first_order_impact(sh, n, a["q"], a["k_fresh"], a["v_fresh"], a["k_cache"], a["v_cache"], a["h"], a["lse"], reused, 1.0, *out, ws)
        return [o.cpu().numpy() for o in out]
    return g, impact


@pytest.mark.parametrize("hq,hk,d", [(4, 2, 128), (3, 3, 64)])
@pytest.mark.parametrize("share", [1.0, 0.3, 0.02])
def test_a_row_adds_nothing_to_tokens_that_it_does_not_see(hq, hk, d, share):
    """An Inf or NaN in a row's H, Q or log-sum-exp reaches the tokens up to the row, and no other: bit for bit."""
    print(f"impact, odd rows: {hq}x{hk} heads, head_dim {d}, {share} reused", flush=True)
    n = 300
    g, impact = small_layer(n, hq, hk, d)
    mask = (torch.rand(n, generator=torch.Generator().manual_seed(3)) < share).to(torch.uint8)
    mask[[0, 150, 299]] = 1
    cand = mask.numpy() != 0
    mask = mask.cuda()
    clean = impact(mask)
    for row in (0, 31, 150, 298):
        for what, at, reaches in (("h", (row, 1, 5), (False, True, True)), ("q", (row, 1, 5), (True, True, True)), ("lse", (row, 1), (True, True, True))):
            x = g[what].clone()
            x[at] = float("nan")
            for name, a, b, r in zip(("value", "key", "both"), impact(mask, **{what: x}), clean, reaches):
                want = b.copy()
                if r:
                    want[:row + 1][cand[:row + 1]] = np.nan
                np.testing.assert_array_equal(a, want, err_msg=f"{what} of row {row}: {name}")


@pytest.mark.parametrize("hq,hk,d", [(4, 2, 128), (3, 3, 64)])
def test_an_infinite_movement_stays_infinite(hq, hk, d):
    print(f"impact, infinite movement: {hq}x{hk} heads, head_dim {d}", flush=True)
    n = 200
    g, impact = small_layer(n, hq, hk, d)
    clean = impact()
    for i in (0, 1, 64, 100, 199):
        v = g["v_cache"].clone()
        v[i, 0, 3] = float("inf")
        for name, a, b, moved in zip(("value", "key", "both"), impact(v_cache=v), clean, (np.inf, clean[1][i], np.inf)):
            want = b.copy()
            want[i] = moved
            np.testing.assert_array_equal(a, want, err_msg=name)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("hq,hk,d", [(4, 2, 128), (3, 3, 64)])
def test_an_odd_output_row_reaches_only_its_own_sums(hq, hk, d, value):
    """One infinite or NaN element of H: every token that its row sees has an infinite or NaN key term and sum, the later ones
    what they have without it."""
    n, row = 150, 77
    print(f"impact: H with {value} at row {row}, {hq}x{hk} heads, head_dim {d}", flush=True)
    lay = synth.make_layer(synth.scaled(synth.LLAMA, n, n_q_heads=hq, n_kv_heads=hk, head_dim=d, coverage=1.0))
    dev = {x: lay[x].cuda() for x in ("q", "k_fresh", "v_fresh", "k_cache", "v_cache")}
    gen = torch.Generator().manual_seed(n)
    h, lse = (torch.randn((n, hq, d), generator=gen) / 4).to(torch.bfloat16), torch.full((n, hq), 3.0)
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.empty(B.kvs_workspace_size("first_order_impact", sh, 1, n), dtype=torch.uint8, device="cuda")
    res = []
    for odd in (False, True):
        if odd:
            h[row, 1, 5] = value
        out = [torch.zeros(n, device="cuda") for _ in range(3)]
        B.kvs_first_order_impact(sh, n, dev["q"], dev["k_fresh"], dev["v_fresh"], dev["k_cache"], dev["v_cache"], h.cuda(), lse.cuda(), None, 1.0, *out, ws)
        res.append([o.cpu().numpy() for o in out])
    np.testing.assert_array_equal(res[1][0], res[0][0])
    for x, y in zip(res[1][1:], res[0][1:]):
        assert np.all(np.isnan(x[: row + 1]) if np.isnan(value) else x[: row + 1] == np.inf)
        # the same fp32 sums of d terms with their last additions in another order at most
        np.testing.assert_allclose(x[row + 1:], y[row + 1:], rtol=d * 2.0 ** -24)
