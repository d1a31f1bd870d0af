"""NaN and infinite scores in the matrix-core attention cut into pieces: they reach the rows that see the key, as in launches that keep whole key
ranges, and no other.  64 heads, 1000 of 1300 tokens: 256 tiles of 256 rows in pieces; 8 heads, 40 of 4000: the 128-row kernel's."""
import numpy as np
import pytest
import torch

import oracle
from attn_check import check_attention
from paper_2503_16525_amd import binding as B

pytestmark = pytest.mark.gpu

SHAPES = [(64, 64, 1300, 1000), (8, 8, 4000, 40), (21, 3, 3000, 1201)]


def _call(q, pos, k, v, want_ws=True):
    (k_sel, hq, _), (n, hk, _) = q.shape, k.shape
    sh = B.make_shape(hq, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, 1, n, k_sel),), 255, dtype=torch.uint8, device="cuda") if want_ws else None
    out, lse = torch.full((k_sel, hq, 128), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((k_sel, hq), 7.0, device="cuda")
    B.kvs_partial_attention(sh, [0], [n], [0, k_sel], q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, lse, ws)
    return out.float().cpu().numpy(), lse.cpu().numpy()


def _inputs(hq, hk, n, k_sel):
    rng = np.random.default_rng(hq + k_sel)
    pos = np.sort(rng.permutation(n)[:k_sel]).astype(np.int32)
    gen = torch.Generator().manual_seed(k_sel)
    q = (torch.randn((k_sel, hq, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    q[..., 3] = q[..., 3].abs() + 2.0 ** -7
    k = torch.randn((n, hk, 128), generator=gen).to(torch.bfloat16)
    v = torch.randn((n, hk, 128), generator=gen).to(torch.bfloat16)
    return q, pos, k, v


@pytest.mark.parametrize("hq,hk,n,k_sel", SHAPES)
@pytest.mark.parametrize("odd", [float("nan"), float("inf")])
def test_they_reach_the_rows(hq, hk, n, k_sel, odd):
    q, pos, k, v = _inputs(hq, hk, n, k_sel)
    grp, at = hq // hk, n // 2 + 5
    ref, lse_ref = oracle.partial_attention(q, pos, oracle._as_np(k), oracle._as_np(v), 1.0)
    mag, _ = oracle.partial_attention(q, pos, oracle._as_np(k), oracle._as_np(v) & np.uint16(0x7FFF), 1.0)
    k[at, hk - 1, 3] = odd                                   # one key of the last KV head
    sees = np.zeros((k_sel, hq), bool)
    sees[pos >= at, (hk - 1) * grp:] = True
    for want_ws in (True, False):
        print(f"attention, {odd} in key {at}: {hq}x{hk} heads, {k_sel} of {n} tokens, workspace {want_ws}", flush=True)
        out, lse = _call(q, pos, k, v, want_ws)
        assert np.all(np.isnan(out[sees])) and np.all(np.isnan(lse[sees])), f"{int(np.isfinite(out[sees]).all(-1).sum())} rows hide it"
        # 256 rows run again with exact maxima where one of them has such a score
        check_attention(out[~sees], ref[~sees], mag[~sees], "bf16", f"{odd} in key {at}, {hq}x{hk} heads, workspace {want_ws}: the other rows")
        np.testing.assert_allclose(lse[~sees], lse_ref[~sees], atol=2e-3)


@pytest.mark.parametrize("hq,hk,n,k_sel", SHAPES)
def test_keys_at_minus_infinity_have_no_weight(hq, hk, n, k_sel):
    """Half of the context scores -inf: in a piece that begins there, rows that end before its first ordinary key see nothing else, and
    those that see it run again, all together, with exact maxima."""
    print(f"attention, keys at -inf: {hq}x{hk} heads, {k_sel} of {n} tokens", flush=True)
    q, pos, k, v = _inputs(hq, hk, n, k_sel)
    q[..., 5] = 1.0
    k[..., 5] = 0.0
    gone = slice(n // 4, 3 * n // 4)
    k[gone.stop + 2, :, 5] = 300.0
    k2 = k.clone()
    k2[gone, :, 3] = -torch.inf
    k[gone, :, 5] = -3.0e4               # what the oracle gets in their place
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0)
    for want_ws in (True, False):
        out, lse = _call(q, pos, k2, v, want_ws)
        check_attention(out, ref, mag, "bf16", f"keys at -inf, {hq}x{hk} heads, workspace {want_ws}")
        np.testing.assert_allclose(lse, lse_ref, rtol=1e-5, atol=2e-3)
