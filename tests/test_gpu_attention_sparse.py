"""Sparse selections on the 256-row attention kernel, whole key ranges and pieces: the waves of a workgroup end far apart in
the context, and each stops computing at its own end.  Spread, clustered, few and single tokens, contexts that end inside a
key tile; every row against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from attn_check import check_attention
from paper_2503_16525_amd import binding as B
from paper_2503_16525_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("with_workspace", [False, True], ids=["whole-range", "pieces"])
@pytest.mark.parametrize("hq,hk,want_lse", [(32, 8, True), (28, 4, False)])
def test_sparse_batch(hq, hk, want_lse, with_workspace):
    print(f"sparse attention: {hq}x{hk} heads, workspace {with_workspace}, lse {want_lse}", flush=True)
    rng = np.random.default_rng(hq)
    grp, n_req = hq // hk, 256 // hk + 10
    off, length, cu, pos = [], [], [0], []
    rows = 0
    for r in range(n_req):
        n = int(rng.integers(2300, 2700)) if hk == 8 else int(rng.integers(1300, 1600))
        k = 256 // grp if r % 5 else int(rng.integers(1, 20))
        if r % 3 == 0:
            p = np.sort(rng.permutation(n)[:k])                          # spread
        elif r % 3 == 1:
            p = np.sort(np.concatenate([np.arange(k - k // 2), n - 1 - np.arange(k // 2)]))        # both ends
        else:
            p = np.sort(rng.permutation(n // 8)[:k] + (n // 8) * (r % 7))  # one eighth
        off.append(rows)
        length.append(n)
        rows += n + 5
        pos.append(p.astype(np.int32))
        cu.append(cu[-1] + k)
    pos = np.concatenate(pos)
    gen = torch.Generator().manual_seed(hk)
    q = (torch.randn((cu[-1], hq, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    k = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    v = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0, off, length, cu)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0, off, length, cu)
    sh = B.make_shape(hq, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, n_req, rows, cu[-1]),), 255, dtype=torch.uint8, device="cuda") if with_workspace else None
    out = torch.full((cu[-1] + 2, hq, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((cu[-1], hq), 7.0, device="cuda") if want_lse else None
    B.kvs_partial_attention(sh, off, length, cu, q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, lse, ws)
    got = out.float().cpu().numpy()
    assert np.all(got[cu[-1]:] == 7.0)
    check_attention(got[:cu[-1]], ref, mag, "bf16", f"sparse batch {hq}x{hk} workspace={with_workspace}")
    if want_lse:
        np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, atol=2e-3)


@pytest.mark.parametrize("order", ["descending", "shuffled", "last-first"])
def test_positions_in_any_order(order):
    """A wave's lower and upper block end at its own positions, whichever of the two ends first; rows in an order that no
    selection gives, tiles that are mostly padding among them."""
    print(f"sparse attention: positions {order}", flush=True)
    rng = np.random.default_rng(11)
    hq, hk, n_req = 8, 8, 33
    off, length, cu, pos = [], [], [0], []
    rows = 0
    for r in range(n_req):
        n, k = int(rng.integers(700, 1300)), (256, 40, 256, 150)[r % 4]
        p = np.sort(rng.permutation(n)[:k])
        if order == "descending":
            p = p[::-1]
        elif order == "shuffled":
            p = rng.permutation(p)
        else:
            p = np.concatenate([np.full(33, p[-1]), p[: k - 33]])
        off.append(rows)
        length.append(n)
        rows += n
        pos.append(p.astype(np.int32))
        cu.append(cu[-1] + k)
    pos = np.concatenate(pos)
    gen = torch.Generator().manual_seed(7)
    q = (torch.randn((cu[-1], hq, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    k = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    v = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, _ = oracle.partial_attention(q, pos, kn, vn, 1.0, off, length, cu)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0, off, length, cu)
    sh = B.make_shape(hq, hk, 128, B.BF16)
    out = torch.full((cu[-1] + 2, hq, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    B.kvs_partial_attention(sh, off, length, cu, q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, None, None)
    got = out.float().cpu().numpy()
    assert np.all(got[cu[-1]:] == 7.0)
    check_attention(got[:cu[-1]], ref, mag, "bf16", f"positions {order}")
