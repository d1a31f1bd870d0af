"""Ragged batches with more row tiles than compute units: one workgroup a unit draws its tiles, in the order of their lengths up to 3.5 tiles a unit.
Around that line and the one to fixed shares (8 requests), requests without and with few selected tokens, head counts that leave units over (52: a workgroup
a tile beyond 3.5), more requests than one launch describes, a request beyond the last-level cache; every row against the oracle.  Tiles that run again."""
import numpy as np
import pytest
import torch

import oracle
from attn_check import check_attention
from paper_2503_16525_amd import binding as B

pytestmark = pytest.mark.gpu


def _batch(rng, kind):
    if kind == "15 tiles":        # 64 heads, 4 units each: up to 14 tiles are put in order
        return [(int(rng.integers(300, 900)), int(k)) for k in (256, 1, 300, 0, 255, 257, 40, 256, 256, 290, 3)]
    if kind == "14 tiles":
        return [(int(rng.integers(300, 900)), int(k)) for k in (256, 1, 300, 0, 255, 257, 40, 256, 256, 290)]
    if kind == "8 requests":      # shares
        return [(int(rng.integers(300, 900)), int(k)) for k in (256, 1, 0, 255, 257, 40, 290, 3)]
    if kind == "70 requests":
        return [(int(rng.integers(20, 200)), int(rng.integers(1, 20))) for _ in range(70)]
    return [(6200, 10)] + [(int(rng.integers(50, 100)), int(rng.integers(1, 40))) for _ in range(16)]


@pytest.mark.parametrize("kind,hk,want_lse", [("15 tiles", 64, True), ("15 tiles", 52, False), ("14 tiles", 64, True), ("14 tiles", 52, False), ("8 requests", 64, True), ("70 requests", 64, False), ("large", 64, True),
                                              ("large", 64, False)])
def test_drawn_tiles(kind, hk, want_lse):
    print(f"attention: {kind}, {hk} heads, lse {want_lse}", flush=True)
    rng = np.random.default_rng(hk + len(kind))
    off, length, cu, pos = [], [], [0], []
    rows = 0
    for n, k in _batch(rng, kind):
        off.append(rows)
        length.append(n)
        rows += n + 3
        pos.append(np.sort(rng.permutation(n)[:k]).astype(np.int32))
        cu.append(cu[-1] + k)
    pos = np.concatenate(pos)
    gen = torch.Generator().manual_seed(hk)
    q = (torch.randn((cu[-1], hk, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    k = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    v = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0, off, length, cu)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0, off, length, cu)
    sh = B.make_shape(hk, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, len(off), rows, cu[-1]),), 255, dtype=torch.uint8, device="cuda")
    for _ in range(2):            # the second call finds the first one's queues
        out = torch.full((cu[-1] + 2, hk, 128), 7.0, dtype=torch.bfloat16, device="cuda")
        lse = torch.full((cu[-1], hk), 7.0, device="cuda") if want_lse else None
        B.kvs_partial_attention(sh, off, length, cu, q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, lse, ws)
        got = out.float().cpu().numpy()
        assert np.all(got[cu[-1]:] == 7.0)
        check_attention(got[:cu[-1]], ref, mag, "bf16", f"{kind}, {hk} heads")
        if want_lse:
            np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, atol=2e-3)


@pytest.mark.parametrize("hq,hk,n_req", [(32, 1, 11), (32, 1, 13), (24, 3, 15), (24, 3, 17)])
def test_drawn_tiles_of_few_heads(hq, hk, n_req):
    """No shares are made for more than 64 units a head: on both sides of 1.5 tiles a unit, where the draw begins."""
    n_tokens = 256 if hk == 1 else 248
    print(f"attention: {n_req} requests of {n_tokens} tokens, {hq}x{hk} heads, {n_tokens * hq // hk / 256 * n_req / (256 // hk):.2f} tiles a unit", flush=True)
    rng = np.random.default_rng(hq + n_req)
    lens = [int(n) for n in rng.integers(300, 700, n_req)]
    off, cu = np.cumsum([0] + [n + 3 for n in lens]).tolist(), [n_tokens * i for i in range(n_req + 1)]
    pos = np.concatenate([np.sort(rng.permutation(n)[:n_tokens]) for n in lens]).astype(np.int32)
    gen = torch.Generator().manual_seed(hq)
    q = (torch.randn((cu[-1], hq, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    k, v = (torch.randn((off[-1], hk, 128), generator=gen).to(torch.bfloat16) for _ in range(2))
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0, off[:-1], lens, cu)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0, off[:-1], lens, cu)
    sh = B.make_shape(hq, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, n_req, off[-1], cu[-1]),), 255, dtype=torch.uint8, device="cuda")
    out, lse = torch.full((cu[-1], hq, 128), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((cu[-1], hq), 7.0, device="cuda")
    B.kvs_partial_attention(sh, off[:-1], lens, cu, q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, lse, ws)
    check_attention(out.float().cpu().numpy(), ref, mag, "bf16", f"{n_req} requests, {hq}x{hk} heads")
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, atol=2e-3)


@pytest.mark.parametrize("kind,hk", [("15 tiles", 64), ("14 tiles", 64), ("large", 64)])
@pytest.mark.parametrize("what", ["band", "first"])
def test_drawn_tiles_that_run_again(kind, hk, what):
    """Keys of 60 times the size in every other request (band), or a first tile far below the rest (first), in some of a workgroup's tiles: those run a
    second time, or move their reference, before the next is drawn.  As without a workspace bit for bit, where nothing is drawn."""
    print(f"attention: {kind}, {hk} heads, {what}", flush=True)
    rng = np.random.default_rng(hk + len(kind))
    off, length, cu, pos, rows = [], [], [0], [], 0
    for n, k in _batch(rng, kind):
        off.append(rows)
        length.append(n)
        rows += n + 3
        pos.append(np.sort(rng.permutation(n)[:k]).astype(np.int32))
        cu.append(cu[-1] + k)
    pos = np.concatenate(pos)
    gen = torch.Generator().manual_seed(hk)
    q = torch.randn((cu[-1], hk, 128), generator=gen) / 128 ** 0.5
    k = torch.randn((rows, hk, 128), generator=gen)
    v = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    checked = np.ones(cu[-1], bool)
    if what == "first":
        q[..., 127], k[..., 127] = 1.0, 0.0
    for r, (o, n) in enumerate(zip(off, length)):
        if r % 2:
            continue
        if what == "band":
            k[o + n // 2 : o + n // 2 + 20] *= 60
        else:
            k[o : o + 32, :, 127] = -4e9
            checked[cu[r] : cu[r + 1]] = pos[cu[r] : cu[r + 1]] >= 32        # (before that a row sees nothing but equals, up to rounding)
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0, off, length, cu)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0, off, length, cu)
    sh = B.make_shape(hk, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, len(off), rows, cu[-1]),), 255, dtype=torch.uint8, device="cuda")
    got = []
    for workspace in (ws, None):
        out, lse = torch.full((cu[-1] + 2, hk, 128), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((cu[-1], hk), 7.0, device="cuda")
        B.kvs_partial_attention(sh, off, length, cu, q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, lse, workspace)
        got.append((out, lse))
    out, lse = got[0]
    assert bool((out[cu[-1]:] == 7.0).all())
    check_attention(out[: cu[-1]].float().cpu().numpy()[checked], ref[checked], mag[checked], "bf16", f"{kind}, {hk} heads, {what}")
    np.testing.assert_allclose(lse.cpu().numpy()[checked], lse_ref[checked], rtol=1e-5, atol=2e-3)
    assert torch.equal(out, got[1][0]) and torch.equal(lse, got[1][1])
