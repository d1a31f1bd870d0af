"""Launches around the line between pieces and whole key ranges: 256 to 311 row tiles of 256 in pieces, 312 whole; every row
against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from attn_check import check_attention
from paper_2503_16525_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hk,k,order", [(64, 1000, "ascending"), (64, 1024, "shuffled"), (62, 1280, "ascending"), (78, 1024, "ascending"), (52, 1281, "ascending")])
def test_tiles_around_the_line(hk, k, order):
    n = 1300
    print(f"attention: {hk} heads, {k} of {n} tokens, {(k + 255) // 256 * hk} tiles, positions {order}", flush=True)
    rng = np.random.default_rng(hk + k)
    pos = np.sort(rng.permutation(n)[:k]).astype(np.int32)
    if order == "shuffled":
        pos = rng.permutation(pos)
    gen = torch.Generator().manual_seed(k)
    q = (torch.randn((k, hk, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    kk = torch.randn((n, hk, 128), generator=gen).to(torch.bfloat16)
    v = torch.randn((n, hk, 128), generator=gen).to(torch.bfloat16)
    kn, vn = oracle._as_np(kk), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0)
    sh = B.make_shape(hk, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, 1, n, k),), 255, dtype=torch.uint8, device="cuda")
    out = torch.full((k + 2, hk, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((k, hk), 7.0, device="cuda")
    B.kvs_partial_attention(sh, [0], [n], [0, k], q.cuda(), torch.from_numpy(pos).cuda(), kk.cuda(), v.cuda(), 1.0, out, lse, ws)
    got = out.float().cpu().numpy()
    assert np.all(got[k:] == 7.0)
    check_attention(got[:k], ref, mag, "bf16", f"{(k + 255) // 256 * hk} tiles {order}")
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, atol=2e-3)


@pytest.mark.parametrize("grp,order", [(7, "ascending"), (7, "shuffled"), (3, "descending"), (8, "edges")])
def test_pieces_of_a_batch(grp, order):
    """Tokens whose rows lie in two tiles, a request without any, positions at the first and last key of key tiles, in orders that put a
    tile's longest row anywhere."""
    print(f"attention: pieces of a batch, {grp} heads a group, positions {order}", flush=True)
    rng = np.random.default_rng(grp)
    hk, hq = 8, 8 * grp
    length, count = [1500, 1100, 2050, 1025], [770 // grp, 0, 560 // grp, 500 // grp]
    off, cu, pos, rows = [], [0], [], 0
    for n, k in zip(length, count):
        p = np.sort(rng.permutation(n)[:k])
        if order == "edges":
            p = np.sort(np.minimum(n - 1, 32 * rng.integers(0, n // 32 + 1, k) - rng.integers(0, 2, k)).clip(0))
        elif order == "shuffled":
            p = rng.permutation(p)
        elif order == "descending":
            p = p[::-1]
        off.append(rows)
        rows += n + 1
        pos.append(p.astype(np.int32))
        cu.append(cu[-1] + k)
    pos = np.concatenate(pos)
    gen = torch.Generator().manual_seed(grp)
    q = (torch.randn((cu[-1], hq, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    k = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    v = torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16)
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0, off, length, cu)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0, off, length, cu)
    sh = B.make_shape(hq, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, len(off), rows, cu[-1]),), 255, dtype=torch.uint8, device="cuda")
    out = torch.full((cu[-1] + 2, hq, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    lse = torch.full((cu[-1], hq), 7.0, device="cuda")
    B.kvs_partial_attention(sh, off, length, cu, q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, lse, ws)
    got = out.float().cpu().numpy()
    assert np.all(got[cu[-1]:] == 7.0)
    check_attention(got[:cu[-1]], ref, mag, "bf16", f"pieces of a batch, {grp} heads a group, {order}")
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, atol=2e-3)


@pytest.mark.parametrize("hq,hk,n,k", [(64, 64, 1300, 1000), (32, 8, 2050, 700), (21, 3, 3000, 1201)])
def test_rows_leave_whole(hq, hk, n, k):
    """Every row gives one key, another for each row and head, all of its weight: its result is that key's V, bit for bit."""
    print(f"attention: one key a row, {hq}x{hk} heads, {k} of {n} tokens", flush=True)
    rng = np.random.default_rng(hq + k)
    pos = np.sort(rng.permutation(n)[:k]).astype(np.int32)
    gen = torch.Generator().manual_seed(k)
    kk = (torch.randint(0, 2, (n, hk, 128), generator=gen) * 2 - 1).to(torch.bfloat16)
    v = torch.randn((n, hk, 128), generator=gen).to(torch.bfloat16)
    v[v == 0] = 1.0                       # (beside an exact 0 the other keys' e^-40 would show)
    key = torch.from_numpy(rng.integers(0, pos[:, None] + 1, (k, hq)))
    head = torch.arange(hq)[None].expand(k, hq) // (hq // hk)
    q = kk[key, head].contiguous()
    # a score is 128 for the row's key and below 70 for every other of some thousand random signs: with 0.7 as scale their weights are e^-40 at most
    assert max(float((q[:, h].float() @ kk[:, h // (hq // hk)].float().t()).scatter_(1, key[:, h:h + 1], 0).max()) for h in range(hq)) < 70
    sh = B.make_shape(hq, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, 1, n, k),), 255, dtype=torch.uint8, device="cuda")
    out = torch.full((k + 2, hq, 128), 7.0, dtype=torch.bfloat16, device="cuda")
    B.kvs_partial_attention(sh, [0], [n], [0, k], q.cuda(), torch.from_numpy(pos).cuda(), kk.cuda(), v.cuda(), 0.7, out, None, ws)
    assert bool((out[k:] == 7.0).all())
    assert torch.equal(out[:k].cpu(), v[key, head])


@pytest.mark.parametrize("hq,hk,lens,counts", [(1, 1, [13000], [12500]), (2, 1, [4000, 9000], [3000, 7000]),
                                               (16, 2, [900 + 7 * i for i in range(64)], [0 if i in (0, 31, 63) else 17 + i % 15 for i in range(64)]),
                                               (8, 8, [1100 + 50 * i for i in range(9)], [160 + 33 * i for i in range(9)])],
                         ids=["12500 tokens", "10000 tokens of two", "64 requests", "9 requests"])
@pytest.mark.parametrize("order", ["ascending", "shuffled"])
def test_every_position_is_in_the_plan(hq, hk, lens, counts, order):
    """More tokens than the plan reads at once, more requests, some of them without tokens: a row whose reach the plan missed has no top piece."""
    print(f"attention: {sum(counts)} tokens of {len(lens)} requests in pieces, {hq}x{hk} heads, {order}", flush=True)
    rng = np.random.default_rng(sum(counts))
    off, cu, pos, rows = [], [0], [], 0
    for n, k in zip(lens, counts):
        off.append(rows)
        rows += n + 1
        p = np.sort(rng.permutation(n)[:k]).astype(np.int32)
        pos.append(rng.permutation(p) if order == "shuffled" else p)
        cu.append(cu[-1] + k)
    pos = np.concatenate(pos)
    gen = torch.Generator().manual_seed(cu[-1])
    q = (torch.randn((cu[-1], hq, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16)
    k, v = (torch.randn((rows, hk, 128), generator=gen).to(torch.bfloat16) for _ in range(2))
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    ref, lse_ref = oracle.partial_attention(q, pos, kn, vn, 1.0, off, lens, cu)
    mag, _ = oracle.partial_attention(q, pos, kn, vn & np.uint16(0x7FFF), 1.0, off, lens, cu)
    sh = B.make_shape(hq, hk, 128, B.BF16)
    ws = torch.full((B.kvs_workspace_size("partial_attention", sh, len(lens), rows, cu[-1]),), 255, dtype=torch.uint8, device="cuda")
    out, lse = torch.full((cu[-1], hq, 128), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((cu[-1], hq), 7.0, device="cuda")
    B.kvs_partial_attention(sh, off, lens, cu, q.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out, lse, ws)
    check_attention(out.float().cpu().numpy(), ref, mag, "bf16", f"{sum(counts)} tokens of {len(lens)} requests, {order}")
    np.testing.assert_allclose(lse.cpu().numpy(), lse_ref, atol=2e-3)


def test_positions_past_a_short_context():
    """A position past its own request's context, but not past the longest one, is taken as the context's last: the pieces that such a context does not have
    are not read for it."""
    print("attention: positions past a short context, pieces of a batch", flush=True)
    hq, hk, lens, counts = 32, 8, [1100, 3000], [120, 200]
    rng = np.random.default_rng(5)
    off, cu = [0, lens[0] + 1], [0, counts[0], sum(counts)]
    pos = np.concatenate([np.sort(rng.permutation(n)[:k]) for n, k in zip(lens, counts)]).astype(np.int32)
    past = [7, 60, counts[0] - 1]
    pos[past] = lens[0] - 1
    gen = torch.Generator().manual_seed(5)
    q = (torch.randn((cu[-1], hq, 128), generator=gen) / 128 ** 0.5).to(torch.bfloat16).cuda()
    k, v = (torch.randn((sum(lens) + 1, hk, 128), generator=gen).to(torch.bfloat16).cuda() for _ in range(2))
    sh = B.make_shape(hq, hk, 128, B.BF16)
    got = []
    for over in (0, 1, 700, 10 ** 9):
        p = pos.copy()
        p[past] += over
        ws = torch.full((B.kvs_workspace_size("partial_attention", sh, 2, sum(lens) + 1, cu[-1]),), 255, dtype=torch.uint8, device="cuda")
        out, lse = torch.full((cu[-1], hq, 128), 7.0, dtype=torch.bfloat16, device="cuda"), torch.full((cu[-1], hq), 7.0, device="cuda")
        B.kvs_partial_attention(sh, off, lens, cu, q, torch.from_numpy(p).cuda(), k, v, 1.0, out, lse, ws)
        got.append((out, lse))
        assert bool(torch.isfinite(out).all()) and bool(torch.isfinite(lse).all()), over
    assert all(torch.equal(o, got[0][0]) and torch.equal(s, got[0][1]) for o, s in got[1:])
