"""Contexts whose K and V outgrow the last-level cache: the softmax reference moves where a row's sum of weights outgrows it,
once or several times, by a little or by more than fp32 holds, in an early, a middle and the last tile, in one row or in all.
Every checked row against softmax in 64 bits; the log-sum-exp with it."""
import numpy as np
import pytest
import torch

from paper_2503_16525_amd import binding as B

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.mark.parametrize("want_lse", [False, True])
@pytest.mark.parametrize("what", ["steps", "jump", "one-row", "last", "infinite"])
def test_reference_moves(what, want_lse):
    print(f"recentred attention: {what}, lse {want_lse}", flush=True)
    hq, hk, d, n, k = 64, 8, 128, 49200, 1600             # 201 MB of K and V; 50 row tiles a KV head
    gen = torch.Generator(device=DEV).manual_seed(3)
    kk = torch.randn((n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    v = torch.randn((n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    q = torch.randn((k, hq, d), generator=gen, device=DEV)
    q = (q / q.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    pos = torch.arange(n - k * 30, n, 30, device=DEV, dtype=torch.int32)
    u = q[7, ::8].float()                                 # the direction that the large keys have, by KV head
    if what == "steps":                                   # each 90 above the one before: one move every few tiles
        for i, at in enumerate((40, 1000, 1017, 20000, 40000)):
            kk[at] = (u * 90 * (i + 1)).to(torch.bfloat16)
        q[:] = q[7:8, ::8].repeat_interleave(8, 1)
    elif what == "jump":                                  # far past what fp32 holds, in every row
        kk[25000] = (u * 3000).to(torch.bfloat16)
        q[:] = q[7:8, ::8].repeat_interleave(8, 1)
    elif what == "one-row":
        kk[25000] = (u * 400).to(torch.bfloat16)          # row 7 of a group's first head sees 400, the others a few tens
    elif what == "last":
        kk[n - 31] = (u * 500).to(torch.bfloat16)         # the last row's own tile
        q[:] = q[7:8, ::8].repeat_interleave(8, 1)
    else:
        kk[30011, 3, 5] = float("inf")
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.empty(B.kvs_workspace_size("partial_attention", sh, 1, n, k), dtype=torch.uint8, device=DEV)
    out = torch.full((k, hq, d), 7.0, dtype=torch.bfloat16, device=DEV)
    lse = torch.full((k, hq), 7.0, device=DEV) if want_lse else None
    B.kvs_partial_attention(sh, [0], [n], [0, k], q, pos, kk, v, 1.0, out, lse, ws)
    for h in (0, 7, 8, 26, 29, 63):
        rows = torch.tensor([0, 7, 8, 31, 32, 250, 800, 833, k - 65, k - 64, k - 2, k - 1], device=DEV)
        s = q[rows, h].double() @ kk[:, h // 8].double().t()
        s.masked_fill_(torch.arange(n, device=DEV)[None] > pos[rows, None].long(), -np.inf)
        z = torch.logsumexp(s, -1)
        ref = torch.softmax(s, -1) @ v[:, h // 8].double()
        got = out[rows, h].double()
        fine = torch.isfinite(ref).all(-1)                # (an infinite key: rows whose product with it is +Inf have no finite result,
        assert torch.equal(torch.isfinite(got).all(-1), fine), (what, h)      # the others give it no weight)
        got, ref, z, rows = got[fine], ref[fine], z[fine], rows[fine]
        # weights and results in bf16: two roundings of 2^-9 of values up to max |v|
        assert float((got - ref).abs().max()) <= 2.0 ** -8 * float(v.abs().max()), (what, h)
        if want_lse:
            assert float((lse[rows, h].double() - z).abs().max()) <= 2e-3 + 1e-6 * float(z.abs().max())


@pytest.mark.parametrize("order", ["ascending", "descending", "shuffled"])
def test_reference_moves_among_a_tiles_own_positions(order):
    """Large keys inside the band of positions of a row tile of 32 tokens: inside a lower block of four tokens, between the lower
    and the upper blocks, inside the first upper block and inside the last.  There a wave compares with its positions, or goes on
    with its upper block alone, while the lower one's scores and weights are stale.  Every token of those tiles: the keys
    that it sees count, the others do not.  A short request rides along."""
    print(f"recentred attention: keys among the positions, {order}", flush=True)
    hq, hk, d, n, n2, k, k2 = 64, 8, 128, 49200, 900, 1600, 40
    gen = torch.Generator(device=DEV).manual_seed(9)
    kk = torch.randn((n2 + n, hk, d), generator=gen, device=DEV)
    v = torch.randn((n2 + n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    u = torch.randn(d, generator=gen, device=DEV)
    u = (u / u.norm()).to(torch.bfloat16)
    q = u.expand(k2 + k, hq, d).contiguous()
    pos = torch.arange(n - k * 30, n, 30, device=DEV, dtype=torch.int32)
    at = [int(pos[32 * tile + token]) + past for tile in (1, 24, 49) for token, past in ((2, 5), (15, 10), (18, 7), (29, 3))]
    for i, key in enumerate(at):
        kk[n2 + key] = 100 * (i + 1) * u.float()
    kk[300], kk[700] = 150 * u.float(), 300 * u.float()
    kk = kk.to(torch.bfloat16)
    pos2 = torch.arange(n2 - k2 * 20, n2, 20, device=DEV, dtype=torch.int32)
    if order != "ascending":
        turn = torch.arange(31, -1, -1, device=DEV) if order == "descending" else torch.randperm(32, generator=gen, device=DEV)
        pos = pos.view(-1, 32)[:, turn].reshape(-1)       # within each row tile
        pos2 = pos2.flip(0)
    sel_pos = torch.cat([pos2, pos]).contiguous()
    sh = B.make_shape(hq, hk, d, B.BF16)
    out, lse = torch.full((k2 + k, hq, d), 7.0, dtype=torch.bfloat16, device=DEV), torch.full((k2 + k, hq), 7.0, device=DEV)
    B.kvs_partial_attention(sh, [0, n2], [n2, n], [0, k2, k2 + k], q, sel_pos, kk, v, 1.0, out, lse)
    tiles = torch.cat([torch.arange(32 * t, 32 * t + 32, device=DEV) for t in (0, 1, 2, 24, 25, 49)])
    for h in (0, 29, 63):
        for first, length, rows in ((0, n2, torch.arange(k2, device=DEV)), (n2, n, k2 + tiles)):
            s = q[rows, h].double() @ kk[first : first + length, h // 8].double().t()
            s.masked_fill_(torch.arange(length, device=DEV)[None] > sel_pos[rows, None].long(), -np.inf)
            ref, z = torch.softmax(s, -1) @ v[first : first + length, h // 8].double(), torch.logsumexp(s, -1)
            # weights and results in bf16, as above
            assert float((out[rows, h].double() - ref).abs().max()) <= 2.0 ** -8 * float(v.abs().max()), (h, length)
            assert float((lse[rows, h].double() - z).abs().max()) <= 2e-3 + 1e-6 * float(z.abs().max()), (h, length)


@pytest.mark.parametrize("want_lse", [False, True])
@pytest.mark.parametrize("first", [-np.inf, -1e12, -4e9, -1e6])
def test_a_first_tile_far_below_the_rest(first, want_lse):
    """The first 32 keys give every row logits of `first`; the next tile has one of 150 for half of the heads, whose other logits are
    around 0, while all of the other half's lie around -250.  Neither half may overflow or vanish."""
    print(f"recentred attention: first tile at {first}, lse {want_lse}", flush=True)
    hq, hk, d, n, k = 64, 8, 128, 49200, 1600
    gen = torch.Generator(device=DEV).manual_seed(5)
    kk = torch.randn((n, hk, d), generator=gen, device=DEV)
    v = torch.randn((n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    u, w = torch.zeros(d, device=DEV), torch.zeros(d, device=DEV)
    u[:60], w[60:120] = 60 ** -0.5, 60 ** -0.5
    q = torch.empty((k, hq, d), device=DEV)
    q[:, 0::2], q[:, 1::2] = u, w
    q[:, :, 127] = -0.125
    kk[:, :, 127] = 0
    kk -= 250 * w
    kk[40] += 150 * u
    kk[:32] = 0
    if np.isinf(first):
        kk[:32, :, 127] = np.inf
    else:
        kk[:32] = first * (u + w)
    kk, q = kk.to(torch.bfloat16), q.to(torch.bfloat16)
    pos = torch.arange(n - k * 30, n, 30, device=DEV, dtype=torch.int32)
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.empty(B.kvs_workspace_size("partial_attention", sh, 1, n, k), dtype=torch.uint8, device=DEV)
    out = torch.full((k, hq, d), 7.0, dtype=torch.bfloat16, device=DEV)
    lse = torch.full((k, hq), 7.0, device=DEV) if want_lse else None
    B.kvs_partial_attention(sh, [0], [n], [0, k], q, pos, kk, v, 1.0, out, lse, ws)
    rows = torch.tensor([0, 7, 8, 31, 32, 250, 800, 833, k - 65, k - 64, k - 2, k - 1], device=DEV)
    for h in (0, 1, 30, 31, 63):
        s = q[rows, h].double() @ kk[:, h // 8].double().t()
        s.masked_fill_(torch.arange(n, device=DEV)[None] > pos[rows, None].long(), -np.inf)
        ref = torch.softmax(s, -1) @ v[:, h // 8].double()
        # weights and results in bf16, as above
        assert float((out[rows, h].double() - ref).abs().max()) <= 2.0 ** -8 * float(v.abs().max()), h
        if want_lse:
            z = torch.logsumexp(s, -1)
            assert float((lse[rows, h].double() - z).abs().max()) <= 2e-3 + 1e-6 * float(z.abs().max()), h


def test_a_workspace_changes_nothing():
    """These launches keep whole key ranges and use no workspace: the bits are the same without one, where references move too."""
    print("recentred attention: without a workspace", flush=True)
    hq, hk, d, n, k = 64, 8, 128, 49200, 1600
    gen = torch.Generator(device=DEV).manual_seed(6)
    kk = torch.randn((n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    v = torch.randn((n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    q = torch.randn((k, hq, d), generator=gen, device=DEV)
    q = (q / q.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    kk[24000:24200] *= 60                                 # logits to both sides, a few hundred at most
    pos = torch.arange(n - k * 30, n, 30, device=DEV, dtype=torch.int32)
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.empty(B.kvs_workspace_size("partial_attention", sh, 1, n, k), dtype=torch.uint8, device=DEV)
    res = []
    for workspace in (ws, None):
        out, lse = torch.full((k, hq, d), 7.0, dtype=torch.bfloat16, device=DEV), torch.full((k, hq), 7.0, device=DEV)
        B.kvs_partial_attention(sh, [0], [n], [0, k], q, pos, kk, v, 1.0, out, lse, workspace)
        res.append((out, lse))
    assert torch.isfinite(res[0][0]).all()
    assert torch.equal(res[0][0], res[1][0]) and torch.equal(res[0][1], res[1][1])


def test_the_log_sum_exp_of_a_long_context():
    """One chain of sums over 131072 keys would show in the log-sum-exp.  What remains is its own rounding: log2 of the sum, around -46,
    is rounded to 2^-18 and the result in base 2, around 17, to 2^-19 (each an error of 0.29 units, 7.6e-7 and 3.8e-7 in natural
    units), the result in natural units to 2^-20 (2.8e-7): 8.9e-7 together."""
    print("recentred attention: log-sum-exp of 131072 keys", flush=True)
    hq, hk, d, n, k = 32, 4, 128, 131072, 3072
    gen = torch.Generator(device=DEV).manual_seed(8)
    kk = torch.randn((n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    v = torch.randn((n, hk, d), generator=gen, device=DEV).to(torch.bfloat16)
    q = (torch.randn((k, hq, d), generator=gen, device=DEV) / d ** 0.5).to(torch.bfloat16)
    pos = torch.arange(n - k * 4, n, 4, device=DEV, dtype=torch.int32)
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.empty(B.kvs_workspace_size("partial_attention", sh, 1, n, k), dtype=torch.uint8, device=DEV)
    out, lse = torch.empty((k, hq, d), dtype=torch.bfloat16, device=DEV), torch.full((k, hq), 7.0, device=DEV)
    B.kvs_partial_attention(sh, [0], [n], [0, k], q, pos, kk, v, 1.0, out, lse, ws)
    rows = torch.arange(5, k, 37, device=DEV)
    err = []
    for h in range(0, hq, 3):
        s = q[rows, h].double() @ kk[:, h // 8].double().t()
        s.masked_fill_(torch.arange(n, device=DEV)[None] > pos[rows, None].long(), -np.inf)
        err.append(lse[rows, h].double() - torch.logsumexp(s, -1))
    std = float(torch.cat(err).std())
    print(f"log-sum-exps off by {std:.2e}", flush=True)
    assert std < 1e-6
