"""Which request a tile belongs to, for as many requests as one launch describes and on both sides of the search's steps (1, 4, 16), with
requests without a context at the front, in between and at the end: decode checks and the attention of selected tokens against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from attn_check import check_attention, check_topk_band
from paper_2503_16525_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hq,hk,d", [("bf16", 8, 2, 128), ("f32", 4, 2, 64)])
@pytest.mark.parametrize("n_req", [2, 3, 4, 5, 8, 15, 16, 17, 20, 32, 33, 48, 49, 63, 64])
def test_requests(dtype, hq, hk, d, n_req):
    print(f"request tables: {n_req} requests, {dtype}", flush=True)
    rng = np.random.default_rng(n_req)
    lens = [int(n) for n in rng.integers(1, 210, n_req)]
    for b in ([], [0, n_req // 2], [0, n_req - 1], [])[n_req % 4]:
        lens[b] = 0
    if not any(lens):
        lens[0] = 77
    want_attn = all(lens)                 # (refused for an empty context)
    off, cu, rows, pos = [], [0], 0, []
    for n in lens:
        off.append(rows)
        rows += n + 2
        k = int(rng.integers(0, min(n, 40) + 1))
        pos.append(np.sort(rng.permutation(n)[:k]).astype(np.int32))
        cu.append(cu[-1] + k)
    pos = np.concatenate(pos)
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    gen = torch.Generator().manual_seed(n_req)
    q, q_sel = ((torch.randn((m, hq, d), generator=gen) / d ** 0.5).to(t) for m in (n_req, cu[-1]))
    k, v = (torch.randn((rows, hk, d), generator=gen).to(t) for _ in range(2))
    dev_v, reused = torch.rand((hk, rows), generator=gen) + 0.1, torch.ones(rows, dtype=torch.uint8)
    sh = B.make_shape(hq, hk, d, B.BF16 if dtype == "bf16" else B.F32)
    ws = torch.full((B.kvs_workspace_size("decode_check", sh, n_req, rows),), 255, dtype=torch.uint8, device="cuda")
    k_req = [n // 9 for n in lens]
    idx, score = torch.full((sum(k_req) + 8,), -7, dtype=torch.int32, device="cuda"), torch.full((rows,), 7.0, device="cuda")
    attn = torch.full((n_req, hq, d), 7.0, dtype=t, device="cuda") if want_attn else None
    B.kvs_decode_check(sh, rows, off, lens, q.cuda(), k.cuda(), v.cuda(), dev_v.cuda(), reused.cuda(), 1.0, k_req, idx, score, attn, ws)
    _, ref, attn_ref = oracle.decode_check(q, k, dev_v, reused, 1.0, off, lens, k_req, v, want_attn)
    if want_attn:
        check_attention(attn.float().cpu().numpy(), attn_ref, None, dtype, f"decode check of {n_req} requests, {dtype}")
    got, got_idx, at = score.cpu().numpy(), idx.cpu().numpy(), 0
    assert np.all(got_idx[sum(k_req):] == -7)
    for o, n, kr in zip(off, lens, k_req):
        np.testing.assert_allclose(got[o:o + n], ref[o:o + n], rtol=1e-5)      # fp32 logits, fp32 softmax
        assert np.all(got[o + n:o + n + 2] == 7.0)
        check_topk_band(got_idx[at:at + kr], ref[o:o + n], kr)
        at += kr
    if cu[-1] == 0:
        return
    kn, vn = oracle._as_np(k), oracle._as_np(v)
    want, _ = oracle.partial_attention(q_sel, pos, kn, vn, 1.0, off, lens, cu)
    mag = oracle.partial_attention(q_sel, pos, kn, vn & np.uint16(0x7FFF), 1.0, off, lens, cu)[0] if dtype == "bf16" else None
    out = torch.full((cu[-1], hq, d), 7.0, dtype=t, device="cuda")
    B.kvs_partial_attention(sh, off, lens, cu, q_sel.cuda(), torch.from_numpy(pos).cuda(), k.cuda(), v.cuda(), 1.0, out)
    check_attention(out.float().cpu().numpy(), want, mag, dtype, f"{n_req} requests, {dtype}")
