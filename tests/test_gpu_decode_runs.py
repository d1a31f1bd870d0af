"""kvs_decode_check's matrix-core logits launch where its runs of 32-token items have edges: contexts around an item, around
a 64-token tile, empty ones, runs that span several requests, more items than workgroups, head counts that leave waves
without a head or need a second block of heads, group sizes on both sides of the result registers' steps; against the
oracle.  Scores 1e-5 relative (fp32 logits of exact bf16 products, fp32 softmax), index lists checked as a valid top-k."""
import numpy as np
import pytest
import torch

import oracle
from attn_check import check_topk_band
from paper_2503_16525_amd import binding as B
from paper_2503_16525_amd import synth

pytestmark = pytest.mark.gpu

EDGES = [1, 31, 32, 0, 33, 63, 64, 65, 0, 95, 96, 97, 128, 300]
CASES = [
    ("edges-4x8", 32, 8, EDGES),
    ("one-kv-head", 8, 1, EDGES),
    ("three-kv-heads-g3", 9, 3, EDGES),
    ("five-kv-heads", 10, 5, EDGES),
    ("nine-kv-heads", 18, 9, EDGES),
    ("sixteen-kv-heads", 16, 16, EDGES),
    ("group-9", 18, 2, EDGES),
    ("group-16", 16, 1, EDGES),
    ("group-17", 34, 2, EDGES),
    ("group-32", 32, 1, EDGES),
    ("70-requests", 8, 4, [7 + 13 * i for i in range(70)]),
    ("more-items-than-workgroups", 16, 4, [9000, 33, 12000]),
    ("more-items-than-workgroups-of-a-head-block", 24, 12, [9000, 33, 700]),
    ("one-context-with-key-counts", 32, 8, [16500]),
    ("one-context-17-heads-with-key-counts", 34, 17, [12400]),
]


@pytest.mark.parametrize("name,hq,hk,lens", CASES, ids=[c[0] for c in CASES])
def test_runs(name, hq, hk, lens):
    print(f"decode runs: {name}", flush=True)
    d, slack = 128, 3
    rng = torch.Generator().manual_seed(len(name))
    off = np.cumsum([0] + [n + slack for n in lens[:-1]])
    rows = int(off[-1]) + lens[-1] + slack
    q = (torch.randn((len(lens), hq, d), generator=rng) / d ** 0.5).to(torch.bfloat16)
    k = torch.randn((rows, hk, d), generator=rng).to(torch.bfloat16)
    dev_v = torch.rand((hk, rows), generator=rng) + 0.1
    reused = (torch.rand(rows, generator=rng) < 0.9).to(torch.uint8)
    k_req = [min(n, max(0, int(reused[o:o + n].sum()) // 10)) for o, n in zip(off, lens)]
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.full((B.kvs_workspace_size("decode_check", sh, len(lens), rows),), 255, dtype=torch.uint8, device="cuda")
    idx = torch.full((sum(k_req) + 8,), -7, dtype=torch.int32, device="cuda")
    score = torch.full((rows,), 7.0, device="cuda")
    for _ in range(2):                    # the second call finds the workspace as the first left it
        B.kvs_decode_check(sh, rows, off, lens, q.cuda(), k.cuda(), None, dev_v.cuda(), reused.cuda(), 1.0, k_req, idx, score, None, ws)
        _, ref, _ = oracle.decode_check(q, k, dev_v, reused, 1.0, off, lens, k_req)
        got, got_idx, at = score.cpu().numpy(), idx.cpu().numpy(), 0
        assert np.all(got_idx[sum(k_req):] == -7)
        for o, n, kr in zip(off, lens, k_req):
            g, r = got[o:o + n], ref[o:o + n]
            assert np.array_equal(np.isneginf(g), np.isneginf(r))
            fin = np.isfinite(r)
            np.testing.assert_allclose(g[fin], r[fin], rtol=1e-5)
            assert np.all(got[o + n:o + n + slack] == 7.0), "rows outside the contexts were written"
            check_topk_band(got_idx[at:at + kr], r, kr)
            at += kr


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64)])
@pytest.mark.parametrize("lens,bad", [([300, 40, 900], 0), ([40, 9000, 300], 1), ([16500], 0)], ids=["short", "many-records", "key-counts"])
def test_a_nan_in_k_reaches_every_score_of_its_request(dtype, d, lens, bad):
    """The softmax over a context that holds a NaN is NaN: no score of that request may look valid, and the other
    requests' may not change."""
    print(f"decode NaN: {dtype}, head_dim {d}, contexts {lens}", flush=True)
    hq, hk = 8, 2
    t = torch.bfloat16 if dtype == "bf16" else torch.float32
    rng = torch.Generator().manual_seed(d + len(lens))
    off = np.cumsum([0] + lens[:-1]).tolist()
    rows = sum(lens)
    q = (torch.randn((len(lens), hq, d), generator=rng) / d ** 0.5).to(t).cuda()
    k, v = (torch.randn((rows, hk, d), generator=rng).to(t).cuda() for _ in range(2))
    dev_v = (torch.rand((hk, rows), generator=rng) + 0.1).cuda()
    reused = (torch.rand(rows, generator=rng) < 0.9).to(torch.uint8).cuda()
    k_req = [n // 20 for n in lens]
    sh = B.make_shape(hq, hk, d, B.BF16 if dtype == "bf16" else B.F32)
    ws = torch.empty(B.kvs_workspace_size("decode_check", sh, len(lens), rows), dtype=torch.uint8, device="cuda")
    idx = torch.empty(sum(k_req), dtype=torch.int32, device="cuda")

    def check(keys):
        score, out = torch.zeros(rows, device="cuda"), torch.zeros_like(q)
        B.kvs_decode_check(sh, rows, off, lens, q, keys, v, dev_v, reused, 1.0, k_req, idx, score, out, ws)
        return score.cpu().numpy(), out.float().cpu().numpy()
    clean, clean_out = check(k)
    assert np.all(np.isfinite(clean_out))
    for at in (0, lens[bad] // 2, lens[bad] - 1):
        hurt = k.clone()
        hurt[off[bad] + at, 1, 5] = float("nan")
        got, out = check(hurt)
        for r, (o, n) in enumerate(zip(off, lens)):
            g, c = got[o:o + n], clean[o:o + n]
            if r != bad:
                np.testing.assert_array_equal(g, c)
                np.testing.assert_array_equal(out[r], clean_out[r])
            else:
                assert np.all(np.isnan(g[np.isfinite(c)])) and np.all(np.isneginf(g[np.isneginf(c)]))
                np.testing.assert_array_equal(out[r, :hq // 2], clean_out[r, :hq // 2])      # the other KV head's
                assert np.all(np.isnan(out[r, hq // 2:]))


@pytest.mark.parametrize("hq,hk", [(8, 2), (16, 1), (32, 1)])
def test_scores_of_logits_far_below_zero(hq, hk):
    """All logits below -1e34: the request's second token is the only one with weight."""
    print(f"decode, logits below -1e34: {hq}x{hk} heads", flush=True)
    lens, d = [300, 1, 40], 128
    off, rows = [0, 300, 301], 341
    q = torch.full((3, hq, d), 2.0 ** 55, dtype=torch.bfloat16, device="cuda")
    k = torch.full((rows, hk, d), -2.0 ** 55, dtype=torch.bfloat16, device="cuda")
    want = np.zeros(rows, np.float32)
    for o, n in zip(off, lens):
        top = o + min(1, n - 1)
        k[top] *= 0.5
        want[top] = 0.25 * hq
    dev_v = torch.full((hk, rows), 0.25, device="cuda")
    sh = B.make_shape(hq, hk, d, B.BF16)
    ws = torch.empty(B.kvs_workspace_size("decode_check", sh, 3, rows), dtype=torch.uint8, device="cuda")
    idx, score = torch.full((3,), -7, dtype=torch.int32, device="cuda"), torch.zeros(rows, device="cuda")
    B.kvs_decode_check(sh, rows, off, lens, q, k, None, dev_v, None, 1.0, [1, 1, 1], idx, score, None, ws)
    np.testing.assert_array_equal(score.cpu().numpy(), want)
    assert idx.tolist() == [1, 0, 1]
