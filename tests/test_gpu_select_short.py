"""kvs_select_topk on rows short enough for one wave each, against the oracle: lengths around a multiple of the lanes and around the
lengths at which the kernel's variants change, ties cut and uncut, more entries asked for than there are finite scores."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_16525_amd import binding as B

pytestmark = pytest.mark.gpu
LENGTHS = [1, 2, 63, 64, 65, 255, 256, 257, 511, 512, 513, 767, 768, 769, 1025]


def scores(kind, n, rng):
    if kind == "spread":                    # every exponent, both signs
        return (np.exp(rng.uniform(-80, 80, n)) * rng.choice([-1.0, 1.0], n)).astype(np.float32)
    if kind == "masked":                    # sums of deviations, a third no candidates
        s = (60 + 8 * rng.random(n)).astype(np.float32)
        s[rng.random(n) < 0.33] = -np.inf
        return s
    if kind == "few-values":
        s = rng.integers(-2, 4, n).astype(np.float32)
        s[rng.random(n) < 0.2] = -np.inf
        return s
    if kind == "near":                      # neighbours in the last place: the search goes down to the last bit
        return (np.float32(1.5).view(np.int32) + rng.integers(0, 4, n).astype(np.int32)).view(np.float32)
    return np.full(n, {"equal": 0.25, "none": -np.inf}[kind], np.float32)


@pytest.mark.parametrize("kind", ["spread", "masked", "few-values", "near", "equal", "none"])
@pytest.mark.parametrize("n", LENGTHS)
def test_short_rows(n, kind):
    rng = np.random.default_rng(n)
    ks = sorted({0, 1, n // 7, n // 2, n - 1, n})
    lens = [n if i % 2 == 0 else max(1, n - 1) for i in range(len(ks))]
    ks = [min(k, m) for k, m in zip(ks, lens)]
    off = np.concatenate([[0], np.cumsum(lens)])
    sc = np.concatenate([scores(kind, m, rng) for m in lens])
    print(f"[case] {kind} rows {lens} k {ks}", flush=True)
    idx = torch.full((sum(ks) + 1,), -7, dtype=torch.int32, device="cuda")
    B.kvs_select_topk(torch.from_numpy(sc).cuda(), off.tolist(), ks, idx)
    got = idx.cpu().numpy()
    np.testing.assert_array_equal(got[:-1], oracle.select_topk(sc, off, ks))
    assert got[-1] == -7


@pytest.mark.parametrize("n", [1, 64, 65, 300, 512, 700, 768])
def test_nan_scores_stay_in_their_row(n):
    """NaN scores are a caller's error with unspecified picks: no row writes past its own k entries, what it writes are ascending
    positions of its own, and the rows beside it have their lists."""
    rng = np.random.default_rng(n)
    odd = np.array([0x7FC00000, 0xFFC00000, 0x7F800001, 0xFFFFFFFF, 0x7FFFFFFF], np.uint32).view(np.float32)
    ks = [max(1, n // 3), n, max(1, n // 3), 1, max(1, n // 3)]
    sc = (60 + 8 * rng.random((5, n))).astype(np.float32)
    sc[1, rng.random(n) < 0.5] = odd[3]
    sc[1, 0] = odd[3]
    sc[3] = rng.choice(odd, n)
    some = rng.random(n) < 0.3
    sc[4, some] = rng.choice(odd, int(some.sum()))
    off, cu = [n * r for r in range(6)], np.concatenate([[0], np.cumsum(ks)])
    print(f"[case] NaN scores, rows of {n}, k {ks}", flush=True)
    idx = torch.full((sum(ks) + 1,), -7, dtype=torch.int32, device="cuda")
    B.kvs_select_topk(torch.from_numpy(sc.reshape(-1)).cuda(), off, ks, idx)
    got = idx.cpu().numpy()
    assert got[-1] == -7
    for r in range(5):
        mine = got[cu[r]:cu[r + 1]]
        if r in (0, 2):
            np.testing.assert_array_equal(mine, oracle.select_topk(sc[r], [0, n], [ks[r]]))
        else:
            wrote = mine[mine != -7]
            assert np.all(wrote >= 0) and np.all(wrote < n) and np.all(np.diff(wrote) > 0)
