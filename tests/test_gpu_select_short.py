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
