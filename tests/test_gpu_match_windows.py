"""kvs_match_tokens over every kind of window length its doubling hash meets (single bits, all bits, both sides of the staged
limit) and over targets around the 1024 positions of a block, bit for bit against the oracle."""
import numpy as np
import pytest

from test_gpu_match import BASE, MOD, check


pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("w", [1, 2, 3, 4, 5, 6, 7, 8, 15, 16, 17, 31, 32, 33, 63, 64, 65, 127, 255, 256, 257, 511, 512, 513, 767, 768, 769])
@pytest.mark.parametrize("b,m", [(BASE, MOD), (4294967295, 4294967295), (10, 1), (0, 97)])
def test_windows(w, b, m):
    print(f"match: window {w}, base {b}, modulus {m}", flush=True)
    rng = np.random.default_rng(w)
    c = rng.integers(0, 2 ** 31 - 1, size=2000)
    t = rng.integers(0, 2 ** 31 - 1, size=1700)
    t[100:100 + 800] = c[700:1500]
    t[1000:1300] = c[:300]
    if m == 1:                         # every pair of windows has one hash: fewer of them
        t, c = t[:w + 300], c[:w + 200]
    check(t, c, w, b, m)


@pytest.mark.parametrize("n", [1023, 1024, 1025, 2047, 2048, 2049, 3073])
def test_stretches_across_blocks(n):
    print(f"match: {n} positions, one stretch and alternating ones", flush=True)
    rng = np.random.default_rng(n)
    t = rng.integers(0, 10 ** 6, size=n)
    assert check(t, t, 16) == n
    c = t.copy()
    c[::7] = 10 ** 7                    # every seventh token differs: stretches of six
    check(t, c, 3)
    check(t, np.concatenate([t[n // 2:], t[:n // 2]]), 16)


@pytest.mark.parametrize("stretches", [1023, 1024, 1025, 4097])
def test_more_stretches_than_waves(stretches):
    """Stretches of three tokens, each from a place of its own in the candidate: none joins the next."""
    print(f"match: {stretches} stretches", flush=True)
    rng = np.random.default_rng(stretches)
    c = np.arange(3 * stretches)
    t = c.reshape(stretches, 3)[rng.permutation(stretches)].reshape(-1)
    assert check(t, c, 3) == 3 * stretches
