"""GPU: the decimated subset against the keyed permutation evaluated index
by index on the host (a four-round Feistel network on 2b bits with cycle
walking), at sizes around the 32-particle words and 8192-particle
workgroups, from one kept particle to all of them.  Indices are integers:
the copies are compared bit for bit."""
import numpy as np
import pytest

from paper_1004_1302_amd import learned as LN

pytestmark = pytest.mark.gpu


def mix64(z):
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def kept(n, m, seed):
    half = 1
    while 4 ** half < n:
        half += 1
    h, mask = np.uint64(half), np.uint64((1 << half) - 1)
    with np.errstate(over="ignore"):
        key = mix64(np.uint64(seed) ^ np.uint64(0xD1B54A32D192ED03))
        x = np.arange(n, dtype=np.uint64)
        todo = np.ones(n, bool)
        while todo.any():
            left, r = x[todo] >> h, x[todo] & mask
            for k in range(4):
                f = mix64(key ^ (r * np.uint64(0x9E3779B97F4A7C15)) ^ np.uint64(k << 58)) & mask
                left, r = r, left ^ f
            x[todo] = (left << h) | r
            todo = x >= n
    return np.nonzero(x < m)[0]


@pytest.mark.parametrize("keep", [1, 3, 16, 1000])
@pytest.mark.parametrize("n", [1, 2, 31, 32, 33, 1025, 8191, 8192, 8193, 100_003])
def test_subset_is_the_permutation(n, keep):
    import torch
    rng = np.random.default_rng(n + keep)
    host = {k: rng.uniform(0.1, 1.0, n).astype(np.float32)
            for k in ("x", "y", "z", "h", "value", "value_g")}
    host["species"] = rng.integers(0, 2, n).astype(np.uint8)
    parts = {k: torch.from_numpy(v).cuda() for k, v in host.items()}
    out = {k: v.cpu().numpy() for k, v in LN.decimate(parts, seed=5, keep=keep).items()}
    pick = kept(n, max(1, n // keep), 5)
    scale = np.float32(np.cbrt(float(keep)))
    for k in ("x", "y", "z", "value", "value_g", "species"):
        assert np.array_equal(out[k], host[k][pick]), k
    assert np.array_equal(out["h"], host["h"][pick] * scale)
    assert np.array_equal(out["rho0"], np.full(pick.size, scale, np.float32))
