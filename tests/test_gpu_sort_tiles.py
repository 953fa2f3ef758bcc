"""Sort at the edges of its tiles (4,096 keys up to a capacity of 2^18, 8,192
above) and with passes left out: the stable order of numpy, exactly."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _keys(kind, n, rng):
    if kind == "one":            # every pass skipped: copied through
        return np.full(n, 0x80C0FFEE, np.uint32)
    if kind == "top":            # one pass left
        return (rng.integers(0, 256, n, dtype=np.uint32) << 24) | 0x00123456
    if kind == "middle":         # two passes left, and a skipped last one
        return (rng.integers(0, 1 << 16, n, dtype=np.uint32) << 8) | 0x11000022
    return rng.integers(0, 1 << 32, n, dtype=np.uint32)


@pytest.mark.parametrize("kind", ["all", "one", "top", "middle"])
@pytest.mark.parametrize("n,cap", [(1, 1), (1023, 1023), (4095, 4096), (4097, 4097), (4097, 1 << 18),
                                   ((1 << 18) - 1, 1 << 18), (1 << 18, 1 << 18), (8193, (1 << 18) + 1),
                                   ((1 << 18) + 1, (1 << 18) + 1), (0, 5000), (0, 1 << 19)])
def test_sort_tile_edges(kind, n, cap):
    import gpu_util
    print(f"[sort tiles] {kind} n={n} cap={cap}", flush=True)
    rng = np.random.default_rng(n + cap)
    keys, ids = _keys(kind, n, rng), rng.permutation(max(n, 1)).astype(np.uint32)[:n]
    gk, gi = gpu_util.gpu_sort(keys, ids, capacity=cap)
    order = np.argsort(keys, kind="stable")
    assert np.array_equal(gk, keys[order])
    assert np.array_equal(gi, ids[order])
