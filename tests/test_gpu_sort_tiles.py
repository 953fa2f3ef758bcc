"""Sort at the edges of its tiles (one workgroup up to 12,288 keys; 4,096 keys up
to a capacity of 2^18, 8,192 above) and with passes left out: the stable order of numpy, exactly."""
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
                                   (64, 4096), (4096, 4096), (8191, 8192), (8193, 8193), (12287, 12288),
                                   (12288, 12288), (12289, 12289), (0, 12288),
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


def test_small_batch_frame_digit():
    """A batch of few rays in all: the frame digit too is sorted by the one
    workgroup; every frame against the oracle."""
    import dataclasses
    from conftest import workload
    from oracle import oracle as O
    from paper_2312_06538_amd.batch import DeviceBatch
    wls = [dataclasses.replace(workload("shadow_128", W=w, H=h), B=16, F=4, n=5)
           for w, h in ((40, 40), (3, 3), (24, 17), (40, 30))]
    db = DeviceBatch(wls, 16, 4, 5, 256, pair_capacity=1 << 20)
    assert db.cap <= 12288
    m = db.run_with_retry()
    for f, (r, wl) in enumerate(zip(db.frame_results(m, with_pairs=False), wls)):
        o = O.run_pipeline(wl)
        assert np.array_equal(r["sorted_ids"], o["sorted_ids"]), f
        assert np.array_equal(r["hit"][0], o["hits"][0]), f
