"""Hierarchies whose level counts lie at the edge of what one block builds
alone (512 nodes, the upper levels in one launch): bit-exact against the
oracle."""
import numpy as np
import pytest

from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("B,F,n_rays,levels", [(1, 2, 1022, 8), (1, 2, 1024, 8), (1, 2, 1025, 3), (1, 2, 1026, 8),
                                               (2, 4, 4096, 6), (2, 4, 4097, 6), (1, 16, 8193, 4), (3, 5, 7, 4),
                                               (16, 8, 16, 2), (1, 2, 2049, 2)])
def test_build_upper_levels(B, F, n_rays, levels):
    import gpu_util
    print(f"[build tail] B={B} F={F} n={n_rays} levels={levels}", flush=True)
    rng = np.random.default_rng(n_rays)
    r = {k: rng.standard_normal(n_rays).astype(np.float32) for k in O.RAY_FIELDS}
    d = np.stack([r["dx"], r["dy"], r["dz"]]).astype(np.float64)
    d = (d / np.linalg.norm(d, axis=0) * 0.05 + np.array([[0.0], [0.0], [1.0]]))     # narrow cones and wide ones
    d[:, ::7] *= -1.0
    for k, x in zip(("dx", "dy", "dz"), d / np.linalg.norm(d, axis=0)):
        r[k] = x.astype(np.float32)
    r["pix"] = np.arange(n_rays, dtype=np.uint32)
    ids = rng.permutation(n_rays).astype(np.uint32)
    o = O.build_tree(r, ids, B, F, levels)
    g = gpu_util.gpu_build(r, ids, B, F, levels)
    assert g["n_levels"] == o["n_levels"]
    assert np.array_equal(g["level_off"], o["level_off"]) and np.array_equal(g["level_cnt"], o["level_cnt"])
    for k in O.NODE_FIELDS:
        assert np.array_equal(g["nodes"][k].view(np.uint32), o["nodes"][k].view(np.uint32)), k
