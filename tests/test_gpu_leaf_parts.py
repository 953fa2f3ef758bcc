"""Fused last level where a chunk of level-2 pairs has more children than the
workgroup holds (it is taken in parts), and where it has few: closest hits and
counters are those of the stored level-1 pairs, exactly."""
import dataclasses

import numpy as np
import pytest

from conftest import small, workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("B,F,n", [(4, 16, 3), (1, 16, 3), (8, 8, 3), (16, 4, 5), (32, 3, 4), (8, 2, 6)])
def test_leaf_hit_in_parts(B, F, n):
    import gpu_util
    base, kw = small("mixed_128x72")
    wl = dataclasses.replace(workload(base, **kw), B=B, F=F, n=n)
    g = gpu_util.run_pipeline(wl, pair_capacity=1 << 24, keep_levels=False)
    f = gpu_util.run_pipeline(wl, pair_capacity=1 << 24, keep_levels=False, leaf_hit=True)
    print(f"[leaf parts] B={B} F={F}: {g['hits'][2]} level-2 pairs, {g['hits'][1]} level-1 pairs", flush=True)
    for a, b in zip(f["hit"], g["hit"]):
        assert np.array_equal(a.view(np.uint32), b.view(np.uint32))
    for k in ("final_tests", "mesh_tests", "mesh_hits"):
        assert f[k] == g[k], k
    for k in ("final_u_pass", "final_uv_pass"):
        assert getattr(f["meta"], k) == getattr(g["meta"], k), k
    for lv in g["tests"]:
        assert f["tests"][lv] == g["tests"][lv] and f["hits"][lv] == g["hits"][lv], lv
