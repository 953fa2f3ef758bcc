"""Batches whose frames are so small that a wave's 64 pixels belong to many:
rays, keys, order and closest hits of every frame exactly the oracle's."""
import dataclasses

import numpy as np
import pytest

from conftest import workload
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("sizes", [[(1, 1)] * 7, [(3, 2), (8, 8), (1, 5), (64, 1), (2, 2)],
                                   [(63, 1), (1, 1), (65, 3), (2, 1), (16, 16), (1, 1)]])
def test_many_frames_in_a_wave(sizes):
    from paper_2312_06538_amd.batch import DeviceBatch
    wls = [dataclasses.replace(workload("refl_1024", W=w, H=h), B=8, F=4, n=4, eye=base_eye(w, h, k))
           for k, (w, h) in enumerate(sizes)]
    db = DeviceBatch(wls, 8, 4, 4, 256, pair_capacity=1 << 20)
    m = db.run_with_retry()
    print(f"[tiny batch] {sizes}: {int(m.n_rays)} rays", flush=True)
    for f, (r, wl) in enumerate(zip(db.frame_results(m, with_pairs=False), wls)):
        o = O.run_pipeline(wl)
        assert r["n"] == o["hash"]["n"], f
        assert np.array_equal(r["keys"], o["hash"]["keys"]), f
        for k in O.RAY_FIELDS:
            assert np.array_equal(r["rays"][k].view(np.uint32), o["hash"]["rays"][k].view(np.uint32)), (f, k)
        assert np.array_equal(r["sorted_ids"], o["sorted_ids"]), f
        assert np.array_equal(r["hit"][0], o["hits"][0]), f


def base_eye(w, h, k):
    """An eye of its own for every frame, so that parameters mixed up between frames show."""
    return workload("refl_1024", W=w, H=h).eye + np.float32(0.125 * k)
