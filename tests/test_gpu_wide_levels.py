"""Level steps whose child nodes do not fit the LDS copy: a top-level node with
more descendants than it holds, so that every child comes from the node arrays
-- for merge factors on both sides of every lane-group width, ragged last nodes,
storage that ends inside a tile, packed pairs and a batch; and a bound on what
such a hierarchy costs."""
import dataclasses

import numpy as np
import pytest

from conftest import oracle_run, small, workload
from oracle import oracle as O

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _tree(B, F, n):
    base, kw = small("refl_96")
    wl = workload(base, **kw)
    o = oracle_run(base, **kw)
    return wl, O.build_tree(o["hash"]["rays"], o["sorted_ids"], B, F, n)


# the children of a top-level node's descendants on level 2: nf F^(n - 2),
# above the 1,024 of the copy for all of these
@pytest.mark.parametrize("B,F,n", [(4, 2, 11), (4, 3, 8), (4, 4, 7), (2, 5, 6), (4, 8, 5), (8, 9, 4), (2, 16, 4)])
@pytest.mark.parametrize("ends", [False, True])
def test_wide_levels_match_oracle(B, F, n, ends):
    import gpu_util
    wl, tree = _tree(B, F, n)
    e = 900
    ot = O.traverse(tree, wl.scene, 0, e)
    counts = {lv: len(t) for lv, (t, _) in ot["pairs"].items()}
    print(f"[wide levels] B={B} F={F} n={n}: {counts} pairs", flush=True)
    # storage for all, or for one pair past 40 % of the level written last
    cap = counts[1] * 2 // 5 + 1 if ends else max(counts.values()) + 1
    assert cap > 2048
    g = gpu_util.gpu_traverse(tree, wl.scene, B, F, batches=[(0, e)], capacity=cap)
    assert (g["status"] == 0) == (cap > max(counts.values()))
    for lv in range(tree["n_levels"], 0, -1):
        t, nd = ot["pairs"][lv]
        whole = all(counts[k] <= cap for k in range(lv + 1, tree["n_levels"] + 1))
        if not whole:       # the level above was cut: what it holds is a prefix of the whole level
            k = int(min(g["meta"].pairs[lv - 1], cap))
            assert k <= len(t)
        else:
            k = min(len(t), cap)
            assert g["tests"][lv] == ot["tests"][lv] and g["hits"][lv] == len(t), lv
        assert np.array_equal(g["pairs"][lv][0][:k], t[:k]) and np.array_equal(g["pairs"][lv][1][:k], nd[:k]), lv


@pytest.mark.parametrize("B,F,n", [(4, 4, 7), (4, 8, 5)])
def test_wide_packed_and_batched(B, F, n):
    import gpu_util
    from paper_2312_06538_amd.batch import DeviceBatch
    wls = [dataclasses.replace(workload(name, **kw), B=B, F=F, n=n)
           for name, kw in (("refl_1024", dict(W=80, H=60)), ("shadow_128", dict(W=40, H=40)))]
    orcs = [O.run_pipeline(wl) for wl in wls]
    g = gpu_util.run_pipeline(wls[0], keep_levels=False, packed=True)
    assert g["tests"] == orcs[0]["trav"]["tests"] and g["final_tests"] == orcs[0]["trav"]["final_tests"]
    db = DeviceBatch(wls, B, F, n, pair_capacity=1 << 20, keep_levels=True)
    m = db.run_with_retry()
    for f, (r, o) in enumerate(zip(db.frame_results(m), orcs)):
        print(f"[wide batch] B={B} F={F} n={n} frame {f}: {r['n']} rays", flush=True)
        for lv, (t, nd) in o["trav"]["pairs"].items():
            assert np.array_equal(r["pairs"][lv][0], t) and np.array_equal(r["pairs"][lv][1], nd), (f, lv)
        for a, b in zip(r["hit"], o["hits"]):
            assert np.array_equal(np.asarray(a).view(np.uint32), np.asarray(b).view(np.uint32))


def _traverse_us(wl):
    import torch
    from paper_2312_06538_amd import crsh as X
    from paper_2312_06538_amd import pipeline as P
    fr = P.DeviceFrame(wl)
    bf, m = P.run_with_retry(fr, P.Buffers(fr, 1 << 22))
    s, best = P.stream_handle(), float("inf")
    for _ in range(8):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        X.crsh_traverse(bf.c_nodes, fr.scene, 0, fr.m, fr.B, fr.F, bf.c_pairs, bf.meta.data_ptr(), bf.ws.data_ptr(),
                        bf.ws_bytes, s)
        b.record()
        torch.cuda.synchronize()
        best = min(best, a.elapsed_time(b) * 1e3)
    return best, int(m.tests[0])


def test_wide_levels_cost():
    """One level more above the same leaves repeats their tests and adds few:
    with the children read by every lane for itself the traversal took 2 to 3
    times as long, read together about as long."""
    wl = workload("refl_1024", W=192, H=192)
    flat, tests4 = _traverse_us(dataclasses.replace(wl, B=4, F=8, n=4))
    wide, tests5 = _traverse_us(dataclasses.replace(wl, B=4, F=8, n=5))
    print(f"[wide levels] traversal {flat:.0f} us with 512 leaves per top node, {wide:.0f} us with 4096", flush=True)
    assert 0.5 < tests5 / tests4 < 2.0
    assert wide / tests5 < 1.6 * flat / tests4
