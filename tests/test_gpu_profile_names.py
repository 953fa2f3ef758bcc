"""crsh_profile_next: every kernel name fires for a frame, at every occurrence
that its stages have, also where one launch does the work of several (a small
sort, rays gathered with the level-1 nodes, a level written and tested)."""
import dataclasses

import pytest

from conftest import workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("w,leaf_hit", [(40, False), (40, True), (110, False)])
def test_names_fire(w, leaf_hit):
    import torch
    from paper_2312_06538_amd import crsh as X
    from paper_2312_06538_amd import pipeline as P
    fr = P.DeviceFrame(dataclasses.replace(workload("shadow_128", W=w, H=40), B=4, F=4, n=5))
    bf, m = P.run_with_retry(fr, P.Buffers(fr, 1 << 20), leaf_hit=leaf_hit)
    steps = int(m.n_levels) - 1                 # levels below the top
    assert steps >= 3 and (fr.max_rays <= 12288) == (w == 40)
    names = [(k, 0) for k in ("k_hash_count", "k_hash_emit", "k_sort_hist", "k_permute", "k_build_leaf", "k_top_count",
                              "k_top_emit", "k_hit", "k_hit_final")]
    names += [("k_sort_pass", i) for i in range(4)] + [("k_level", i) for i in range(steps)]
    names += [("k_level_emit", i) for i in range(steps - leaf_hit)]     # fused: level 1 is not written
    # (what does not fire stays armed until the next call: it comes first, and its
    # events live on)
    kept = []
    for name, occ in [("k_sort_pass", 4), ("k_level", steps), ("k_permute", 1)] + names:
        start, stop, before = (torch.cuda.Event(enable_timing=True) for _ in range(3))
        kept += [start, stop]
        for e in (start, stop, before):
            e.record()
        X.crsh_profile_next(name, occ, start.cuda_event, stop.cuda_event)
        P.run_frame(fr, bf, leaf_hit=leaf_hit)
        torch.cuda.synchronize()
        fired = before.elapsed_time(start) > 0.0
        print(f"[profile] {name} {occ}: {fired}", flush=True)
        assert fired == ((name, occ) in names), (name, occ)
        assert not fired or start.elapsed_time(stop) > 0.0
