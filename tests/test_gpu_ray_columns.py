"""Ray columns of caller tensors in any layout, fewer rays than the scene holds,
and refusals: the differentiable closest hit gives the same bits for all, and
results of one call are untouched by the next."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _case(n):
    import torch
    from paper_2312_06538_amd.autograd import RayScene
    rng = np.random.default_rng(5)
    verts = rng.uniform(-1, 1, (90, 3)).astype(np.float32)
    faces = np.arange(90, dtype=np.int32).reshape(30, 3)
    o = rng.uniform(-1, 1, (n, 3)).astype(np.float32)
    d = rng.standard_normal((n, 3))
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    sc = lambda: RayScene(faces, [0], [30], (-1, -1, -1), (0.5, 0.5, 0.5), B=8, F=4, levels=3,
                          pair_capacity=1 << 14)
    return [torch.tensor(x, device="cuda") for x in (verts, o, d)], sc


def _run(verts, o, d, scene):
    import torch
    from paper_2312_06538_amd.autograd import ClosestHit
    ins = [x.detach().requires_grad_(True) for x in (verts, o, d)]
    out = ClosestHit.apply(*ins, scene)
    g = torch.autograd.grad([x.sum() for x in out[1:]], ins[1:])
    return list(out) + list(g)


@pytest.mark.parametrize("n", [1, 63, 64, 1000])
def test_layouts_and_smaller_calls(n):
    import torch
    (verts, o, d), sc = _case(n)
    want = _run(verts, o, d, sc())
    scene = sc()
    big = _run(verts, torch.cat([o, o.flip(0)]), torch.cat([d, d]), scene)      # the scene now holds 2 n
    kept = [x.clone() for x in big]
    wide = torch.zeros((n, 5), device="cuda")
    wide[:, 1:4] = o
    for oo in (o, wide[:, 1:4], o.t().contiguous().t()):
        got = _run(verts, oo, d, scene)
        for a, b in zip(got, want):
            assert torch.equal(a, b)
    for a, b in zip(big, kept):
        assert torch.equal(a, b)


def test_refusals():
    (verts, o, d), sc = _case(64)
    scene = sc()
    with pytest.raises(IndexError):
        scene.closest_hit(verts, o[:, :1], d)
    with pytest.raises(RuntimeError):
        scene.closest_hit(verts, o, d[:32])
