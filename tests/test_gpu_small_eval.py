"""Evaluations on both sides of the rules that join launches (view and pair
setup in one, the cost summed by the last workgroup): cost, per-pair terms and
gradient against the FP64 oracle at the sizes around each rule, and equal
results on repeated calls and replayed graphs (the tickets start at zero each
time)."""
import numpy as np
import pytest

import oracle
from paper_1806_02637_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def eng():
    import torch

    from paper_1806_02637_amd import engine

    assert torch.cuda.is_available()
    e = engine.Engine(0)
    yield e
    e.close()


def _scan(eng, n_views, dtype="f32"):
    g = inputs.ScanGeometry(n_views, 64, 64, 4.8)
    imgs = inputs.project(g, inputs.random_phantom(2, 6))
    grid = oracle.SinoGrid(g.W, g.H, 90, 91, 0.5)
    sino = oracle.FullSinograms.build(imgs, grid, g.intrinsics())
    scan = eng.load_scan(g.projection_matrices(), g.intrinsics(), imgs)
    scan.set_sinograms(sino.data.astype(np.float32), dtype)
    return g, grid, sino, scan


# one workgroup; 24 and 48 work items (the last the ticket rule takes); 80;
# 2 hypotheses; many hypotheses of few views
@pytest.mark.parametrize("n_views,B", [(2, 1), (16, 1), (24, 1), (25, 1), (16, 2), (9, 40)])
@pytest.mark.parametrize("geom", ["f32", "f64"])
def test_cost_and_gradient(eng, n_views, B, geom):
    print(f"case: small evaluation {n_views} views, B {B}, geom {geom}", flush=True)
    g, grid, sino, scan = _scan(eng, n_views)
    th = inputs.random_motion(3, B, n_views)
    K, R = 64, g.default_object_radius()
    cost, e = scan.cost(th, K, R, geom=geom, with_pairs=True)
    again, _ = scan.cost(th, K, R, geom=geom, with_pairs=True)
    c2, grad = scan.cost_grad(th, K, R, geom=geom)
    cost, again, c2, e = (x.cpu().numpy() for x in (cost, again, c2, e))
    assert np.array_equal(cost, again)
    # the adjoint sums the planes in its own order
    assert np.allclose(c2, cost, rtol=1e-5, atol=0)
    assert np.allclose(e.astype(np.float64).sum(1), cost, rtol=1e-6, atol=0)
    P, intr, prm = g.projection_matrices(), g.intrinsics(), oracle.EccParams(K, R)
    for h in sorted({0, B - 1}):
        ref, e_ref, _, _ = oracle.ecc_cost(P, intr, th[h], grid, sino, prm)
        scale = np.abs(e_ref).max()
        # per pair 2e-4 of its size (nearly equal values cancel in FP32), as in the other tests
        assert np.abs(e[h] - e_ref).max() <= 2e-4 * scale
        assert abs(cost[h] - ref) <= 2e-4 * scale * len(e_ref) ** 0.5 + 1e-5 * ref
    assert np.isfinite(grad.cpu().numpy()).all()
    scan.free()


def test_replayed_graph_equals_eager(eng):
    """A captured cost (one fused setup, tickets) replayed several times on new
    motions, eager work between the replays."""
    import torch

    print("case: small evaluation in a graph", flush=True)
    g, _, _, scan = _scan(eng, 16)
    ths = [torch.as_tensor(inputs.random_motion(s, 1, 16), device="cuda") for s in range(4)]
    K, R = 64, g.default_object_radius()
    eager = [scan.cost(t, K, R).item() for t in ths]
    buf = ths[0].clone()
    ws = scan.workspace(1, False).clone()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        scan.cost(buf, K, R, workspace=ws)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        out = scan.cost(buf, K, R, workspace=ws)
    for t, want in zip(ths * 2, eager * 2):
        buf.copy_(t)
        graph.replay()
        got = out.item()
        assert got == want
        assert scan.cost(t, K, R).item() == want
    scan.free()
