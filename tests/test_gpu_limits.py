"""GPU checks of the calls at the limits of their arguments and buffers."""
import numpy as np
import pytest

import oracle as O
import synth
from test_gpu_parity import P  # noqa: F401 (the package fixture)

pytestmark = pytest.mark.gpu


# pairs_per_step above 2^31 on a graph whose step's pairs are split between threads: path p receives m |p| pairs,
# none lost and none twice.  One step of length 5: a pair has d = 5 when its two endpoint coins differ (half of
# them; the bound is ten standard deviations) and, laid out at twice its length, stress 1
@pytest.mark.parametrize("m", [2 ** 31 + 1, 2 ** 32 - 1])
def test_sps_draws_every_pair_of_a_huge_count(P, m):  # noqa: F811
    import torch
    sg = synth.SynthGraph(np.array([5], np.uint32), np.array([0, 1], np.uint64), np.array([0], np.uint32), {}, "one")
    g = P.Graph.from_synth(sg)
    c = torch.tensor([0.0, 10.0, 0.0, 0.0], device="cuda")
    r = P.path_stress(g, c, m, 3)
    assert r["n_valid"] + r["n_skipped"] == m
    assert abs(r["n_valid"] - m / 2) < 10 * (m / 4) ** 0.5
    assert r["sum"] == r["n_valid"] and r["mean"] == 1.0 and r["sumsq_dev"] == 0.0


# an infinite upstream gradient (a loss scale that overflowed), in every form of the adjoint: unstaged and staged
# tiles, the image in float, the window-major waves, the plain order.  Two nodes whose pairs all lie further apart
# than their distance: the left node's entries go to -inf and the right node's to +inf, as IEEE division gives
@pytest.mark.parametrize("pairs,window,schedule", [(64, 1000, 3), (20000, 1000, 3), (20000, 9000, 3), (20000, 20000, 3),
                                                   (20000, 30000, 3), (20000, 1000, 1)])
def test_loss_gradient_of_an_infinite_upstream(P, pairs, window, schedule):  # noqa: F811
    import torch
    sg = synth.SynthGraph(np.array([10, 10], np.uint32), np.array([0, 2], np.uint64), np.array([0, 1], np.uint32), {},
                          "two")
    g = P.Graph.from_synth(sg)
    c = torch.tensor([0.0, 30.0, 33.0, 60.0] * 2, device="cuda")
    kw = dict(seed=11, zipf_window=window, schedule=schedule)
    _, nv = P.stress_forward(g, c, pairs, 0, **kw)
    for up in (float("inf"), float("-inf")):
        grad = torch.zeros_like(c)
        P.stress_backward(g, c, pairs, 0, torch.tensor([up], device="cuda"), nv, grad, **kw)
        assert grad.tolist() == [-up, -up, up, up] * 2


def _device_bytes(P, g):  # noqa: F811
    import ctypes
    from paper_2409_00876_amd import _lib
    info = _lib.GraphInfo()
    _lib.check(P.lib().pgsgd_graph_get_info(g.handle, ctypes.byref(info)))
    return int(info.device_bytes)


def test_term_list_gives_way_to_other_buffers(P, monkeypatch):  # noqa: F811
    # a budget that the one-wave layout's list fills: the metric of two layouts, the window-major metric and the loss
    # still find room for their buffers, and the layout is the same bit for bit with the list and without
    import torch
    sg = synth.generate(1500, 0.2, 8, 23)
    g = P.Graph.from_synth(sg)
    first = P.init_coords(g, g.new_coords())
    P.sample_terms(g, 0, 0, 64)  # the window tables; the recording hook takes no list
    tables = _device_bytes(P, g)
    P.layout(g, first, n_iters=4)
    cap = _device_bytes(P, g)
    assert cap > tables
    monkeypatch.setenv("PGSGD_MAX_DEVICE_BYTES", str(cap))
    again = P.init_coords(g, g.new_coords())
    P.layout(g, again, n_iters=4)
    assert torch.equal(first, again) and _device_bytes(P, g) == cap
    r = P.path_stress_compare(g, first, again, 5)
    assert r["ratio"] == 1.0 and _device_bytes(P, g) <= cap
    P.path_stress(g, first, 5, pairs="uniform_windowed")
    loss, nv = P.stress_forward(g, first, 5000, 0)
    P.stress_backward(g, first, 5000, 0, torch.ones(1, device="cuda"), nv, torch.zeros_like(first))
    assert _device_bytes(P, g) <= cap
    P.init_coords(g, again)
    P.layout(g, again, n_iters=4)
    torch.cuda.synchronize()
    assert torch.equal(first, again) and _device_bytes(P, g) <= cap


def test_captured_layout_outlives_the_term_list(P):  # noqa: F811
    # a captured one-wave layout, larger than any before it, replayed around eager layouts that grow the list
    import torch
    sg = synth.generate(700, 0.2, 4, 29)
    g = P.Graph.from_synth(sg)
    c, ref = g.new_coords(), g.new_coords()
    kw = dict(n_iters=4, terms_per_step=20)
    P.init_coords(g, ref)
    P.layout_noalloc(g, ref, **kw)
    P.init_coords(g, c)
    P.layout(g, c, n_iters=4, terms_per_step=2)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        P.init_coords(g, c)
        P.layout(g, c, **kw)
    other = g.new_coords()
    for terms in (0, 30, 60):
        if terms:
            P.init_coords(g, other)
            P.layout(g, other, n_iters=4, terms_per_step=terms)
        c.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c, ref)
    P.init_coords(g, c)
    P.layout(g, c, **kw)
    torch.cuda.synchronize()
    assert torch.equal(c, ref)


def test_exact_path_stress_with_the_most_paths(P):  # noqa: F811
    # 16,000 paths: their table and the kernel's own tiles together still fit a block's LDS; twice as many do not
    import torch
    for n_paths in (16000, 33000):
        sg = synth.SynthGraph(np.full(100, 5, np.uint32), (2 * np.arange(n_paths + 1)).astype(np.uint64),
                              (np.arange(2 * n_paths) % 100).astype(np.uint32), {}, "many-paths")
        og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg)
        c = O.init_coords(og) + np.random.default_rng(3).normal(scale=4.0, size=400).astype(np.float32)
        if n_paths > 16384:
            with pytest.raises(P.PgsgdError, match="too many paths"):
                P.path_stress_exact(g, torch.from_numpy(c).cuda())
            continue
        mean, pairs = P.path_stress_exact(g, torch.from_numpy(c).cuda())
        ref = O.path_stress_exact(og, c)
        assert pairs == ref[1] == n_paths and abs(mean - ref[0]) <= 1e-9 * abs(ref[0])


# an infinite coordinate in every form of the tiles (unstaged and staged, the image in double and in float, beyond the
# tiles) and in the plain order: the loss is infinite where a pair names its endpoint and unmoved where none does; the
# gradient is NaN where a pair reaches it, as in the oracle's FP64, and the oracle's elsewhere
@pytest.mark.parametrize("backbone,paths,pairs,window,renumber,schedule", [
    (300, 3, 40, 1000, "auto", 3), (9000, 5, 200, 1000, "auto", 3), (900, 4, 60000, 1000, "auto", 3),
    (9000, 5, 300000, 1000, "always", 3), (9000, 5, 100003, 9000, "auto", 3), (5000, 6, 30011, 20000, "auto", 3),
    (5000, 6, 30011, 30000, "auto", 3), (5000, 6, 30011, 1000, "auto", 1)])
def test_loss_of_an_infinite_coordinate(P, backbone, paths, pairs, window, renumber, schedule):  # noqa: F811
    import torch
    sg = synth.generate(backbone, 0.2, paths, 31)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg, renumber=renumber)
    rng = np.random.default_rng(pairs)
    c = (O.init_coords(og) + rng.normal(scale=5.0, size=4 * sg.n_nodes)).astype(np.float32)
    kw = dict(seed=11, zipf_window=window, schedule=schedule)
    oracle = O.stress_loss_grad_windowed if schedule == 3 else O.stress_loss_grad
    loss0, nv0, grad0 = oracle(og, c, pairs, seed=11, step=0, window=window)
    touched = (np.abs(grad0).reshape(2, -1) > 0).any(axis=0)
    assert touched.any()
    for k in (int(np.argmax(np.abs(grad0[: touched.size]))), *np.nonzero(~touched)[0][:1]):
        far = c.copy()
        far[k] = np.inf
        t = torch.from_numpy(far).cuda()
        loss, nv = P.stress_forward(g, t, pairs, 0, **kw)
        grad = torch.zeros_like(t)
        P.stress_backward(g, t, pairs, 0, torch.ones(1, device="cuda"), nv, grad, **kw)
        _, _, ref = oracle(og, far, pairs, seed=11, step=0, window=window)
        assert int(nv.item()) == nv0
        if touched[k]:
            assert loss.item() == float("inf")
        else:
            assert abs(loss.item() - loss0) <= 1e-5 * abs(loss0)
        got, nan = grad.cpu().numpy().astype(np.float64), np.isnan(ref)
        assert np.array_equal(np.isnan(got), nan) and nan[k] == touched[k]
        err = np.abs(got[~nan] - ref[~nan])
        assert np.all(err <= 1e-4 * np.abs(ref[~nan]) + 1e-6 * np.abs(ref[~nan]).max())
