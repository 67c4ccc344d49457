"""GPU checks of launch shapes and kernel variants at the sizes where they change, against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
import synth
from test_gpu_parity import P, _compare_windowed  # noqa: F401 (P: the package fixture)

pytestmark = pytest.mark.gpu


# 33K, 44K and 65K nodes: the automatic grids whose XCDs have equal (16 waves at n_nodes / 2048) and
# unequal (21 and 31) numbers of blocks; every slot of an early, a mixed and a cooling iteration is processed once
@pytest.mark.parametrize("backbone,paths", [(28300, 4), (38000, 4), (55500, 4)])
def test_windowed_sampling_in_the_automatic_grids(P, backbone, paths):  # noqa: F811
    sg = synth.generate(backbone, 0.2, paths, 17)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg)
    assert g.n_nodes >= 32768
    for it in (0, 9, 20):
        _compare_windowed(P, g, og, it, 0, 10 * og.S)


# few steps with many pairs each (split between threads, the last chunk of a step shorter), one pair a step, and more
# steps than threads; the deviations about the mean to the sums' bar (FP64 terms in another order)
@pytest.mark.parametrize("backbone,paths,m", [(2, 1, 1), (2, 1, 977), (40, 3, 1000), (700, 3, 257), (3000, 4, 63),
                                              (250000, 3, 2)])
@pytest.mark.parametrize("pairs", ["uniform", "power_law", "uniform_windowed"])
def test_sps_in_one_pass_at_its_split_sizes(P, backbone, paths, m, pairs):  # noqa: F811
    import torch
    sg = synth.generate(backbone, 0.2, paths, 5)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg)
    rng = np.random.default_rng(backbone)
    c = (O.init_coords(og) + rng.normal(scale=4.0, size=4 * sg.n_nodes)).astype(np.float32)
    a, b = P.path_stress(g, torch.from_numpy(c).cuda(), m, 3, pairs=pairs), O.sampled_path_stress(og, c, m, 3,
                                                                                                pairs=pairs)
    assert (a["n_valid"], a["n_skipped"]) == (b["n_valid"], b["n_skipped"])
    for k in ("sum", "sumsq_dev", "mean", "stddev"):
        assert abs(a[k] - b[k]) <= 1e-9 * abs(b[k]), (k, a[k], b[k])


@pytest.mark.parametrize("pairs", ["uniform", "power_law", "uniform_windowed"])
def test_sps_deviations_cancel_exactly(P, pairs):  # noqa: F811
    # a straight path laid out at three times its length: every stress is exactly 4, so its sum is exact, its
    # deviations from the mean are 0, and so are those of two equal layouts from their ratio 1
    import torch
    sg = synth.linear_path(5000)
    g = P.Graph.from_synth(sg)
    x = np.cumsum(np.concatenate([[0], sg.node_len.astype(np.int64)]))
    c = np.zeros((2, sg.n_nodes, 2), np.float32)
    c[0, :, 0], c[0, :, 1] = 3 * x[:-1], 3 * x[1:]
    t = torch.from_numpy(c.reshape(-1)).cuda()
    r = P.path_stress(g, t, 20, 3, pairs=pairs)
    assert r["sum"] == 4.0 * r["n_valid"] and r["sumsq_dev"] == 0.0 and r["ci_lo"] == r["ci_hi"] == 4.0
    noisy = t + 5 * torch.randn(t.numel(), generator=torch.Generator().manual_seed(1)).cuda()
    q = P.path_stress_compare(g, noisy, noisy.clone(), 20, pairs=pairs)
    assert q["ratio"] == 1.0 and q["sd_diff"] == 0.0 and q["sd_a"] == q["sd_b"] > 0
    inf = t.clone()
    inf[7] = float("inf")
    r = P.path_stress(g, inf, 20, 3, pairs=pairs)  # as the plain FP64 sums: inf, and no deviation from it
    assert r["sum"] == r["mean"] == float("inf") and np.isnan(r["stddev"])


# one column, one row tile and its neighbours, a chunk of columns and its neighbours, several row tiles; with
# the long nodes the paths of 256 steps and more pass 2^40 nucleotides (the integer variant)
@pytest.mark.parametrize("steps", [1, 2, 3, 255, 256, 257, 511, 512, 513, 514, 1300])
@pytest.mark.parametrize("length", [9, 4_000_000_000])
def test_exact_path_stress_at_the_edges_of_its_tiles(P, steps, length):  # noqa: F811
    import torch
    rng = np.random.default_rng(steps)
    n = 700
    paths = [steps, 5, 0, steps // 2 + 1]
    off = np.cumsum([0] + paths).astype(np.uint64)
    node_len = rng.integers(max(1, length - 8), length + 1, size=n).astype(np.uint32)
    node = rng.integers(0, n, size=int(off[-1])).astype(np.uint32)
    node |= np.where(rng.random(node.size) < 0.3, np.uint32(synth.REV_BIT), np.uint32(0)).astype(np.uint32)
    sg = synth.SynthGraph(node_len, off, node, {}, "tiles")
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg)
    c = rng.normal(scale=50.0, size=4 * n).astype(np.float32)
    mean, pairs = P.path_stress_exact(g, torch.from_numpy(c).cuda())
    ref = O.path_stress_exact(og, c)
    assert pairs == ref[1]
    assert abs(mean - ref[0]) <= 1e-9 * abs(ref[0])


# the ordered form of one-wave layouts against k_layout_local (which layout_noalloc keeps), bit for bit: a single item,
# a chunk of items and its neighbours, the last size with the coordinates in LDS and the first in memory, many short
# paths, iteration ranges and parameters
@pytest.mark.parametrize("backbone,paths,nodes,kw", [
    (2, 1, 0, {}), (7, 1, 0, {}), (200, 1, 0, {}), (211, 1, 0, {}), (300, 3, 0, {"terms_per_step": 1}),
    (1000, 40, 0, {"n_iters": 6}), (3448, 4, 4095, {"n_iters": 4}),
    (3448, 4, 4096, {"n_iters": 4, "max_inflight_waves": 1}), (3448, 4, 4097, {"n_iters": 4, "max_inflight_waves": 1}),
    (9000, 4, 0, {"n_iters": 4, "max_inflight_waves": 1}), (500, 5, 0, {"first_iter": 13, "last_iter": 17}),
    (500, 5, 0, {"zipf_window": 7, "zipf_theta": 0.5, "eta_min": 1e-9, "eta_max": 1e30, "graph_id": 3})])
def test_ordered_layout_equals_the_window_kernel(P, backbone, paths, nodes, kw):  # noqa: F811
    import torch
    sg = synth.generate(backbone, 0.2, paths, 23)
    if nodes:  # nodes that no path visits
        sg.node_len = np.concatenate([sg.node_len, np.ones(nodes - sg.n_nodes, np.uint32)])
    g = P.Graph.from_synth(sg)
    a, b = g.new_coords(), g.new_coords()
    for f, c in ((P.layout, a), (P.layout_noalloc, b)):
        P.init_coords(g, c)
        f(g, c, **kw)
    torch.cuda.synchronize()
    assert torch.equal(a, b)


@pytest.mark.parametrize("span", [40, 60, 70])
def test_ordered_layout_with_coincident_and_distant_points(P, span):  # noqa: F811
    # the ranges of the update's short sequences: equal points, distances below 2^-48 and above 2^48; with the widest
    # span squares overflow and both forms end with the same infinities and NaN
    import torch
    sg = synth.generate(300, 0.2, 4, 3)
    g = P.Graph.from_synth(sg)
    rng = np.random.default_rng(8)
    c = (rng.normal(size=4 * g.n_nodes) * 2.0 ** rng.integers(-span, span, size=4 * g.n_nodes)).astype(np.float32)
    c[rng.random(c.size) < 0.3] = 0.0
    a, b = torch.from_numpy(c).cuda(), torch.from_numpy(c).cuda()
    P.layout(g, a, n_iters=8)
    P.layout_noalloc(g, b, n_iters=8)
    torch.cuda.synchronize()
    assert bool(((a == b) | (a.isnan() & b.isnan())).all())
    assert span > 60 or bool(torch.isfinite(a).all())


# few pairs (tiles not staged, one unit each), a tile cut into many units, every tile staged, zipf windows whose tables
# leave room for a shorter range, for none staged and for the image in float alone, renumbered ids
@pytest.mark.parametrize("backbone,paths,pairs,window,renumber", [
    (300, 3, 40, 1000, "auto"), (900, 4, 60000, 1000, "auto"), (9000, 5, 200, 1000, "auto"),
    (9000, 5, 300000, 1000, "always"), (5000, 6, 100001, 4000, "auto"), (9000, 5, 100003, 9000, "auto"),
    (5000, 6, 30011, 20000, "auto")])
def test_loss_tiles_at_their_split_sizes(P, backbone, paths, pairs, window, renumber):  # noqa: F811
    import torch
    sg = synth.generate(backbone, 0.2, paths, 31)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg, renumber=renumber)
    rng = np.random.default_rng(pairs)
    c = (O.init_coords(og) + rng.normal(scale=5.0, size=4 * sg.n_nodes)).astype(np.float32)
    t = torch.from_numpy(c).cuda()
    kw = dict(seed=11, zipf_window=window)
    for step in (0, 3):
        ol, ov, ograd = O.stress_loss_grad_windowed(og, c, pairs, seed=11, step=step, window=window)
        loss, nv = P.stress_forward(g, t, pairs, step, **kw)
        grad = torch.zeros_like(t)
        P.stress_backward(g, t, pairs, step, torch.ones(1, device="cuda"), nv, grad, **kw)
        assert int(nv.item()) == ov
        assert abs(loss.item() - ol) <= 1e-5 * abs(ol)
        err = np.abs(grad.cpu().numpy().astype(np.float64) - ograd)
        assert np.all(err <= 1e-4 * np.abs(ograd) + 1e-6 * np.abs(ograd).max())
    t[: 2 * sg.n_nodes] = float("inf")  # as the plain FP64 sum
    assert np.isnan(P.stress_forward(g, t, pairs, 0, **kw)[0].item())
    t[: 2 * sg.n_nodes] = 0.0
    t[0] = float("inf")
    assert P.stress_forward(g, t, pairs, 0, **kw)[0].item() in (float("inf"), 0.0) or pairs < 1000


# an odd number of nodes (the copy's halves meet inside a node) and renumbered ids; FP64 terms summed in
# another order: 1e-9
@pytest.mark.parametrize("pairs", ["uniform", "power_law", "uniform_windowed"])
@pytest.mark.parametrize("backbone,renumber", [(301, "auto"), (1203, "always")])
def test_two_layouts_side_by_side(P, backbone, renumber, pairs):  # noqa: F811
    import torch
    sg = synth.generate(backbone, 0.2, 5, 23)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg, renumber=renumber)
    rng = np.random.default_rng(backbone)
    ca = (O.init_coords(og) + rng.normal(scale=3.0, size=4 * sg.n_nodes)).astype(np.float32)
    cb = (O.init_coords(og) + rng.normal(scale=9.0, size=4 * sg.n_nodes)).astype(np.float32)
    ref = O.sps_compare(og, ca, cb, m=7, seed=5, pairs=pairs)
    ta, tb = torch.from_numpy(ca).cuda(), torch.from_numpy(cb).cuda()
    r = P.path_stress_compare(g, ta, tb, 7, 5, pairs=pairs)
    assert r["n_valid"] == ref["n_valid"] and r["n_skipped"] == ref["n_skipped"]
    for k in ("sum_a", "sum_b", "ratio", "sd_a", "sd_b", "sd_diff"):
        assert abs(r[k] - ref[k]) <= 1e-9 * abs(ref[k]), k
    one = P.path_stress(g, ta, 7, seed=5, pairs=pairs)  # the copy of one layout afterwards
    assert one["n_valid"] == r["n_valid"] and abs(one["mean"] - ref["mean_a"]) <= 1e-9 * abs(ref["mean_a"])


# coordinates read in place at an odd float offset, and calls one after another that share the work queue (several
# tiles a block, then few); the same pairs of the same floats: equal up to the order of the sums
@pytest.mark.parametrize("backbone,pairs", [(300011, 300000), (9000, 200)])
def test_loss_reads_coordinates_in_place(P, backbone, pairs):  # noqa: F811
    import torch
    sg = synth.generate(backbone, 0.2, 4, 29)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg)
    rng = np.random.default_rng(pairs)
    c = (O.init_coords(og) + rng.normal(scale=5.0, size=4 * sg.n_nodes)).astype(np.float32)
    t = torch.empty(c.size + 1, device="cuda")[1:]
    t.copy_(torch.from_numpy(c))
    one = torch.ones(1, device="cuda")
    for step in (0, 0, 1):
        ol, ov, ograd = O.stress_loss_grad_windowed(og, c, pairs, seed=11, step=step, window=1000)
        loss, nv = P.stress_forward(g, t, pairs, step, seed=11)
        assert int(nv.item()) == ov and abs(loss.item() - ol) <= 1e-5 * abs(ol)
        for _ in range(2):
            grad = torch.zeros_like(t)
            P.stress_backward(g, t, pairs, step, one, nv, grad, seed=11)
            err = np.abs(grad.cpu().numpy().astype(np.float64) - ograd)
            assert np.all(err <= 1e-4 * np.abs(ograd) + 1e-6 * np.abs(ograd).max())
