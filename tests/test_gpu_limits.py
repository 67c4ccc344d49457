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
