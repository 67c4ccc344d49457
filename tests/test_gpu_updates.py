"""GPU checks of the layout kernels' own updates in the automatic grids of many waves."""
import numpy as np
import pytest

import batch_check as B
import oracle as O
import synth
from test_gpu_parity import P  # noqa: F401 (the package fixture)

pytestmark = pytest.mark.gpu


# an early and a mixed iteration (the next item drawn ahead beside uniform partners, the far end read first) and a
# cooling one, at sizes whose XCDs share unequally and equally.  With one term for sixteen steps many terms share no
# coordinate slot with any other of the iteration: whatever the order, those have one result, bounded as in
# batch_check against the FP64 update, and a slot that no term names keeps its value
@pytest.mark.parametrize("backbone,paths", [(30000, 12), (75000, 12)])
@pytest.mark.parametrize("it", [0, 7, 20])
def test_updates_of_the_waves_that_draw_ahead(P, backbone, paths, it):  # noqa: F811
    import torch
    sg = synth.generate(backbone, 0.2, paths, 19)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg)
    assert g.n_nodes >= 32768
    kw = dict(terms_per_step=1, step_reduction=16)
    T = -(-og.S // 16)
    i, j, f = (t.cpu().numpy() for t in P.sample_terms(g, it, 0, T, **kw))
    i, j = i.astype(np.uint64), j.astype(np.uint64)
    # the windowed slots of such an iteration are the oracle's
    oi, oj, of = O.sample_terms_windowed(og, it, 0, T, offsets=O.window_offsets(og, it, threads=8, step_reduction=16,
                                                                               terms_per_step=1))
    assert np.array_equal(i, oi) and np.array_equal(j, oj) and np.array_equal(f, of)
    a, b = B.slots(og, i, j, f)
    named = (f & 8) == 0
    uses = np.bincount(np.concatenate([a[named], b[named]]), minlength=2 * og.n_nodes)
    keep = np.nonzero(named & (uses[a] == 1) & (uses[b] == 1))[0]  # a = b counts twice
    assert keep.size > 5000
    eta = float(O.schedule(30, float(og.d_max) ** 2, 0.01).astype(np.float32)[it])
    start = B.start_coords(og, it)
    c = torch.from_numpy(start).cuda()
    P.layout(g, c, first_iter=it, last_iter=it + 1, **kw)
    got = c.cpu().numpy().astype(np.float64)
    ref, applied = B.fp64_result(og, eta, i[keep], j[keep], f[keep], start)
    assert applied == keep.size
    worst, _ = B.check(og, og.pos, i[keep], j[keep], f[keep], eta, start, got, ref)
    assert worst <= 1.0, f"worst error / bound = {worst:.3f}"
    idle = np.tile(uses == 0, 2)
    assert idle.sum() > 1000 and np.array_equal(got[idle], start[idle].astype(np.float64))
