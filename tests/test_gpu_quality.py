"""GPU checks of layout quality at the automatic wave caps: more waves lose more concurrent updates, so the path stress
over all step pairs (Eq. 1, no sampling error) is compared with that of n_nodes / 2048 waves, about n_nodes / 32 terms
in flight, over several seeds.  The bar is 3% on the means, plus three standard errors of the two means for the spread
between runs."""
import numpy as np
import pytest

import synth
from test_gpu_parity import P  # noqa: F401 (the package fixture)

pytestmark = pytest.mark.gpu

SEEDS = 6


def _check(label, many, few):
    many, few = np.array(many), np.array(few)
    error = np.sqrt((many.var(ddof=1) + few.var(ddof=1)) / len(many))
    print(f"[quality] {label}: {many.mean() / few.mean():.4f} +- {error / few.mean():.4f}", flush=True)
    assert many.mean() <= 1.03 * few.mean() + 3 * error, label


# the first sizes with many waves in the plain order and in the windowed one, one below it, sizes whose XCDs share
# unequally (below 65,536 nodes) and equally, one path (few updates a node), and where n_nodes / 64 waves are the
# most.  Two to six paths are left out: which XCD ends last puts their layouts in one of several states, a few percent
# apart
@pytest.mark.parametrize("schedule,nodes,paths", [(1, 20000, 8), (1, 85000, 12), (1, 84000, 1), (3, 34500, 24),
                                                  (3, 38500, 24), (3, 49000, 24), (3, 52000, 1), (3, 125000, 12),
                                                  (3, 84000, 1), (3, 200000, 8), (3, 330000, 1)])
def test_automatic_wave_caps_keep_the_stress(P, schedule, nodes, paths):  # noqa: F811
    sg = synth.generate(int(nodes / (2.0 - 0.95 ** paths)), 0.2, paths, 13)
    g = P.Graph.from_synth(sg)
    stress = {}
    for waves in (0, g.n_nodes // 2048):
        stress[waves] = []
        for seed in range(SEEDS):
            c = P.init_coords(g, g.new_coords())
            P.layout(g, c, seed=seed, schedule=schedule, max_inflight_waves=waves)
            stress[waves].append(P.path_stress_exact(g, c)[0])
    _check(f"schedule {schedule}, {g.n_nodes} nodes, {paths} paths", *stress.values())


@pytest.mark.parametrize("small", [False, True])
def test_batched_wave_caps_keep_the_stress(P, small):  # noqa: F811
    # several graphs at a time, at the caps of batches without and with a graph of fewer than 32,768 nodes, against
    # each graph by itself at n_nodes / 2048 waves
    shapes = [(34000, 24), (60000, 12), (84000, 1), (120000, 8)]
    graphs = [P.Graph.from_synth(synth.generate(int(n / (2.0 - 0.95 ** p)), 0.2, p, 13)) for n, p in shapes]
    batch = graphs + [P.Graph.from_synth(synth.generate(700, 0.2, 4, 13))] * small
    many, few = [[] for _ in shapes], [[] for _ in shapes]
    for seed in range(SEEDS):
        coords = [P.init_coords(g, g.new_coords()) for g in batch]
        P.layout_batched(batch, coords, seed=seed)
        for k, g in enumerate(graphs):
            c = P.init_coords(g, g.new_coords())
            P.layout(g, c, seed=seed, graph_id=k, max_inflight_waves=g.n_nodes // 2048)
            many[k].append(P.path_stress_exact(g, coords[k])[0])
            few[k].append(P.path_stress_exact(g, c)[0])
    for k, shape in enumerate(shapes):
        _check(f"batch, {shape[0]} nodes, {shape[1]} paths", many[k], few[k])
