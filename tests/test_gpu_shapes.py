"""GPU checks of launch shapes and kernel variants at the sizes where they change, against the CPU oracle."""
import numpy as np
import pytest

import oracle as O
import synth
from test_gpu_parity import P, _compare_windowed  # noqa: F401 (P: the package fixture)

pytestmark = pytest.mark.gpu


# 33K, 45K and 65.5K nodes: the automatic grids whose XCDs have equal (16 and 32 waves at n_nodes / 2048) and
# unequal (21) numbers of blocks; every slot of an early, a mixed and a cooling iteration is processed once
@pytest.mark.parametrize("backbone,paths", [(28000, 4), (38000, 4), (55500, 4)])
def test_windowed_sampling_in_the_automatic_grids(P, backbone, paths):  # noqa: F811
    sg = synth.generate(backbone, 0.2, paths, 17)
    og, g = O.Graph.from_synth(sg), P.Graph.from_synth(sg)
    assert g.n_nodes >= 32768
    for it in (0, 9, 20):
        _compare_windowed(P, g, og, it, 0, 10 * og.S)
