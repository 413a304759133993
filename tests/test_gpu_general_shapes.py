"""GPU: geometries given by their metric take a launch shape by a rule on their
grid: the shapes on both sides of its lines, and the results against those of
64 x 8 (or 32 x 8) tiles of 16 planes, which every shape gives bit for bit (the
same arithmetic per node).
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw
import workloads as W

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shape", [((20, 20, 20), (32, 8, 1)), ((32, 60, 128), (32, 8, 2)), ((33, 60, 40), (64, 4, 1)),
                                     ((40, 80, 100), (64, 4, 2)), ((128, 96, 128), (64, 4, 2)),
                                     ((128, 97, 128), (64, 8, 16)), ((5, 3, 2), (32, 8, 1))], ids=str)
def test_default_shape(n, shape):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    print("general shape", n, cus, flush=True)
    geom = W.general_duct(n=n)
    geom = dict(geom, coeffs=W.general_coefficients(geom))
    N = n[0] * n[1] * n[2]
    P0 = np.random.default_rng(1).uniform(-1, 1, N)
    got = []
    for explicit in (False, True):
        g = lbw.Geometry(geom)
        if explicit:
            g.set_step_config(64 if n[0] > 32 else 32, 8, 16)
        elif cus == 256:
            assert g.step_config()[:3] == shape
        sim = lbw.Simulation(g, P0, [0, N // 2, N - 1], t_max=10)
        sim.step(10)
        got.append((sim.populations().clone(), sim.probe()))
    assert torch.equal(got[0][0], got[1][0])
    assert np.array_equal(got[0][1], got[1][1])
