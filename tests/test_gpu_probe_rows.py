"""GPU: trace rows of more probes than a workgroup has threads, up to and beyond
the last row, by single steps of 2-D, 3-D and per-node geometries and by two
steps per launch: the rows of a longer trace, and nothing after them.
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu

RING = dict(bc_lo=("bounceback", "periodic", "bounceback"), bc_hi=("bounceback", "periodic", "fixed"))


def geometry(kind):
    if kind == "disk":
        return dict(kind="polar2d", dim=2, n=(30, 41), qmin=(0.05, 0.0), qmax=(1.0, 2 * np.pi), bc_lo=RING["bc_lo"][:2],
                    bc_hi=RING["bc_hi"][:2], h_ref=0.95 / 30, c=0.1, damp=1.0, params=())
    g = dict(kind="cylinder", dim=3, n=(19, 10, 33), qmin=(1.0, 0.0, 0.0), qmax=(20.0, 2 * np.pi, 33.0), h_ref=1.0,
             damp=0.7, params=(), c=0.05, **RING)
    if kind == "metric":  # the identity metric, per node
        N = 19 * 10 * 33
        g.update(kind="general", qmin=(0.0,) * 3, qmax=(19.0, 10.0, 33.0))
        g["coeffs"] = np.concatenate([np.ones((4, N)), np.zeros((6, N))])
    return g


@pytest.mark.parametrize("kind,two", [("disk", False), ("cylinder", False), ("cylinder", True), ("metric", False)])
@pytest.mark.parametrize("probes", [256, 257, 1500])
def test_rows_up_to_the_last(kind, two, probes):
    print("probe rows", kind, two, probes, flush=True)
    geom = geometry(kind)
    N = int(np.prod(geom["n"]))
    rng = np.random.default_rng(probes)
    P0 = rng.uniform(-1, 1, N)
    at = rng.integers(0, N, probes) if not two else np.sort(rng.choice(N, probes, replace=False))
    g = lbw.Geometry(geom)
    if kind == "cylinder":
        g.set_step_config(16, 16, 4)
    if two:
        g.set_step2_config(96, 6, 1)
    a, b = (lbw.Simulation(g, P0, at, t_max=t) for t in (5, 30))
    for s in (a, b):
        for _ in range(4):
            s.step(1)
        s.step(2)
        s.step(2)
        for _ in range(4):
            s.step(1)
    torch.cuda.synchronize()
    assert torch.equal(a.trace, b.trace[:5])
    assert torch.equal(a.populations(), b.populations())
    assert (b.trace[12:] == 0.0).all() and b.trace[11].abs().max() > 0.0
    f = lbw.Simulation(g, P0, at, t_max=1)
    f.step(1)
    assert torch.equal(f.trace[0], b.trace[0])
