"""GPU: several steps per launch of a 2-D grid against single steps.

Sim.step(n) with n > 1 takes tiles that stay on chip for several steps,
step(1) the one-step kernel; both run the same per-node routine, so
populations and probe traces must agree bit for bit, at the sizes where the
tiling changes: an axis held whole (walled, 64 nodes and fewer), a periodic
axis 1 closing into a ring of strips (full and partial last strip, one row
over), one node more than a tile, several tiles along each axis, and more
probes than one tile records (which falls back to single steps).
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu


def plane(n0, n1, lo, hi):
    return dict(kind="box", dim=2, n=(n0, n1), qmin=(0.0, 0.0), qmax=(float(n0), float(n1)), bc_lo=lo, bc_hi=hi,
                h_ref=1.0, c=0.5, damp=0.8, params=())


def disk(n0, n1):
    return dict(kind="polar2d", dim=2, n=(n0, n1), qmin=(0.05, 0.0), qmax=(1.0, 2 * np.pi),
                bc_lo=("bounceback", "periodic"), bc_hi=("fixed", "periodic"), h_ref=0.95 / n0, c=0.1, damp=1.0,
                params=())


W2 = ("fixed", "bounceback"), ("free", "fixed")
P0_ = ("periodic", "free"), ("periodic", "bounceback")
PP = ("periodic", "periodic"), ("periodic", "periodic")
CASES = [disk(64, 64), disk(63, 65), disk(16, 33), disk(12, 2), disk(65, 64), disk(40, 1), disk(100, 150),
         plane(1, 1, *W2), plane(1, 9, *W2), plane(64, 128, *W2), plane(64, 129, *W2), plane(65, 17, *W2),
         plane(130, 70, *W2), plane(301, 203, *W2), plane(5, 3, *P0_), plane(64, 40, *P0_), plane(150, 90, *PP),
         plane(1, 300, *PP)]


@pytest.mark.parametrize("geom", CASES, ids=lambda g: "%s-%dx%d-%s" % (g["kind"], *g["n"], g["bc_lo"][0][:2]))
@pytest.mark.parametrize("probes", [3, 200])
def test_blocks_of_steps_equal_single_steps(geom, probes):
    n = geom["n"][0] * geom["n"][1]
    rng = np.random.default_rng(n + probes)
    P0 = rng.uniform(-1, 1, n)
    pr = rng.integers(0, n, probes)
    steps = 37
    print("tile2d", geom["n"], probes, flush=True)
    g = lbw.Geometry(geom)
    a = lbw.Simulation(g, P0, pr, t_max=steps - 2)
    b = lbw.Simulation(g, P0, pr, t_max=steps - 2)
    for part in (2, 19, 16):
        a.step(part)
    for _ in range(steps):
        b.step(1)
    assert a.t == b.t == steps
    assert torch.equal(a.populations(), b.populations())
    assert torch.equal(a.trace, b.trace)
    # and the scheme itself against the FP64 oracle: 1e-5 of the initial field
    # (37 steps of FP32 rounding; a single node between lossy walls decays, so
    # the final field is no scale)
    o = oracle.Oracle(geom)
    f0 = o.init(P0)
    f, tr = o.run(f0, steps, pr)
    err = np.linalg.norm(a.populations().double().cpu().numpy() - f) / np.linalg.norm(o.init(P0))
    assert err <= 1e-5, err
