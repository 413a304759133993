"""GPU: batches of small geometries, many steps per launch with the state on
chip, against single steps (an explicit step configuration) of the same batch.

Both update a node by the same arithmetic, so populations and traces are equal
bit for bit.  Sizes: runs of every length (2 .. 16 planes, the last runs one
shorter), 768 threads exactly, one thread more or one probe more than the
kernel takes (single steps then), every wall rule on every axis, driven nodes
with one and with two of them in one thread's run.
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu

B, P, F, X = "bounceback", "periodic", "free", "fixed"


def pipe(n, lo, hi):
    return dict(kind="cylinder", dim=3, n=n, qmin=(1.0, 0.0, 0.0), qmax=(25.0, 2.0 * np.pi, 100.0), bc_lo=lo,
                bc_hi=hi, h_ref=1.0, damp=0.65, params=(), c=0.02)


CASES = [((20, 5, 100), (B, P, B), (B, P, X), 8), ((20, 5, 113), (B, P, B), (F, P, F), 8),
         ((7, 9, 31), (X, B, F), (F, X, X), 8), ((33, 4, 41), (F, F, X), (X, B, B), 32),
         ((5, 1, 17), (B, P, P), (B, P, P), 33), ((16, 24, 3), (B, P, F), (X, P, B), 3),
         ((16, 24, 4), (B, P, F), (X, P, B), 3), ((6, 4, 2), (B, B, B), (B, F, F), 4),
         ((12, 2, 300), (B, P, P), (X, P, P), 4), ((24, 32, 9), (B, P, P), (F, P, P), 2),
         ((8, 3, 512), (B, P, B), (B, P, F), 2), ((8, 3, 513), (B, P, B), (B, P, F), 2)]


@pytest.mark.parametrize("n,lo,hi,probes", CASES, ids=str)
@pytest.mark.parametrize("sources", ["none", "ends", "run"])
def test_many_steps_equal_single_steps(n, lo, hi, probes, sources):
    print("resident", n, lo, hi, sources, flush=True)
    N, plane = n[0] * n[1] * n[2], n[0] * n[1]
    rng = np.random.default_rng(N + probes)
    other = (n[0], n[1], max(2, n[2] - 1))  # a shorter geometry in the same batch
    geoms = [pipe(n, lo, hi), pipe(other, lo, hi), pipe(n, lo, hi)]
    sizes = [N, plane * other[2], N]
    P0 = [rng.uniform(-1, 1, s) for s in sizes]
    where = [rng.integers(0, sizes[0], size=probes), rng.integers(0, sizes[1], size=1), np.array([0, 0, N - 1])]
    nodes = {"none": [], "ends": [1, 3, N - 2], "run": [1, 1 + plane]}[sources]  # (1 + plane: the same run)
    got = []
    for single in (False, True):
        b = lbw.Batch(geoms, P0, where, t_max=140)
        if nodes:
            k = len(nodes)
            b.set_sources(nodes + nodes, [0] * k + [2] * k, 0.7, [0.05] * k + [0.11] * k,
                          flux_axis=[-1] * k + [2] * k)
        if single:
            b.set_step_config(16, 8)
        for steps in (1, 2, 31, 32, 33, 64):  # the last beyond t_max
            b.step(steps)
        got.append(([b.populations(h).clone() for h in range(3)], b.probe().copy(), b.t))
    assert got[0][2] == got[1][2] == 163
    for a, c in zip(got[0][0], got[1][0]):
        assert torch.equal(a, c)
    assert np.array_equal(got[0][1], got[1][1])
    assert np.abs(got[0][1]).max() > 1e-3
