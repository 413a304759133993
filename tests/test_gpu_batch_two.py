"""GPU: batches that the tuner may advance two steps per launch, against single
steps (an explicit step configuration) of the same batch.

Both update a node by the same arithmetic, so populations and traces are equal
bit for bit, whichever launches the tuner keeps.  The cross-sections are too
large for the many-step kernel and small enough that two steps per launch win
(5 against 9 us per step for the first): the shortest and longest rows the tiles
take, one row tile and several, a last tile of fewer rows, one plane, walls of
every kind, and a batch that mixes walled and periodic axes.
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu

B, P, F, X = "bounceback", "periodic", "free", "fixed"


def geom(n, lo, hi):
    return dict(kind="cylinder", dim=3, n=n, qmin=(1.0, 0.0, 0.0), qmax=(1.0 + n[0], 2.0 * np.pi, 1.0 * n[2]), bc_lo=lo,
                bc_hi=hi, h_ref=1.0, damp=0.65, params=(), c=0.02)


CASES = {"horn": [((20, 52, 40), (B, P, B), (B, P, X))], "short_rows": [((4, 250, 37), (B, P, B), (F, P, F))],
         "long_rows": [((96, 14, 41), (F, P, X), (X, P, B))], "walls": [((25, 61, 50), (F, F, P), (B, X, P))],
         "closed": [((33, 30, 17), (X, B, F), (F, X, X))], "flat": [((64, 13, 1), (B, P, B), (B, P, F))],
         "mixed": [((20, 52, 40), (B, P, B), (B, P, X)), ((25, 61, 50), (X, F, F), (B, X, B)),
                   ((17, 100, 5), (B, P, F), (X, P, B))],
         "three_columns": [((3, 300, 20), (B, P, B), (B, P, B))]}  # (rows too short: single steps)


@pytest.mark.parametrize("name", sorted(CASES))
def test_tuned_batch_equals_single_steps(name):
    print("two-step batch", name, flush=True)
    geoms = [geom(*c) for c in CASES[name]]
    N = [int(np.prod(g["n"])) for g in geoms]
    rng = np.random.default_rng(sum(N))
    P0 = [rng.uniform(-1, 1, k) for k in N]
    probes = [rng.integers(0, k, size=5) for k in N]
    got = []
    for tuned in (True, False):
        b = lbw.Batch(geoms, P0, probes, t_max=100)
        if tuned:
            b.autotune(reps=2)
        else:
            b.set_step_config(16, 8)
        for k in (1, 2, 32, 33, 7):  # (33: a graph block and a step more)
            b.step(k)
        b.set_graph_block(5)  # an odd block: two launches of two steps and one single
        b.step(31)
        got.append(([b.populations(h).clone() for h in range(len(geoms))], b.probe().copy()))
    for a, c in zip(*[f for f, _ in got]):
        assert torch.equal(a, c)
    assert np.array_equal(got[0][1], got[1][1])
