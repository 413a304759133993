"""GPU: the launches of a batch, asked for and reported, against single steps.

Two steps per launch and up to 32 of them update a node by the arithmetic of
single steps, so populations and traces are equal bit for bit.  Every case
asserts which launches ran: run lengths of 2 to 16 planes per thread with driven
nodes at several planes of a run, in two runs and up to the most that fit, of
both source kinds; two-step tiles of every kind, more segments than workgroups,
and the most probes that a segment records; and what falls back.
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu

B, P, F, X = "bounceback", "periodic", "free", "fixed"


def pipe(n, lo, hi):
    return dict(kind="cylinder", dim=3, n=n, qmin=(1.0, 0.0, 0.0), qmax=(1.0 + n[0], 2.0 * np.pi, 1.0 * n[2]), bc_lo=lo,
                bc_hi=hi, h_ref=1.0, damp=0.65, params=(), c=0.02)


def same(geoms, steps_per_launch, planes, probes, steps, sources=None, t_max=200):
    N = [int(np.prod(g["n"])) for g in geoms]
    rng = np.random.default_rng(sum(N))
    P0 = [rng.uniform(-1, 1, k) for k in N]
    got = []
    for want in (steps_per_launch, 1):
        b = lbw.Batch(geoms, P0, probes, t_max=t_max)
        if sources:
            b.set_sources(**sources)
        b.set_steps_per_launch(want)
        assert b.steps_per_launch() == ((want, planes) if want > 2 else (want, 0))
        for k in steps:
            b.step(k)
        got.append((torch.cat([b.populations(h).reshape(-1) for h in range(len(geoms))]).clone(), b.trace.clone()))
    assert torch.equal(got[0][0], got[1][0])
    assert torch.equal(got[0][1], got[1][1])
    assert got[0][1].abs().max() > 1e-3


# ---- many steps per launch ----

def ends(r):
    """Two driven nodes: the last plane of the first run and, in another
    column, the first of the second."""
    return dict(nodes=[5 + 96 * (r - 1), 7 + 96 * r], geom=[0, 0], amplitude=[0.7, 0.4], omega=[0.05, 0.11],
                flux_axis=[-1, 2])


def most(r):
    """32 driven nodes on two planes inside a run, each in a column of its
    own, of every kind."""
    z = r // 2
    at = [3 * i + 96 * (z + i % 2) for i in range(32)]
    return dict(nodes=at, geom=[2] * 32, amplitude=0.5, omega=0.01 * np.arange(1, 33),
                flux_axis=[-1 + i % 4 for i in range(32)])


@pytest.mark.parametrize("run", range(2, 17))
@pytest.mark.parametrize("walls", [((B, P, B), (B, P, X)), ((X, F, P), (F, B, P))], ids=["periodic_theta", "walled_theta"])
@pytest.mark.parametrize("driven", ["none", "ends", "most"])
def test_runs_of_every_length(run, walls, driven):
    # 96 columns in 8 runs of `run` planes are 768 threads: no shorter run fits
    print("many steps", run, walls, driven, flush=True)
    geoms = [pipe((8, 12, 8 * run), *walls), pipe((8, 12, 8 * run - 3), *walls), pipe((8, 12, 8 * run), *walls)]
    probes = [np.arange(0, 96 * 8 * run, 24 * run + 1), [11], [5 + 96 * (run - 1), 7 + 96 * run]]
    sources = {"none": None, "ends": ends(run), "most": most(run)}[driven]
    same(geoms, 32, run, probes, (1, 2, 31, 32, 33, 64, 9), sources)


@pytest.mark.parametrize("n,planes", [((24, 32, 9), 9), ((8, 8, 1), 2), ((1, 1, 2), 2), ((12, 2, 190), 6),
                                      ((60, 2, 40), 7)])
def test_shapes_that_fit(n, planes):
    print("many steps", n, flush=True)
    same([pipe(n, (B, P, F), (X, P, B))] * 2, 32, planes, [np.arange(32) % np.prod(n), [0]], (3, 32, 40))


def refused(geoms, probes, sources=None, steps=32):
    N = [int(np.prod(g["n"])) for g in geoms]
    b = lbw.Batch(geoms, [np.ones(k) for k in N], probes, t_max=8)
    if sources:
        b.set_sources(**sources)
        assert b.steps_per_launch()[0] == 1
    before = b.steps_per_launch()
    with pytest.raises(lbw.LbwError):
        b.set_steps_per_launch(steps)
    assert b.steps_per_launch() == before
    b.step(5)
    assert b.t == 5


def test_what_many_steps_refuse():
    walls = (B, P, B), (B, P, X)
    refused([pipe((8, 3, 512), *walls)], [[0]])                                     # the coefficient table
    refused([pipe((20, 5, 113), *walls)], [[0]])                                    # 769 threads and more
    refused([pipe((8, 8, 8), *walls)], [np.arange(33)])                             # probes
    refused([pipe((20, 5, 100), *walls), pipe((8, 8, 16), *walls)], [[0], [0]])     # no common run
    one = dict(amplitude=1.0, omega=0.1)
    long = [pipe((8, 12, 64), *walls)]
    refused(long, [[0]], dict(nodes=np.arange(33), geom=[0] * 33, **one))           # driven nodes
    refused(long, [[0]], dict(nodes=[5, 5 + 96], geom=[0] * 2, **one))              # two in a thread's run
    refused(long, [[0]], dict(nodes=[5, 6 + 96 * 8], geom=[0] * 2, **one))          # over many planes


# ---- two steps per launch ----

TWO = {"horn": [((20, 52, 40), (B, P, B), (B, P, X))], "short_rows": [((4, 250, 37), (B, P, B), (F, P, F))],
       "long_rows": [((96, 14, 41), (F, P, X), (X, P, B))], "walls": [((25, 61, 50), (F, F, P), (B, X, P))],
       "closed": [((33, 30, 17), (X, B, F), (F, X, X))], "flat": [((64, 13, 1), (B, P, B), (B, P, F))],
       "mixed": [((20, 52, 40), (B, P, B), (B, P, X)), ((25, 61, 50), (X, F, F), (B, X, B)),
                 ((17, 100, 5), (B, P, F), (X, P, B))],
       "many_segments": [((16, 20 + h % 7, 1 + h % 3), (B, P, B), (X, P, F)) for h in range(700)]}


@pytest.mark.parametrize("name", sorted(TWO))
def test_two_steps_per_launch(name):
    print("two steps", name, flush=True)
    geoms = [pipe(*c) for c in TWO[name]]
    rng = np.random.default_rng(len(name))
    same(geoms, 2, 0, [rng.integers(0, np.prod(g["n"]), size=3) for g in geoms], (1, 2, 3, 4, 32, 33, 7, 64))


def test_two_steps_with_the_most_probes_of_a_segment():
    geoms = [pipe((20, 52, 40), (B, P, B), (B, P, X))]
    near = 20 * 52 * 17 + np.arange(17)  # one row of one plane: one segment
    same(geoms, 2, 0, [near[:16]], (4, 8, 33))
    same(geoms, 2, 0, [np.repeat(near[:1], 16)], (4, 8, 33))
    refused(geoms, [near], steps=2)


def test_what_two_steps_refuse():
    walls = (B, P, B), (B, P, X)
    refused([pipe((3, 300, 20), *walls)], [[0]], steps=2)
    refused([pipe((97, 30, 20), *walls)], [[0]], steps=2)
    refused([pipe((20, 52, 40), (P, P, B), (P, P, X))], [[0]], steps=2)
    refused([pipe((20, 52, 40), *walls)], [[0]], dict(nodes=[3], geom=[0], amplitude=1.0, omega=0.1), steps=2)
    refused([pipe((20, 52, 40), *walls)], [[0]], steps=3)
