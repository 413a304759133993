"""GPU: blocks of few steps of a batch whose geometries fit one workgroup each.

A launch of many steps costs more to start than a single step, so short blocks,
and the rest of long ones, may take single steps; the bits are the same.  And a
single step must not be slower for it: a tuned batch of 16 pipes took 19.7 us a
call where its single-step launches take 8.9; held to half as much again.
"""
import time

import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu


def pipe(n):
    return dict(kind="cylinder", dim=3, n=n, qmin=(1.0, 0.0, 0.0), qmax=(1.0 + n[0], 2.0 * np.pi, 1.0 * n[2]),
                bc_lo=("bounceback", "periodic", "bounceback"), bc_hi=("bounceback", "periodic", "fixed"), h_ref=1.0,
                damp=0.65, params=(), c=0.02)


def batch(n, count, driven):
    N = int(np.prod(n))
    P0 = np.random.default_rng(N).uniform(-1, 1, N)
    b = lbw.Batch([pipe(n)] * count, [P0] * count, [[1, N // 2]] * count, t_max=200)
    if driven:
        ring = n[0] * np.arange(n[1])
        b.set_sources(np.tile(ring, count), np.repeat(np.arange(count), n[1]), 1.0,
                      np.repeat(np.linspace(0.001, 0.03, count), n[1]))
    return b


@pytest.mark.parametrize("n,count", [((8, 12, 96), 3), ((8, 12, 104), 3), ((20, 5, 100), 16), ((16, 24, 31), 2)])
@pytest.mark.parametrize("driven", [False, True])
@pytest.mark.parametrize("tuned", [False, True])
def test_short_blocks_equal_single_steps(n, count, driven, tuned):
    print("short blocks", n, count, driven, tuned, flush=True)
    a, b = batch(n, count, driven), batch(n, count, driven)
    if tuned:
        a.autotune(reps=5)
    else:
        assert a.steps_per_launch()[0] == 32
    b.set_steps_per_launch(1)
    for k in (1, 1, 2, 3, 1, 4, 5, 33, 34, 35, 64, 1):
        a.step(k)
        b.step(k)
    assert torch.equal(a.trace, b.trace)
    for h in range(count):
        assert torch.equal(a.populations(h), b.populations(h))


def test_a_single_step_is_not_slower():
    b = batch((20, 5, 100), 16, True)
    b.autotune(reps=20)

    def best():
        times = []
        for _ in range(8):
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(100):
                b.step(1)
            torch.cuda.synchronize()
            times.append(time.perf_counter() - t0)
        return min(times)

    best()
    tuned = best()
    b.set_steps_per_launch(1)
    best()
    assert tuned <= 1.5 * best()
