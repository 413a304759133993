"""GPU: the spectrum of a group of more columns than one launch takes (65,532
pairs), alone, with one column more than the limit, and among other groups,
against the oracle's numpy FFT.

Tolerance: the powers of up to 131,072 columns are added up, all positive, so
their sum is off by at most 131072 eps = 1.5e-11 of itself besides the
transform's own 4e-13 of a peak; the parabola's place moves by about ten times
that in bins, of at least 16.  Held to 1e-10.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu

BOX = dict(kind="box", dim=3, n=(3, 3, 3), qmin=(0.0,) * 3, qmax=(3.0,) * 3, bc_lo=("bounceback",) * 3,
           bc_hi=("bounceback",) * 3, h_ref=1.0, c=0.5, damp=1.0, params=())


def ring_down(T, cols, rng):
    t = np.arange(T)[:, None]
    x = np.full((T, cols), 0.1)
    for i in range(1, 4):
        x += (rng.uniform(0.3, 1.0, cols) * np.exp(-rng.uniform(0.5, 2.0) / T * t)
              * np.sin(2 * np.pi * t * (6.3 * i / T + 0.001) + rng.uniform(0, 6, cols)))
    return x


def close(got, want):
    assert np.array_equal(np.isnan(got), np.isnan(want)) and not np.isnan(want).all()
    m = ~np.isnan(want)
    assert np.allclose(got[m], want[m], rtol=1e-10, atol=0)


@pytest.mark.parametrize("T,groups", [(64, [131065]), (40, [131072]), (50, [3, 131071, 0, 2])])
def test_a_group_of_many_columns(T, groups):
    print("modes many", T, groups, flush=True)
    n, k = len(groups), 3
    x = ring_down(T, sum(groups), np.random.default_rng(T))
    b = lbw.Batch([BOX] * n, [np.zeros(27)] * n, [np.arange(c) % 27 for c in groups], t_max=T)
    b.step(T)
    b.trace.copy_(torch.as_tensor(x))
    freq, power = b.modes(k)
    col = 0
    for h, c in enumerate(groups):
        if c == 0:
            assert np.isnan(freq[h]).all()
            continue
        fo, po = oracle.modes(x[:, col:col + c], k)
        col += c
        close(freq[h], fo)
        close(power[h], po)
    if n == 1:  # a state, and the fixed work space: the same bits
        sim = lbw.Simulation(lbw.Geometry(BOX), np.zeros(27), np.arange(groups[0]) % 27, t_max=T)
        sim.step(T)
        sim.trace.copy_(torch.as_tensor(x))
        fs, ps = sim.modes(k)
        fd, pd = (torch.zeros(k, dtype=torch.float64, device="cuda") for _ in range(2))
        sim.modes_noalloc(k, fd, pd)
        torch.cuda.synchronize()
        for got, want in ((fs, freq[0]), (ps, power[0]), (fd.cpu().numpy(), freq[0]), (pd.cpu().numpy(), power[0])):
            assert np.array_equal(got, want, equal_nan=True)
