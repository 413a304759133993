"""GPU: spectra of recorded traces over the lengths and group sizes at which
the device transform changes its split (n = n1 n2 held in LDS, 4 to 8192
points a line) and its pairing of columns, against the oracle's numpy FFT.

Tolerance: an FP64 transform of n points is off by about eps log2(n) of its
largest amplitude; a peak is kept from 1e-3 of the largest power, 0.03 of the
largest amplitude, so its power is off by at most 2 eps log2(n) / 0.03 =
4e-13 of itself at n = 2^21, and the parabola through the logarithms (whose
curvature at a Hann-windowed peak padded four to eight times is about 0.1)
moves by about ten times that, in bins, of at least 16.  Held to 1e-10.
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
    """Six decaying lines per column, 6.3 / T apart, on a constant."""
    t = np.arange(T)[:, None]
    x = np.full((T, cols), 0.1)
    for i in range(1, 7):
        x += (rng.uniform(0.3, 1.0, cols) * np.exp(-rng.uniform(0.5, 2.0) / T * t)
              * np.sin(2 * np.pi * t * (6.3 * i / T + 0.001) + rng.uniform(0, 6, cols)))
    return x


@pytest.mark.parametrize("T,groups", [(8, [1]), (9, [2, 0, 3]), (33, [1, 2]), (1000, [9, 1, 0, 4]), (2049, [3]),
                                      (5000, [8] * 30), (40000, [16]), (70000, [3, 9]), (131072, [7]),
                                      (300000, [1, 2])])
def test_spectra_match_the_oracle_at_every_split(T, groups):
    print("modes", T, groups, flush=True)
    n, k = len(groups), 6
    b = lbw.Batch([BOX] * n, [np.zeros(27)] * n, [list(range(c)) for c in groups], t_max=T)
    b.step(T)
    x = ring_down(T, sum(groups), np.random.default_rng(T))
    b.trace.copy_(torch.as_tensor(x))
    freq, power = b.modes(k)
    col = 0
    for h, c in enumerate(groups):
        if c == 0:
            assert np.isnan(freq[h]).all() and np.isnan(power[h]).all()
            continue
        fo, po = oracle.modes(x[:, col:col + c], k)
        col += c
        assert np.array_equal(np.isnan(freq[h]), np.isnan(fo))
        m = ~np.isnan(fo)
        assert np.allclose(freq[h][m], fo[m], rtol=1e-10, atol=0) and np.allclose(power[h][m], po[m], rtol=1e-10, atol=0)
    if n == 1:  # the same columns through a state, and through the fixed work space: the same bits
        sim = lbw.Simulation(lbw.Geometry(BOX), np.zeros(27), list(range(groups[0])), t_max=T)
        sim.step(T)
        sim.trace.copy_(torch.as_tensor(x))
        fs, ps = sim.modes(k)
        fd, pd = (torch.zeros(k, dtype=torch.float64, device="cuda") for _ in range(2))
        sim.modes_noalloc(k, fd, pd)
        torch.cuda.synchronize()
        for got, want in ((fs, freq[0]), (ps, power[0]), (fd.cpu().numpy(), freq[0]), (pd.cpu().numpy(), power[0])):
            assert np.array_equal(got, want, equal_nan=True)
