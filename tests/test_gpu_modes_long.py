"""GPU: the spectrum of a trace of more than 2^24 rows, whose transform (2^27
points) is too long for the LDS kernels and runs in radix-2 passes over memory.

The trace is four lines of known frequency and amplitude, far apart.  Their
peaks lie within a quarter of a padded bin of 1 / 2^27 (three-point interpolation
of a Hann main lobe eight padded bins half wide: its error is below a tenth of a
bin), and powers relate as the amplitudes squared to 1 % (the interpolated
top of the lobe, sampled at least every half padded bin: below 0.4 %).
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu


def test_more_rows_than_the_lds_kernels_take():
    T = 2 ** 24 + 5
    g = dict(kind="box", dim=3, n=(4, 4, 4), qmin=(0.0,) * 3, qmax=(4.0,) * 3, bc_lo=("bounceback",) * 3,
             bc_hi=("bounceback",) * 3, h_ref=1.0, c=0.5, damp=1.0, params=())
    b = lbw.Batch([g], [np.zeros(64)], [[0]], t_max=T)
    for part in range(4):
        b.step(T - b.t if part == 3 else T // 4)
        torch.cuda.synchronize()
        print("modes long: stepped", b.t, flush=True)
    freq, amp = np.array([0.010001, 0.0234567, 0.1100003, 0.3333]), np.array([1.0, 0.8, 0.6, 0.9])
    t = torch.arange(T, dtype=torch.float64, device="cuda")
    x = torch.zeros(T, dtype=torch.float64, device="cuda")
    for f, a in zip(freq, amp):
        x += a * torch.sin(2.0 * np.pi * ((f * t) % 1.0) + 0.3)
    b.trace[:T, 0] = x
    fr, pw = b.modes(4)
    print("modes long", fr, pw, flush=True)
    fr, pw = np.asarray(fr).reshape(-1), np.asarray(pw).reshape(-1)
    assert np.abs(fr - freq).max() <= 0.25 / 2 ** 27
    assert np.abs(pw / pw[0] - amp ** 2).max() <= 1e-2
