"""GPU: a tuning that ends in an error leaves the launches of the batch as they
were.

The error is forced from the host: the batch's stream is being captured, where
waiting for it is an error that ends the capture; no kernel runs for it.  Such a
stream takes no further work, so this happens in a process of its own.
"""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = """
import ctypes
import numpy as np, torch
import paper_1705_01801_amd as lbw

def pipe(n):
    return dict(kind="cylinder", dim=3, n=n, qmin=(1.0, 0.0, 0.0), qmax=(1.0 + n[0], 2.0 * np.pi, 1.0 * n[2]),
                bc_lo=("bounceback", "periodic", "bounceback"), bc_hi=("bounceback", "periodic", "fixed"), h_ref=1.0,
                damp=0.65, params=(), c=0.02)

cases = []
for n, launch in (((20, 52, 40), 1), ((20, 52, 40), 2), ((8, 12, 40), 2), ((8, 12, 40), 32)):
    side = torch.cuda.Stream()
    b = lbw.Batch([pipe(n)] * 2, [np.ones(n[0] * n[1] * n[2])] * 2, [[3], [7]], t_max=60, stream=side)
    b.set_step_config(16, 5)
    b.set_steps_per_launch(launch)
    b.step(9)
    cases.append((n, launch, side, b))
torch.cuda.synchronize()
hip = ctypes.CDLL(next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l))
for n, launch, side, b in cases:
    shape, launches = b.step_config(), b.steps_per_launch()
    assert launches[0] == launch, launches
    graph = ctypes.c_void_p()
    assert hip.hipStreamBeginCapture(ctypes.c_void_p(side.cuda_stream), 2) == 0  # (relaxed: allocations are allowed)
    try:
        b.autotune(reps=2)
        raise SystemExit("the tuning did not fail")
    except lbw.LbwError as e:
        print(n, launch, e, flush=True)
    assert hip.hipStreamEndCapture(ctypes.c_void_p(side.cuda_stream), ctypes.byref(graph)) != 0
    hip.hipGetLastError()
    assert b.step_config() == shape, (n, launch, b.step_config())
    assert b.steps_per_launch() == launches, (n, launch, b.steps_per_launch())
print("launches kept", flush=True)
"""


def test_failed_tuning_keeps_the_launches():
    print("tuning fails", flush=True)
    r = subprocess.run([sys.executable, "-c", CHILD], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and "launches kept" in r.stdout, r.stdout + r.stderr
