"""GPU: the buffer that holds a state after n steps is that of n single steps,
however many steps a launch takes (2-D tiles, and the two-step launches that an
untuned 3-D grid takes by rule), so an even number of steps captured by a
caller and replayed goes on where it ended.

Sizes: a 2-D grid in one workgroup and one in tiles, a 3-D grid whose rule
takes two steps per launch and one whose rule does not.
"""
import numpy as np
import pytest
import torch

import paper_1705_01801_amd as lbw

pytestmark = pytest.mark.gpu


def disk(n0, n1):
    return dict(kind="polar2d", dim=2, n=(n0, n1), qmin=(0.05, 0.0), qmax=(1.0, 2 * np.pi),
                bc_lo=("bounceback", "periodic"), bc_hi=("fixed", "periodic"), h_ref=0.95 / n0, c=0.1, damp=1.0,
                params=())


def torus(n0, n1, n2):
    return dict(kind="torus", dim=3, n=(n0, n1, n2), qmin=(0.05, 0.0, 0.0), qmax=(1.0, 2 * np.pi, 2 * np.pi),
                bc_lo=("bounceback", "periodic", "periodic"), bc_hi=("bounceback", "periodic", "periodic"),
                h_ref=0.95 / n0, c=0.05, damp=1.0, params=(3.0,))


CASES = {"disk_whole": (disk(40, 50), None), "disk_tiles": (disk(150, 203), None),
         "torus_two": (torus(96, 200, 201), True), "torus_one": (torus(20, 31, 50), False)}


@pytest.mark.parametrize("name", sorted(CASES))
def test_state_ends_in_the_buffer_of_single_steps(name):
    geom, two = CASES[name]
    print("buffers", name, flush=True)
    g = lbw.Geometry(geom)
    if two is not None:
        assert (g.step2_config()[0] > 0) == two
    N = int(np.prod(geom["n"]))
    P0 = np.random.default_rng(N).uniform(-1, 1, N)
    a, b = (lbw.Simulation(g, P0, [0, 1, N - 1], t_max=400) for _ in range(2))
    for n in (1, 1, 2, 3, 4, 5, 6, 7, 8, 13, 22, 36, 50, 67):
        before = a.populations().data_ptr()
        a.step(n)
        assert (a.populations().data_ptr() == before) == (n % 2 == 0), n
    for _ in range(a.t):
        b.step(1)
    assert torch.equal(a.populations(), b.populations())
    assert torch.equal(a.trace, b.trace)


@pytest.mark.parametrize("n", [2, 6, 12])
@pytest.mark.parametrize("name", sorted(CASES))
def test_replays_of_an_even_number_of_steps_go_on(name, n):
    geom = CASES[name][0]
    print("replays", name, n, flush=True)
    g = lbw.Geometry(geom)
    N = int(np.prod(geom["n"]))
    P0 = np.random.default_rng(N).uniform(-1, 1, N)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    a = lbw.Simulation(g, P0, [0, N - 1], t_max=100, stream=side)
    b = lbw.Simulation(g, P0, [0, N - 1], t_max=100)
    side.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        a.step(n)
    work = torch.ones(1 << 16, device="cuda")
    for replay in range(4):
        with torch.cuda.stream(side):
            graph.replay()
        side.synchronize()
        work = work.mul(1.5).sub(0.5)  # (the program's own work in between)
        torch.cuda.synchronize()
        b.step(n)
        torch.cuda.synchronize()
        assert torch.equal(a.populations(), b.populations()), replay
        assert torch.equal(a.trace[:n * (replay + 1)], b.trace[:n * (replay + 1)]), replay
    a.close()
    b.close()
