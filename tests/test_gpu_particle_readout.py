"""lb_get_particles into every kind of memory that a copy of the runtime reaches
(a kernel writes to the context's own GPU only), either array alone, and under
graph capture."""
import ctypes as C

import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I

pytestmark = pytest.mark.gpu


def _lattice(n, stream=None):
    import torch
    from paper_1406_2211_amd import lbc as L
    lat = L.Lattice(24, 20, 18, max_particles=n, stream=stream, tau=0.8, coupling=L.LB_COUPLE_FC, gamma=1.0)
    lat.lb_set_particles(I.uniform_positions(n, (24, 20, 18), 3), np.full((n, 3), 1e-3), np.ones(n))
    lat.lb_step(2)
    torch.cuda.synchronize()
    return lat


def _get(lat, pos, vel):
    p = [None if t is None else C.c_void_p(t.data_ptr()) for t in (pos, vel)]
    lat._call("lb_get_particles", *p)


@pytest.mark.parametrize("n", [1, 85, 86, 700])
@pytest.mark.parametrize("kind", ["device", "pinned", "device and pinned"])
def test_kinds_of_memory(kind, n):
    import torch
    lat = _lattice(n)
    pos, vel = lat.lb_get_particles()
    print(f"[gpu] particles into {kind}, n={n}", flush=True)

    def new(k):
        return torch.zeros((n, 3), dtype=torch.float64, pin_memory=True) if k == "pinned" else \
            torch.zeros((n, 3), dtype=torch.float64, device="cuda")

    kinds = kind.split(" and ") * 2
    p, v, only = new(kinds[0]), new(kinds[1]), new(kinds[1])
    _get(lat, p, v)
    _get(lat, None, only)
    _get(lat, None, None)
    torch.cuda.synchronize()
    assert torch.equal(p.cpu(), pos.cpu()) and torch.equal(v.cpu(), vel.cpu())
    assert torch.equal(only.cpu(), vel.cpu())


def test_captured_readout():
    """A captured read-out, replayed between eager steps, gives the state of each time."""
    import torch
    n, s = 40, torch.cuda.Stream()
    lat = _lattice(n, s)
    pos, vel = (torch.zeros((n, 3), dtype=torch.float64, device="cuda") for _ in range(2))
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    print("[gpu] captured read-out of particles", flush=True)
    with torch.cuda.graph(g, stream=s):
        _get(lat, pos, vel)
    for _ in range(3):
        lat.lb_step(2)
        with torch.cuda.stream(s):
            g.replay()
        want = lat.lb_get_particles()
        torch.cuda.synchronize()
        assert torch.equal(pos, want[0]) and torch.equal(vel, want[1])
