"""Population arrays of 4 GiB and more take 64-bit offsets inside an array: a box
made of many copies of a small one along z, 540 million FP64 sites (about 200 GB
of device memory), moves as the small box does, within the rounding of the two
kernels (1e-12)."""
import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I

pytestmark = pytest.mark.gpu
NX, NY, NZ, COPIES, STEPS = 1001, 540, 10, 100, 3


def _flow():
    import torch
    return torch.from_numpy(I.noise_velocity((NZ, NY, NX), 1e-3, 5)).cuda()


def _room():
    import torch
    torch.cuda.empty_cache()
    if torch.cuda.mem_get_info()[0] < 240e9:
        pytest.skip("needs 240 GB of free device memory")


def _compare(u, want):
    worst = max(float((u[:, k * NZ:(k + 1) * NZ] - want).abs().max()) for k in range(COPIES))
    assert worst <= 1e-12 * float(want.abs().max())


@pytest.mark.parametrize("wall", [0, 1])
def test_big_linear_box(wall):
    import torch
    from paper_1406_2211_amd import lbc as L
    _room()
    p = dict(wall_y=wall, tau=0.7, collision=L.LB_TRT, body_force=(1e-6, 0.0, 2e-6), storage=L.LB_F64)
    small = L.Lattice(NX, NY, NZ, **p)
    small.lb_init_fluid(None, _flow())
    small.lb_step(STEPS)
    want = small.lb_moments()[1]
    print(f"[gpu] big box, walls {wall}", flush=True)
    lat = L.Lattice(NX, NY, NZ * COPIES, **p)
    lat.lb_init_fluid(None, _flow().repeat(1, COPIES, 1, 1))
    torch.cuda.synchronize()
    lat._keep = ()
    lat.lb_step(STEPS)
    _compare(lat.lb_moments()[1], want)
    lat.lb_destroy()
    lat.workspace = None


def test_big_ensemble_box():
    """A big box beside a small one in an ensemble, admitted after a step without it
    (the captured steps change over to 64-bit offsets)."""
    import torch
    from paper_1406_2211_amd import lbc as L
    _room()
    p = dict(tau=0.7, collision=L.LB_TRT, body_force=(1e-6, 0.0, 2e-6))
    pool = sum(L.ensemble_footprint(NX, NY, nz, storage=L.LB_F64, **p) for nz in (NZ, NZ * COPIES)) + (2 << 30)
    ens = L.Ensemble(pool, 2, storage=L.LB_F64)
    got = {}
    for nz in (NZ, NZ * COPIES):
        slot, lat = ens.admit(NX, NY, nz, STEPS, **p)
        lat.lb_init_fluid(None, _flow().repeat(1, nz // NZ, 1, 1))
        torch.cuda.synchronize()
        lat._keep = ()
        print(f"[gpu] ensemble box of nz {nz}", flush=True)
        ens.step(STEPS)
        assert ens.query(slot) == (STEPS, True)
        got[nz] = lat.lb_moments()[1]
        torch.cuda.synchronize()
    _compare(got[NZ * COPIES], got[NZ])
    ens.destroy()
    ens.pool = None
