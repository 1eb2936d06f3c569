"""Spreading of coupling forces in partly filled wavefronts: particle counts at
the edges of a wavefront's 8, 2 or 1 particles (2-, 3-, 4-point kernel) and of
a workgroup's four wavefronts, FP64 against the oracle at 1e-12 and FP32 at
1e-5 (the tolerances of the parity tests)."""
import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I
from parity import Case, compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu


def _case(kernel, n, coupling, storage, wall=0):
    box = (20, 17, 19)
    pos = I.uniform_positions(n, box, 40 + n)
    if wall:
        pos[:, 1] = np.clip(pos[:, 1], 0.6, box[1] - 1.6)
    pos[1::2] = pos[:-1:2] + 0.4 if n % 2 == 0 else pos[1::2]  # neighbours share nodes
    vel = np.random.default_rng(n).normal(0.0, 1e-3, (n, 3)) if coupling != 3 else np.zeros((n, 3))
    return Case(name=f"spread_k{kernel}_n{n}_c{coupling}_s{storage}_w{wall}", nx=box[0], ny=box[1],
                nz=box[2], tau=0.8, steps=6, wall_y=wall, coupling=coupling, gamma=1.0,
                kernel=kernel, storage=storage, u_noise=1e-3, pos=pos, vel=vel, mass=np.ones(n))


@pytest.mark.parametrize("kernel", [2, 3, 4])
@pytest.mark.parametrize("n", [1, 2, 7, 8, 9, 31, 33, 64])
def test_partial_wavefronts_fp64(kernel, n):
    c = _case(kernel, n, 1, 0)
    compare(c, run_gpu(c), run_oracle(c), 1e-12)


@pytest.mark.parametrize("kernel,coupling,storage,wall", [(2, 2, 1, 1), (3, 2, 1, 0), (4, 1, 1, 1)])
def test_partial_wavefronts_fp32(kernel, coupling, storage, wall):
    c = _case(kernel, 35, coupling, storage, wall)
    compare(c, run_gpu(c), run_oracle(c), 1e-5)


@pytest.mark.parametrize("kernel,n,box", [(2, 4100, (40, 36, 33)), (3, 4096, (33, 40, 36)), (4, 4353, (64, 24, 20))])
def test_spatial_order(kernel, n, box):
    """Dense free particles are processed in tile order, rebinned every 32 steps:
    counts at the edges of the 8 equal runs of workgroups, across a rebinning."""
    pos = I.uniform_positions(n, box, 7 + kernel)
    vel = np.random.default_rng(n).normal(0.0, 2e-2, (n, 3))  # crosses tiles between binnings
    c = Case(name=f"order_k{kernel}_n{n}", nx=box[0], ny=box[1], nz=box[2], tau=0.8, steps=35,
             coupling=1, gamma=0.5, kernel=kernel, storage=0, u_noise=1e-3, pos=pos, vel=vel,
             mass=np.full(n, 2.0), extra=dict(chunks=[33, 2]))
    compare(c, run_gpu(c), run_oracle(c), 1e-12)


@pytest.mark.parametrize("kernel,n,coupling,inside,free", [
    (2, 12, 1, 0, 1), (2, 60, 2, 0, 1), (3, 20, 1, 0, 1), (4, 20, 2, 0, 1), (2, 60, 1, 1, 0)])
def test_lost_particle(kernel, n, coupling, inside, free):
    """A particle whose position is not a number (in one component or in all) neither
    reads nor forces the fluid: fluid and other particles are those of the run without it."""
    box = (20, 17, 19)
    pos = I.uniform_positions(n, box, 3 + n)
    vel = np.random.default_rng(n).normal(0.0, 1e-3, (n, 3))
    mts = dict(mts=3, extra=dict(mts_inside=1)) if inside else {}
    bonds = {} if free else dict(bonds=np.array([[0, 1], [2, 3]], np.int32), bond_k=1e-3, bond_r0=1.0)
    runs = []
    for lost in (0, 2):
        p, v = pos.copy(), vel.copy()
        if lost:
            p = np.concatenate([p, [[np.nan] * 3, [3.2, np.nan, 4.1]]])
            v = np.concatenate([v, np.zeros((2, 3))])
        c = Case(name=f"lost{lost}_k{kernel}_n{n}_c{coupling}_i{inside}", nx=box[0], ny=box[1],
                 nz=box[2], tau=0.8, steps=5, coupling=coupling, gamma=1.0, kernel=kernel,
                 storage=0, u_noise=1e-3, pos=p, vel=v, mass=np.ones(n + lost), **bonds, **mts)
        g = run_gpu(c)
        runs.append((g["df"], g["u"], g["pos"][:n], g["vel"][:n]))
    for a, b in zip(*runs):
        assert np.isfinite(b).all()
        assert np.abs(a - b).max() <= 1e-12 * np.abs(a).max()
