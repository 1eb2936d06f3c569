"""The cache policies of the lattice pass, chosen by the size of the two
population buffers (cached from 32 MiB, cached with alternating sweeps from 240
to 290 MiB, non-temporal loads with cached stores and alternating sweeps from
500 MiB): an odd number of force-coupled steps on the row-mapped and the
linear-site pass against the oracle, FP64 at 1e-12, FP32 at 1e-5 and FP16 at
1e-3 (the tolerances of the parity and precision tests)."""
import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I
from parity import Case, compare, run_gpu, run_oracle

pytestmark = pytest.mark.gpu

# box, storage, collision, wall, kT
CASES = [
    ((64, 60, 66), 0, 0, 0, 0.0),       # 74 MiB, rows
    ((75, 60, 72), 0, 1, 1, 0.0),       # 94 MiB, linear sites, walls
    ((96, 96, 96), 0, 0, 0, 0.0),       # 257 MiB, linear sites, alternating
    ((128, 112, 128), 1, 2, 0, 0.0),    # 266 MiB, rows, MRT, alternating
    ((64, 128, 128), 1, 1, 0, 1e-5),    # 152 MiB, rows, noise
    ((128, 96, 128), 2, 1, 0, 0.0),     # 114 MiB, rows, FP16
    ((128, 112, 128), 0, 1, 1, 0.0),    # 532 MiB, rows, walls, written lines kept
    ((160, 160, 160), 1, 2, 0, 0.0),    # 594 MiB, linear sites, MRT, written lines kept
]


@pytest.mark.parametrize("box,storage,collision,wall,kT", CASES)
def test_cache_policy(box, storage, collision, wall, kT):
    n = 40
    pos = I.uniform_positions(n, box, 9)
    if wall:
        pos[:, 1] = np.clip(pos[:, 1], 0.6, box[1] - 1.6)
    vel = np.random.default_rng(3).normal(0.0, 1e-3, (n, 3))
    extra = dict(mrt_rates=(1.4, 1.2, 1.2, 1.5, 1.5))
    if kT > 0:
        extra.update(kT=kT, seed=5)
    c = Case(name=f"cache_{'x'.join(map(str, box))}_s{storage}_c{collision}", nx=box[0], ny=box[1],
             nz=box[2], tau=0.7, steps=3, wall_y=wall, collision=collision, coupling=1, gamma=1.0,
             storage=storage, u_noise=1e-3, pos=pos, vel=vel, mass=np.ones(n),
             f16_scale_log2=20 if storage == 2 else 0, extra=extra)
    compare(c, run_gpu(c), run_oracle(c), {0: 1e-12, 1: 1e-5, 2: 1e-3}[storage])
