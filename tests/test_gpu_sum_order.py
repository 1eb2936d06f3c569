"""How far the order of the spreading's atomic additions moves a 16-bit run."""
import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I
from parity import Case, run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("storage,scale,quantum", [(2, 20, 2.0**-10), (3, 0, 2.0**-7)])
@pytest.mark.parametrize("kernel,n", [(2, 5000), (3, 2500)])
def test_16_bit_run_moves_by_quanta(kernel, n, storage, scale, quantum):
    """A dense box by floating-point atomics (unordered sums) against the exact sums of the
    deterministic mode.  The FP32 sums differ in their last bits, which now and then flips a
    stored population by its quantum; ten of them make up a velocity component, so the
    velocities lie within ten quanta of the largest population."""
    box = (32, 32, 32)
    pos = I.uniform_positions(n, box, 7)
    vel = np.random.default_rng(n).normal(0.0, 1e-3, (n, 3))
    runs = []
    for det in (0, 1):
        c = Case(name=f"quanta_s{storage}_k{kernel}_d{det}", nx=32, ny=32, nz=32, tau=0.8, steps=20, coupling=1,
                 gamma=1.0, kernel=kernel, storage=storage, u_noise=1e-3, pos=pos, vel=vel,
                 mass=np.ones(n), f16_scale_log2=scale, extra=dict(deterministic=det))
        runs.append(run_gpu(c))
    a, b = runs
    worst = np.abs(a["u"] - b["u"]).max()
    print(f"[order] storage {storage} kernel {kernel}: {worst:.2e}, rms {np.sqrt((b['u']**2).mean()):.2e}", flush=True)
    assert worst <= 10 * quantum * np.abs(b["df"]).max()
    assert np.abs(a["pos"] - b["pos"]).max() <= 20 * 10 * quantum * np.abs(b["df"]).max()
