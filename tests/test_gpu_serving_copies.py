"""Kept velocity fields of a served batch, which threads copy beside the steps."""
import numpy as np
import pytest

from paper_1406_2211_amd import inputs as I

pytestmark = pytest.mark.gpu


def _requests(n, side=12, steps=20):
    return [I.Request(rid=k, arrival=0.0, side=side, nparticles=0, tau=0.8, fext=1e-6, steps=steps + k,
                      seed=k) for k in range(n)]


def _serve(reqs, pool=64 << 20, **kw):
    from paper_1406_2211_amd import serving as S
    return S.serve_batched(reqs, pool, max_slots=len(reqs), chunk=7, autotune=False, **kw)


@pytest.mark.parametrize("keep", [np.array([1, 2]), np.array([3]), np.array([], int), [0], (2, 3), set()])
def test_any_container_of_ids_is_kept(keep):
    print("[gpu] kept ids", keep, flush=True)
    fields = _serve(_requests(4), keep=keep)[1]
    assert sorted(fields) == sorted(int(k) for k in keep)
    for u in fields.values():
        assert u.shape == (3, 12, 12, 12) and np.isfinite(u).all() and u[0].mean() > 0


def test_an_exception_ends_the_copies_and_the_ensemble():
    """A log callback that raises while kept copies are under way: the threads have
    ended and the ensemble is gone when the exception arrives."""
    import threading
    import torch
    from paper_1406_2211_amd import lbc as L
    print("[gpu] exception in a served batch", flush=True)
    before, made = set(threading.enumerate()), []
    real = L.Ensemble

    class Seen(real):
        def __init__(self, *a, **kw):
            super().__init__(*a, **kw)
            made.append(self)

    def log(msg):
        if len(seen) == 2:
            raise RuntimeError("stop")
        seen.append(msg)

    seen = []
    L.Ensemble = Seen
    try:
        with pytest.raises(RuntimeError, match="stop"):
            _serve(_requests(8, side=64), pool=1 << 30, keep=range(8), log=log)
        assert not [t for t in threading.enumerate() if t not in before]
        assert len(made) == 1 and not made[0].ens
    finally:
        L.Ensemble = real
    torch.cuda.synchronize()
