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
