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


def test_fields_under_way_are_bounded(monkeypatch):
    """However slowly the host takes them, at most 1 GiB of kept fields (or one field) waits in
    device memory beside the pool: 14 boxes of 160^3, 98 MB each, with copies that dawdle."""
    import time
    from paper_1406_2211_amd import serving as S
    reqs = _requests(14, side=160, steps=2)
    reqs = [I.Request(**{**r.__dict__, "steps": 2}) for r in reqs]
    state, high = {"now": 0}, []
    submit, copy = S._FieldCopier.submit, S._FieldCopier._copy

    def slow(self, src, dst, stream):
        time.sleep(0.05)
        t = copy(self, src, dst, stream)
        state["now"] -= dst.nbytes
        return t

    def counted(self, field, ready):
        state["now"] += 24 * field[0].numel()
        high.append(state["now"])
        return submit(self, field, ready)

    monkeypatch.setattr(S._FieldCopier, "_copy", slow)
    monkeypatch.setattr(S._FieldCopier, "submit", counted)
    print("[gpu] 14 kept fields of 160^3", flush=True)
    fields = _serve(reqs, pool=8 << 30, keep=range(14))[1]
    assert len(fields) == 14 and state["now"] == 0
    assert max(high) <= 1 << 30


def test_memory_held_by_copies_is_waited_for(monkeypatch):
    """Where a read-out finds no memory while copies are under way, it is made again after them."""
    import torch
    from paper_1406_2211_amd import lbc as L
    moments, calls = L.Lattice.lb_moments, []

    def short(self):
        calls.append(1)
        if len(calls) == 2:
            raise torch.OutOfMemoryError("no memory beside the copies")
        return moments(self)

    print("[gpu] a read-out refused once", flush=True)
    want = _serve(_requests(4), keep=range(4))[1]
    monkeypatch.setattr(L.Lattice, "lb_moments", short)
    got = _serve(_requests(4), keep=range(4))[1]
    assert len(calls) == 5 and sorted(got) == sorted(want)
    for k in want:
        assert np.abs(got[k] - want[k]).max() <= 1e-6 * np.abs(want[k]).max()
