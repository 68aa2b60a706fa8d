"""The adjoint from the states that the forward run kept and from recomputed
ones, on the GPU: a tracker whose capacity leaves no room for all of them
(kept, recomputed and single-step segments in one tape) against one that keeps
them all, and both against the FP64 oracle's adjoint."""
import numpy as np
import pytest

from gpu_helpers import fields, oracle_mesh, state, tracker, workload
from oracle.oracle import load as load_oracle

pytestmark = pytest.mark.gpu

SAVED = 2 << 30      # bytes of kept states at most


def _gradients(t, w, U, K, nsteps, nsub, reserve):
    import torch
    x, up, d = w.particles()
    t.inject(x, up, d)
    t.step(U, w.dt)
    t.sources(reset=True)
    s0 = state(t)
    if reserve:
        t.tape_reserve(K, nsteps * nsub)
    t.timing(True)
    for _ in range(nsteps):
        t.step(U, w.dt, nsub=nsub, tape=K)
    assert t.timing(False)[1] == nsteps * nsub     # taped steps are timed too
    S = t.sources()
    end = state(t)
    lam = torch.cos(S * 1e3).contiguous()
    out = [g.cpu().numpy() for g in t.backward(lam)]
    after = state(t)
    for k in end:
        assert np.array_equal(end[k], after[k]), k   # the store is as the run left it
    return s0, lam.cpu().numpy(), out


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("form,interp,tol", [("fp64", "trilinear", 1e-9), ("fp64", "ngp", 1e-9),
                                             ("fp32_local", "trilinear", 1e-4)])
@pytest.mark.parametrize("K,nsteps,nsub,reserve", [(3, 10, 1, False), (2, 4, 2, True),
                                                   (1, 3, 1, False)])
def test_kept_and_recomputed(form, interp, tol, K, nsteps, nsub, reserve):
    orc = load_oracle()
    w = workload("tg32", n=(24, 16, 32), L=(0.075, 0.05, 0.1), P=6000, noise=0.2, dt=4e-4)
    U, Uor = fields(w, form)
    # about 1 GB a state: two of them are kept
    big = 14_000_000 if form == "fp64" else 26_000_000
    grads = []
    for capacity in (w.P, big):
        t = tracker(w, form, capacity=capacity, interp=interp)
        s0, lam, g = _gradients(t, w, U, K, nsteps, nsub, reserve)
        if grads:   # the same loss derivative to the sums' rounding
            assert _rel(lam, grads[0][1]) < 1e-6
        grads.append((s0, lam, g))
        if capacity == big:   # a second run on the same tracker, on kept buffers
            for _ in range(nsteps):
                t.step(U, w.dt, nsub=nsub, tape=K)
            assert all(np.isfinite(v.cpu().numpy()).all() for v in t.backward(t.sources()))
        t.close()
    (s0, lam, a), (_, _, b) = grads
    assert _rel(a[0], b[0]) < 1e-6 and _rel(a[1], b[1]) < 1e-6
    mesh = oracle_mesh(w, interp=1 if interp == "ngp" else 0)
    dts = [w.dt] * nsteps
    oU, od = orc.adjoint_run(mesh, np.stack([Uor]), [0] * nsteps, dts, nsub, s0["x"], s0["up"],
                             s0["d"], lam)
    for g in (a, b):
        assert _rel(g[0], oU) < tol and _rel(g[1], od) < tol, (_rel(g[0], oU), _rel(g[1], od))
