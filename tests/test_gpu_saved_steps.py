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


@pytest.mark.parametrize("K", [1, 4])
def test_timing_counts_the_steps_of_the_run(K):
    """The step-kernel timing counts a taped run's steps, and none of those
    that its reverse recomputes (states of about 1 GB: those of 4 steps are not
    kept)."""
    w = workload("tg32", n=(16, 16, 16), P=2000, noise=0.2, dt=4e-4)
    U = fields(w, "fp32_local")[0]
    t = tracker(w, "fp32_local", capacity=26_000_000)
    t.inject(*w.particles())
    t.timing(True)
    for _ in range(6):
        t.step(U, w.dt, tape=K)
    ms, n = t.timing(True)
    assert n == 6 and ms > 0.0
    t.backward(t.sources())
    assert t.timing(False) == (0.0, 0)
    t.close()


def _free():
    """Free device memory once it has settled (freed memory comes back late)."""
    import time
    import torch
    torch.cuda.synchronize()
    seen = []
    while len(seen) < 4 or len(set(seen[-4:])) > 1:
        assert len(seen) < 100
        seen.append(torch.cuda.mem_get_info()[0])
        time.sleep(0.05)
    return seen[-1]


@pytest.mark.parametrize("K,steps,kept", [(3, 4, 2), (4, 4, 0), (2, 6, 2), (5, 3, 0)])
def test_states_of_whole_segments_only(K, steps, kept):
    """States of about 1 GiB, two of which may be kept: a segment keeps its
    states only where all of them fit."""
    import torch
    w = workload("tg32", n=(16, 16, 16), P=2000, noise=0.2, dt=4e-4)
    x, up, d = w.particles()
    U = fields(w, "fp32_local")[0]
    t = tracker(w, "fp32_local", capacity=26_000_000)
    t.inject(x, up, d)
    t.step(U, w.dt)
    t.sources(reset=True)
    for reserve in (False, True):
        t.tape_clear()
        free0 = _free()
        if reserve:
            t.tape_reserve(K, steps)
            reserved = _free()
        for _ in range(steps):
            t.step(U, w.dt, tape=K)
        states = -(-steps // K) + kept     # checkpoints too
        if reserve:
            assert _free() == reserved      # the run allocates nothing
        else:
            used = (free0 - _free()) / 2**30
            assert 0.95 * states < used < 1.35 * states, (used, states)
        lam = torch.cos(t.sources()).contiguous()
        dU, dd = t.backward(lam)
        if reserve:
            assert _free() == reserved      # nor does its reverse
        assert torch.isfinite(dU).all() and torch.isfinite(dd).all()
    t.close()


def test_reserve_gives_up_states_for_the_workspace():
    """Where the kept states leave no room for the reverse's workspace, the
    reservation gives them up instead of failing."""
    import torch
    w = workload("tg32", n=(16, 16, 16), P=2000, noise=0.2, dt=4e-4)
    x, up, d = w.particles()
    U = fields(w, "fp32_local")[0]
    ref = tracker(w, "fp32_local")
    t = tracker(w, "fp32_local", capacity=26_000_000)
    for v in (ref, t):
        v.inject(x, up, d)
        v.step(U, w.dt)
        v.sources(reset=True)
    # two checkpoints, then two states of the first segment and a workspace of
    # three states and the records: with the states it does not fit
    fill = torch.empty(_free() - (27 << 28), dtype=torch.uint8, device="cuda")
    t.tape_reserve(3, 6)
    del fill
    torch.cuda.empty_cache()
    for v in (ref, t):
        for _ in range(6):
            v.step(U, w.dt, tape=3)
    lam = torch.cos(ref.sources() * 1e3).contiguous()
    got, want = t.backward(lam), ref.backward(lam)
    for a, b in zip(got, want):
        assert float((a - b).norm()) < 1e-6 * float(b.norm())
    t.close()
    ref.close()
