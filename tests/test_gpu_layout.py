"""The layout of a full re-bin on the GPU, made by one workgroup and by several
launches, at chunk counts on either side of where they meet (behind injections
and behind steps) and at ones that fill no whole blocks, with a chunk of two
containers that empties into its neighbours: lockstep against the FP64 oracle."""
import numpy as np
import pytest

from gpu_helpers import band, fields, lockstep_check, oracle_mesh, state, tracker, workload
from oracle.oracle import load as load_oracle

pytestmark = pytest.mark.gpu

TOL = {   # as in the lockstep parity tests
    "fp64": {"pos": 1e-13, "vel": 1e-12, "src": 1e-10},
    "fp32_local": {"pos": 1e-5, "vel": 1e-5, "src": 1e-6},
}
TOL_FP32 = {"pos": 1e-5, "vel": 1e-5, "src": 1e-4}


@pytest.mark.parametrize("form", sorted(TOL))
@pytest.mark.parametrize("n,chunks", [((32, 32, 16), 2048), ((32, 34, 16), 2176),
                                      ((32, 32, 32), 4096), ((32, 34, 32), 4352),
                                      ((64, 64, 64), 32768), ((64, 66, 64), 33792),
                                      ((66, 70, 62), 35805)])
def test_layouts(form, n, chunks):
    orc = load_oracle()
    P = 60_000
    w = workload("tg32", n=n, L=tuple(0.1 * v / 64 for v in n), P=P, noise=0.3, chunk_edge=2)
    assert n[0] * n[1] * n[2] // 8 == chunks
    rng = np.random.default_rng(chunks)
    x = rng.random((P, 3)) * np.array(w.L)
    x[:20_000] = rng.random((20_000, 3)) * 2 * w.h         # one chunk
    up = rng.normal(0.0, 1.0, (P, 3))
    d = np.full(P, 60e-6)
    t = tracker(w, form, capacity=P + 100)
    Udev, Uor = fields(w, form)
    vmax = float(np.abs(up).max())
    tol = dict(TOL[form], vel=TOL[form]["vel"] * vmax)
    t.inject(x[:40_000], up[:40_000], d[:40_000])
    lockstep_check(t, orc, oracle_mesh(w), Udev, Uor, 1e-3, 2, tol)
    t.inject(x[40_000:], up[40_000:], d[40_000:])
    before = t.stats()["repacks"]
    lockstep_check(t, orc, oracle_mesh(w), Udev, Uor, 1e-3, 4, tol)
    st = t.stats()
    assert st["repacks"] > before + 1, st                  # (one places the injection)
    assert np.array_equal(state(t)["id"], np.arange(P))
    t.close()


def _lockstep_mixing(form, n, P, steps, t_of):
    """A tracker of a sparse mesh of 2-cell chunks, a few thousand droplets in one
    of them, most droplets in another chunk after every step."""
    orc = load_oracle()
    w = workload("tg32", n=n, L=tuple(0.1 * v / 64 for v in n), P=P, noise=0.3, chunk_edge=2)
    rng = np.random.default_rng(P)
    x = rng.random((P, 3)) * np.array(w.L)
    x[:3000] = rng.random((3000, 3)) * 2 * w.h
    up = rng.normal(0.0, 2.0, (P, 3))
    d = np.full(P, 60e-6)
    Udev, Uor = fields(w, form)
    t = t_of(w)
    vmax = float(np.abs(up).max())
    tol = dict(TOL[form], vel=TOL[form]["vel"] * vmax)
    t.inject(x, up, d)
    lockstep_check(t, orc, oracle_mesh(w), Udev, Uor, 1e-3, steps, tol)
    assert np.array_equal(state(t)["id"], np.arange(P))
    st = t.stats()
    assert st["movers"] > P // 3, st
    t.close()
    return st


@pytest.mark.parametrize("form,n,leave,least", [("fp64", 96, 10, 1), ("fp64", 128, 20, 3),
                                                ("fp32_local", 128, 11, 3)])
def test_small_inboxes_where_memory_is_short(form, n, leave, least):
    """A device that has room for the store, but only for smaller inboxes beside
    it (of the first or the second smaller size), holds the tracker all the same."""
    import torch
    from test_gpu_blocks import _fill
    import paper_2603_26691_amd as pkg
    pkg.release_memory()

    def make(w):
        held = _fill(leave)
        t = tracker(w, form)
        del held
        torch.cuda.empty_cache()
        return t

    st = _lockstep_mixing(form, (n, n, n), 30_000, 3, make)
    assert st["repacks"] >= least        # (the smallest inboxes mostly hold one record)


@pytest.mark.parametrize("form,n,edge,P,crowd", [
    ("fp32", (64, 66, 64), 2, 100_000, 5000), ("fp32_local", (64, 66, 64), 2, 33_792 * 12, 5000),
    ("fp32_local", (64, 66, 64), 2, 33_792 * 12 + 1, 5000),      # on either side of the line
    ("fp64", (128, 132, 128), 4, 60_000, 20_000), ("fp32", (128, 128, 128), 4, 90_000, 20_000)])
def test_steps_of_sparse_small_chunks(form, n, edge, P, crowd):
    """Few droplets a chunk but for one that holds more than a workgroup stages
    of movers and arrivals."""
    orc = load_oracle()
    w = workload("tg32", n=n, L=tuple(0.1 * v / 64 for v in n), P=P, noise=0.3, chunk_edge=edge)
    rng = np.random.default_rng(P)
    x = rng.random((P, 3)) * np.array(w.L)
    x[:crowd] = rng.random((crowd, 3)) * edge * w.h
    up = rng.normal(0.0, 1.0, (P, 3))
    up[:crowd] += 1.5                                   # most of them leave it together
    d = np.full(P, 60e-6)
    t = tracker(w, form)
    Udev, Uor = fields(w, form)
    vmax = float(np.abs(up).max())
    tol = dict(TOL.get(form, TOL_FP32))
    tol["vel"] *= vmax
    bnd = band(form, w.n)
    if form == "fp32":   # the binary32 rounding of the largest position
        bnd = max(bnd, 2.0 ** -21 * (max(w.L) + vmax * 1e-3) / min(w.h))
    t.inject(x, up, d)
    lockstep_check(t, orc, oracle_mesh(w), Udev, Uor, 1e-3, 3, tol, band_=bnd)
    assert np.array_equal(state(t)["id"], np.arange(P))
    assert t.stats()["movers"] > P // 4
    t.close()


@pytest.mark.parametrize("form,interp,tol", [("fp64", "trilinear", 1e-9), ("fp32_local", "ngp", 1e-4)])
def test_adjoint_of_sparse_small_chunks(form, interp, tol):
    import torch
    orc = load_oracle()
    n, P, steps, dt = (64, 66, 64), 4000, 6, 5e-4
    w = workload("tg32", n=n, L=tuple(0.1 * v / 64 for v in n), P=P, noise=0.2, chunk_edge=2)
    x, up, d = w.particles()
    Udev, Uor = fields(w, form)
    t = tracker(w, form, interp=interp)
    t.inject(x, up, d)
    s0 = state(t)
    for _ in range(steps):
        t.step(Udev, dt, tape=3)
    lam = torch.from_numpy(np.random.default_rng(1).normal(size=Uor.shape)).cuda()
    dU, dd = (v.cpu().numpy() for v in t.backward(lam))
    oU, od = orc.adjoint_run(oracle_mesh(w, interp=1 if interp == "ngp" else 0), np.stack([Uor]),
                             [0] * steps, [dt] * steps, 1, s0["x"], s0["up"], s0["d"],
                             lam.cpu().numpy())
    assert np.linalg.norm(dU - oU[0]) <= tol * np.linalg.norm(oU)
    assert np.linalg.norm(dd - od) <= tol * np.linalg.norm(od)
    t.close()


@pytest.mark.parametrize("form", ["fp64", "fp32_local", "fp32"])
@pytest.mark.parametrize("per", [64, 65])
def test_scatter_by_waves_and_workgroups(form, per):
    """Particles a container on either side of where the re-bin's scatter goes by
    waves, with containers of more slots than a wave takes, of one wave's and of none;
    droplets whose inbox is full among them."""
    orc = load_oracle()
    n, edge = (32, 32, 40), 4
    w = workload("tg32", n=n, L=tuple(0.1 * v / 32 for v in n), P=1, noise=0.3, chunk_edge=edge)
    chunks = n[0] * n[1] * n[2] // edge ** 3
    # (particles per container: a container more per 16384 of the capacity)
    P = per * (chunks + 3)
    assert -(-P // 16384) == 3
    w = workload("tg32", n=n, L=w.L, P=P, noise=0.3, chunk_edge=edge)
    rng = np.random.default_rng(per)
    x = rng.random((P, 3)) * np.array(w.L)
    k = P // 2
    x[:k] = rng.random((k, 3)) * (8 * w.h) + 5 * w.h          # a few crowded chunks
    x[k: k + P // 4, 0] *= 0.05                               # and a thin layer
    up = rng.normal(0.0, 2.0, (P, 3))
    d = np.full(P, 60e-6)
    t = tracker(w, form)
    Udev, Uor = fields(w, form)
    vmax = float(np.abs(up).max())
    tol = dict(TOL.get(form, TOL_FP32))
    tol["vel"] *= vmax
    bnd = band(form, w.n)
    if form == "fp32":   # the binary32 rounding of the largest position
        bnd = max(bnd, 2.0 ** -21 * (max(w.L) + vmax * 1e-3) / min(w.h))
    t.inject(x[:P - 500], up[:P - 500], d[:P - 500])
    lockstep_check(t, orc, oracle_mesh(w), Udev, Uor, 1e-3, 2, tol, band_=bnd)
    t.inject(x[P - 500:], up[P - 500:], d[P - 500:])
    before = t.stats()["repacks"]
    lockstep_check(t, orc, oracle_mesh(w), Udev, Uor, 1e-3, 3, tol, band_=bnd)
    assert t.stats()["repacks"] > before
    assert np.array_equal(state(t)["id"], np.arange(P))
    t.close()
