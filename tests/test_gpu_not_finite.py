"""Droplets that no slot can hold, on the GPU: a field with cells that are no
numbers or infinite takes the droplets that read them out of the store, and a
batch injected in parts leaves its bad droplets out.  Every other droplet and
cell stays what it would be without them, across arrivals into the slots they
leave and full re-bins."""
import numpy as np
import pytest

from gpu_helpers import (FORMS, band, face_distance, fields, min_image, oracle_mesh, state,
                         tracker, workload)
from oracle.oracle import load as load_oracle

pytestmark = pytest.mark.gpu

TOL = {   # as in the lockstep parity tests
    "fp64": {"pos": 1e-13, "vel": 1e-12, "src": 1e-10},
    "fp32_local": {"pos": 1e-5, "vel": 1e-5, "src": 1e-6},
    "fp32": {"pos": 1e-5, "vel": 1e-5, "src": 1e-4},
}


def _finite(*arrays):
    return np.logical_and.reduce([np.isfinite(a).all(axis=1) for a in arrays])


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("P,interp", [(40_000, "trilinear"), (150_000, "trilinear"),
                                      (40_000, "ngp")])
def test_field_with_cells_that_are_not_finite(form, P, interp):
    import torch
    orc = load_oracle()
    w = workload("tg32", P=P, noise=0.1)
    mesh = oracle_mesh(w, interp=1 if interp == "ngp" else 0)
    rng = np.random.default_rng(P)
    x, _, d = w.particles()
    up = rng.normal(0.0, 3.0, (P, 3))       # about a cell a step, 3 in 10 change chunk
    d[:] = 60e-6                            # and keep their velocity
    vmax = float(np.abs(up).max())
    Udev, Uor = fields(w, form)
    Uor = Uor.copy()
    for c, v in [(0, np.nan), (0, np.inf), (0, -np.inf), (1, np.nan), (2, np.inf)]:
        k, j, i = rng.integers(0, 32, (3, 4))
        Uor[c, k, j, i] = v
    Udev = torch.from_numpy(Uor).to(Udev.dtype).cuda()
    t = tracker(w, form, capacity=P + 4000, interp=interp)
    t.inject(x, up, d)
    h, L = w.h, np.array(w.L)
    bnd = band(form, w.n)
    if form == "fp32":   # the binary32 rounding of the largest position
        bnd = max(bnd, 2.0 ** -21 * (max(w.L) + vmax * 1e-3) / min(h))
    gone = 0
    for step in range(10):
        if step in (4, 7):                  # a full re-bin; new droplets read the same cells
            n = 1500
            t.inject(rng.random((n, 3)) * L, rng.normal(0.0, 3.0, (n, 3)), np.full(n, 60e-6))
        s0 = state(t)
        live = (s0["id"] >= 0) & _finite(s0["x"], s0["up"])
        ill = (s0["id"] >= 0) & ~live     # a finite first coordinate keeps them in the store
        q = {k: v[live] for k, v in s0.items()}
        t.sources(reset=True)
        t.step(Udev, 1e-3)
        s1 = state(t)
        S = t.sources(reset=True).cpu().numpy()
        xo, uo, So = orc.run(mesh, Uor, q["x"], q["up"], q["d"], 1e-3, 1)
        # droplets that the two sides may give another cell or stencil
        c0 = orc.cells(mesh, q["x"])
        split = (c0 != q["cell"]).any(axis=1)
        assert not (split & ~(face_distance(q["x"], h) < bnd).any(axis=1)).any()
        edge = split | (face_distance(q["x"] - 0.5 * h, h) < bnd).any(axis=1)
        # the first coordinate decides whether a droplet is still there
        at = np.nonzero(live)[0]
        assert np.array_equal(s1["id"][at][~edge] >= 0, np.isfinite(xo[:, 0])[~edge])
        gone += int((s1["id"][at] < 0).sum())
        ok = _finite(xo, uo) & ~edge
        there = {k: v[at][ok] for k, v in s1.items()}
        assert np.array_equal(there["id"], at[ok])
        assert np.array_equal(there["d"], q["d"][ok])
        assert np.abs(min_image(there["x"] - xo[ok], L)).max() <= TOL[form]["pos"] * L.max()
        assert np.abs(there["up"] - uo[ok]).max() <= TOL[form]["vel"] * vmax
        # and no droplet but these adds to the sources
        keep = np.ones(S.shape[1:], dtype=bool)
        for c in s0["cell"][ill]:
            keep[c[2], c[1], c[0]] = False
        for p in np.nonzero(edge)[0]:
            for c in (c0[p], q["cell"][p]):
                keep[c[2], c[1], c[0]] = False
        for comp in range(3):
            fin = keep & np.isfinite(So[comp])
            assert np.isfinite(S[comp][fin]).all()
            err = np.abs(S[comp][fin] - So[comp][fin]).max() / np.abs(So[comp][fin]).max()
            assert err <= TOL[form]["src"], (step, comp, err)
    assert gone > 50, gone
    assert t.stats()["repacks"] >= 3
    t.close()


@pytest.mark.parametrize("form", FORMS)
def test_batch_in_parts_with_bad_droplets(form):
    """A device batch larger than the staging area is partly in the store when
    its bad values are found; in binary32 a diameter can round to zero.  The
    store then holds the others, as if the bad ones had never been there."""
    import torch
    from paper_2603_26691_amd._native import STError
    P, first = 240_000, 5_000
    w = workload("tg32", P=P, noise=0.2)
    x, _, d = w.particles()
    up = np.random.default_rng(4).normal(0.0, 2.0, (P, 3))
    g = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    bad = {10: ("d", -1.0), 11: ("x", np.nan), 70_000: ("up", np.inf), 200_001: ("d", 0.0),
           P - first - 1: ("d", np.nan)}
    tiny = [] if form == "fp64" else [300, 170_000]       # below binary32's least value
    ill = {"x": x[first:].copy(), "up": up[first:].copy(), "d": d[first:].copy()}
    for i, (k, v) in bad.items():
        ill[k][i] = v
    ill["d"][tiny] = 1e-60
    gone = np.zeros(P, dtype=bool)
    gone[[first + i for i in list(bad) + tiny]] = True
    a, b = tracker(w, form), tracker(w, form)
    a.inject(x[:first], up[:first], d[:first])
    a.particles()                                          # places them
    with pytest.raises(STError, match="partially"):
        a.inject(g(ill["x"]), g(ill["up"]), g(ill["d"]))
    b.inject(g(x[~gone]), g(up[~gone]), g(d[~gone]))
    Udev, _ = fields(w, form)
    for t in (a, b):
        t.sources(reset=True)
    for step in range(6):
        sa, sb = state(a), state(b)
        assert np.array_equal(sa["id"], np.where(gone, -1, np.arange(P))[: len(sa["id"])])
        for k in ("x", "up", "d", "cell"):
            assert np.array_equal(sa[k][~gone], sb[k]), (step, k)
        a.step(Udev, 1e-3)
        b.step(Udev, 1e-3)
        Sa, Sb = a.sources(reset=True), b.sources(reset=True)
        # (sums ordered by atomics; stored in binary32 in the FP32-everywhere form)
        tol = 1e-5 if form == "fp32" else 1e-12
        assert float((Sa - Sb).abs().max() / Sb.abs().max()) < tol
    a.close()
    b.close()


@pytest.mark.parametrize("form,tol", [("fp64", 1e-9), ("fp32_local", 1e-4)])
def test_adjoint_of_a_run_that_loses_droplets(form, tol):
    """Taped steps over a field with cells that are not finite: droplets that a
    checkpoint holds are not in later ones.  The gradients of the others' diameters
    are the oracle's, from kept states and (on a tracker whose states are too large to
    keep) from recomputed ones, and these two agree in every entry."""
    import torch
    orc = load_oracle()
    P, nsteps, K, dt = 20_000, 9, 3, 5e-4
    w = workload("tg32", P=P, noise=0.1)
    rng = np.random.default_rng(8)
    x, _, d = w.particles()
    up = rng.normal(0.0, 3.0, (P, 3))
    Udev, Uor = fields(w, form)
    Uor = Uor.copy()
    k, j, i = rng.integers(0, 32, (3, 40))
    Uor[0, k, j, i] = np.nan
    Udev = torch.from_numpy(Uor).to(Udev.dtype).cuda()
    lam = torch.from_numpy(rng.normal(size=Uor.shape)).cuda()
    # about 1 GB a state: two of them are kept
    big = 14_000_000 if form == "fp64" else 26_000_000
    got = []
    for capacity in (P, big):
        t = tracker(w, form, capacity=capacity)
        t.inject(x, up, d)
        s0 = state(t)
        for _ in range(nsteps):
            t.step(Udev, dt, tape=K)
        there = t.particles()["id"].cpu().numpy() >= 0
        assert (~there).sum() > 100
        got.append([v.cpu().numpy() for v in t.backward(lam)])
        after = t.particles()["id"].cpu().numpy() >= 0
        assert np.array_equal(after, there)
        t.close()
    q = {k: v[there] for k, v in s0.items()}
    mesh = oracle_mesh(w)
    Uz = np.where(np.isfinite(Uor), Uor, 0.0)      # (the others never read those cells)
    _, od = orc.adjoint_run(mesh, np.stack([Uz]), [0] * nsteps, [dt] * nsteps, 1, q["x"], q["up"],
                            q["d"], lam.cpu().numpy())
    for dU, dd in got:
        assert np.isfinite(dd[there]).all()
        assert np.linalg.norm(dd[there] - od) <= tol * np.linalg.norm(od)
    for a, b in zip(*got):
        fin = np.isfinite(a)
        assert np.array_equal(fin, np.isfinite(b))
        assert np.linalg.norm(a[fin] - b[fin]) <= 1e-6 * np.linalg.norm(b[fin])
