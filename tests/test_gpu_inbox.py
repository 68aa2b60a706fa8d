"""Droplets in flight between containers on the GPU, against the FP64 oracle
step by step, where their route changes: more movers than a workgroup's LDS
stage, more arrivals than its LDS pool, more than an inbox or the free slots
hold (a full re-bin then takes the droplets that stayed in place), a chunk
that is its own neighbour along a periodic axis, and chunks of several
containers.  Tolerances as in the lockstep parity tests.
"""
import numpy as np
import pytest

from gpu_helpers import FORMS, band, fields, lockstep_check, oracle_mesh, state, tracker, workload
from oracle.oracle import load as load_oracle

pytestmark = pytest.mark.gpu

TOL = {
    "fp64": {"pos": 1e-13, "vel": 1e-12, "src": 1e-10},
    "fp32_local": {"pos": 1e-5, "vel": 1e-5, "src": 1e-6},
    "fp32": {"pos": 1e-5, "vel": 1e-5, "src": 1e-4},
}
WHOLE = 1 << 17      # slots up to which inboxes hold whole rooms


@pytest.fixture(scope="module")
def orc():
    return load_oracle()


def _lockstep(orc, w, form, x, up, d, dt, steps, capacity=None):
    t = tracker(w, form, capacity=capacity)
    t.inject(x, up, d)
    Udev, Uor = fields(w, form)
    vmax = max(1.0, float(np.abs(up).max()))
    tol = dict(TOL[form], vel=TOL[form]["vel"] * vmax)
    bnd = band(form, w.n)
    if form == "fp32":   # the binary32 rounding of the largest position
        bnd = max(bnd, 2.0 ** -21 * (max(w.L) + vmax * dt) / min(w.h))
    print(form, lockstep_check(t, orc, oracle_mesh(w), Udev, Uor, dt, steps, tol, band_=bnd))
    s = state(t)
    assert np.array_equal(s["id"], np.arange(len(d)))
    st = t.stats()
    print(st)
    return t, st


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n,share", [((32, 32, 32), 0.05), ((32, 32, 32), 0.25),
                                     ((32, 32, 32), 1.0), ((8, 8, 64), 1.0)])
def test_many_movers(orc, form, n, share):
    """A share of the droplets cross one chunk face at once.  0.05 passes the
    LDS stage and pool of a workgroup but fits the inboxes, 0.25 does not fit
    them, and nor does the whole store, which in the 8 x 8 x 64 mesh (one
    chunk across) mostly lands in the chunk it left."""
    P = 150_000
    w = workload("tg32", n=n, L=tuple(0.1 * v / 32 for v in n), P=P, noise=0.1)
    x, _, d = w.particles()
    d = np.full(P, 60e-6)           # a response time of 11 ms: they keep their velocity
    rng = np.random.default_rng(3)
    up = np.zeros((P, 3))
    fast = rng.random(P) < share
    up[fast, 0] = 25.0              # one chunk (0.025 m) per step of 1 ms
    t, st = _lockstep(orc, w, form, x, up, d, 1e-3, 4)
    assert st["slots"] > WHOLE      # inboxes of an eighth of the rooms
    assert st["movers"] > 0.5 * share * P * (0 if n[0] == 8 and form == "fp32" else 1)
    if share >= 0.25:
        assert st["repacks"] >= 2 or (n[0] == 8 and form == "fp32")
    t.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("P", [33_000, 100_000])
def test_several_containers_per_chunk(orc, form, P):
    """8 chunks of 2 and of 6 to 7 containers with heavy traffic between them
    (some of it from corner to corner)."""
    w = workload("tg32", n=(16, 16, 16), L=(0.05, 0.05, 0.05), P=P, noise=0.3)
    rng = np.random.default_rng(P)
    x = rng.random((P, 3)) * np.array(w.L)
    x[: P // 2] *= 0.499            # half of them in one chunk
    up = rng.normal(0.0, 1.0, (P, 3))
    d = np.exp(rng.normal(np.log(30e-6), 0.3, P))
    t, st = _lockstep(orc, w, form, x, up, d, 1e-3, 5, capacity=2 * P)
    assert st["movers"] > P // 100
    t.close()


@pytest.mark.parametrize("form", ["fp64", "fp32_local"])
def test_rejected_injection_leaves_no_trace(form):
    """A device injection with a bad value leaves the counts that the next
    full re-bin sorts by as they were."""
    import torch
    from paper_2603_26691_amd._native import STError
    w = workload("tg32", n=(16, 16, 16), P=3000)
    x, up, d = w.particles()
    t = tracker(w, form, capacity=10000)
    g = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    t.inject(g(x[:1000]), g(up[:1000]), g(d[:1000]))
    bad = d[1000:2000].copy()
    bad[500] = -1.0
    with pytest.raises(STError):
        t.inject(g(x[1000:2000]), g(up[1000:2000]), g(bad))
    t.inject(g(x[1000:]), g(up[1000:]), g(d[1000:]))
    assert t.count() == 3000
    s = state(t)
    assert np.array_equal(s["id"], np.arange(3000))
    ref = tracker(w, form)
    ref.inject(x, up, d)
    r = state(ref)
    for k in s:
        assert np.array_equal(s[k], r[k]), k
    t.close()
    ref.close()


def test_captured_step_replays():
    """A captured step holds no state of the host: replayed, with reads of the
    state between the replays, it steps as eager calls do."""
    import torch
    w = workload("tg32", P=20000, noise=0.3)
    x, up, d = w.particles()
    a, b = tracker(w, "fp64"), tracker(w, "fp64")
    U = fields(w, "fp64")[0]
    for t in (a, b):
        t.inject(x, up, d)
        t.step(U, 1e-3)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.step(U, 1e-3)
    torch.cuda.synchronize()
    for k in range(7):
        graph.replay()
        b.step(U, 1e-3)
        torch.cuda.synchronize()
        if k % 3 == 1:
            sa, sb = state(a), state(b)
            for key in sa:
                assert np.array_equal(sa[key], sb[key]), (k, key)
    Sa, Sb = a.sources(), b.sources()
    assert float((Sa - Sb).norm() / Sb.norm()) < 1e-12   # (sums ordered by atomics)
    assert a.stats()["movers"] == b.stats()["movers"] > 0
    a.close()
    b.close()


@pytest.mark.parametrize("form", FORMS)
def test_captured_step_replays_after_more_droplets(form):
    """A step captured with a quarter of the droplets in the store is replayed
    with all of them, through full re-bins: their layout is made for what the
    store holds by then."""
    import torch
    P, P0 = 24_000, 6_000
    w = workload("tg32", P=P, noise=0.3)
    x, _, d = w.particles()
    d = np.full(P, 60e-6)
    up = np.random.default_rng(5).normal(0.0, 6.0, (P, 3))
    a, b = tracker(w, form), tracker(w, form)
    U = fields(w, form)[0]
    for t in (a, b):
        t.inject(x[:P0], up[:P0], d[:P0])
        t.step(U, 1e-3)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.step(U, 1e-3)
    torch.cuda.synchronize()
    for t in (a, b):
        t.inject(x[P0:], up[P0:], d[P0:])
        t.particles()                     # places them
    before = a.stats()["repacks"]
    for k in range(24):
        graph.replay()
        b.step(U, 1e-3)
        torch.cuda.synchronize()
        if k % 4 == 3:
            sa, sb = state(a), state(b)
            assert np.array_equal(sa["id"], np.arange(P))
            for key in sa:
                assert np.array_equal(sa[key], sb[key]), (k, key)
    Sa, Sb = a.sources(), b.sources()
    tol = 1e-5 if form == "fp32" else 1e-12      # (sums ordered by atomics)
    assert float((Sa - Sb).norm() / Sb.norm()) < tol
    assert a.stats()["repacks"] == b.stats()["repacks"] > before
    a.close()
    b.close()


@pytest.mark.parametrize("form", FORMS)
def test_captured_step_replays_beside_staged_droplets(form):
    """Droplets that are staged while a captured step is replayed change
    nothing of what the replays do, and are placed by the next call that
    needs them; a rejected batch leaves no trace either."""
    import torch
    from paper_2603_26691_amd._native import STError
    P, P0 = 24_000, 10_000
    w = workload("tg32", P=P, noise=0.3)
    x, _, d = w.particles()
    d = np.full(P, 60e-6)
    up = np.random.default_rng(6).normal(0.0, 6.0, (P, 3))
    g = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    a, b = tracker(w, form), tracker(w, form)
    U = fields(w, form)[0]
    for t in (a, b):
        t.inject(x[:P0], up[:P0], d[:P0])
        t.step(U, 1e-3)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.step(U, 1e-3)
    torch.cuda.synchronize()
    bad = d[:100].copy()
    bad[7] = -1.0
    cuts = [P0, P0 + 3000, P0 + 3100, P]
    for p, q in zip(cuts, cuts[1:]):
        a.inject(g(x[p:q]), g(up[p:q]), g(d[p:q]))         # staged
        with pytest.raises(STError):
            a.inject(g(x[:100]), g(up[:100]), g(bad))
        for _ in range(6):
            graph.replay()
            b.step(U, 1e-3)
        torch.cuda.synchronize()
        Sa, Sb = a.sources(reset=True), b.sources(reset=True)
        tol = 1e-5 if form == "fp32" else 1e-12            # (sums ordered by atomics)
        assert float((Sa - Sb).norm() / Sb.norm()) < tol
        assert a.stats()["movers"] == b.stats()["movers"] > 0
        b.inject(x[p:q], up[p:q], d[p:q])
        sa, sb = state(a), state(b)                        # places them
        assert np.array_equal(sa["id"], np.arange(q))
        for key in sa:
            assert np.array_equal(sa[key], sb[key]), (q, key)
    a.close()
    b.close()


@pytest.mark.parametrize("form", FORMS)
def test_injection_beside_a_read_out_on_another_stream(form):
    """Boxes and particles that another stream is still to read are those of the
    store, not of droplets injected meanwhile."""
    import torch
    P, P0 = 100_000, 70_000
    w = workload("tg32", P=P, noise=0.3)
    x, _, d = w.particles()
    d = np.full(P, 60e-6)
    up = np.random.default_rng(7).normal(0.0, 6.0, (P, 3))
    g = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    t = tracker(w, form)
    U = fields(w, form)[0]
    late = (g(x[P0:]), g(up[P0:]), g(d[P0:]))
    t.inject(x[:P0], up[:P0], d[:P0])
    for _ in range(3):
        t.step(U, 1e-3)                                    # arrivals wait in the inboxes
    want, box = state(t), t.bounding_boxes(0, 1000, 200).cpu().numpy()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        torch.cuda._sleep(400_000_000)                     # some 0.2 s
        late_box = t.bounding_boxes(0, 1000, 200)
        late_state = t.particles()
    t.inject(*late)
    waiting = not side.query()
    side.synchronize()
    assert waiting, "the injection was to end before the read-out began"
    assert np.array_equal(late_box.cpu().numpy(), box)
    for k in want:
        assert np.array_equal(late_state[k].cpu().numpy(), want[k]), k
    s = state(t)
    assert np.array_equal(s["id"], np.arange(P))
    assert np.array_equal(s["x"][:P0], want["x"])
    t.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("P", [1000, 200_000])
def test_first_load_in_parts(form, P):
    """A first load in several injections (host and device arrays), staged in
    the empty store, is the one in a single injection; so is one that follows
    a flush, staged in the inboxes' memory over several re-bins."""
    import torch
    w = workload("tg32", n=(32, 16, 24), L=(0.1, 0.05, 0.075), P=P, noise=0.1)
    x, up, d = w.particles()
    up = np.random.default_rng(2).normal(0.0, 0.3, up.shape)
    g = lambda a: torch.from_numpy(a).cuda()  # noqa: E731
    whole = tracker(w, form)
    whole.inject(x, up, d)
    want = state(whole)
    for cuts, read in [([0, P // 3, P // 2, P], False), ([0, 10, P], True)]:
        t = tracker(w, form)
        for k, (a, b) in enumerate(zip(cuts, cuts[1:])):
            part = (x[a:b], up[a:b], d[a:b])
            t.inject(*(part if k % 2 else (g(v) for v in part)))
            if read:
                t.particles()      # places what is staged
        got = state(t)
        for key in want:
            assert np.array_equal(got[key], want[key]), (cuts, key)
        t.close()
    whole.close()
