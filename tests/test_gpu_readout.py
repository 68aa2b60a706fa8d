"""Read-out of the state on the GPU where its routes change: the particles by
way of records in id order against the direct read-out (bit for bit), the
sources in every chunk edge into an output of any alignment, bounding boxes of
partitions whose droplets lie everywhere, and Hilbert placement with 32-bit
and with 64-bit divisions.  Every comparison is exact: these calls move or
round values once, or take minima and maxima.
"""
import ctypes

import numpy as np
import pytest

from gpu_helpers import FORMS, fields, oracle_mesh, tracker, workload  # noqa: F401
from oracle.oracle import load as load_oracle

pytestmark = pytest.mark.gpu

RECORDS_MIN = 1 << 16    # particles from which the read-out takes records


def _moved(P, form, n=(24, 16, 40), edge=8, capacity=None):
    import torch
    w = workload("tg32", n=n, L=(0.075, 0.05, 0.125), P=P, noise=0.3, chunk_edge=edge)
    t = tracker(w, form, capacity=capacity)
    x, up, d = w.particles()
    # in two parts, the second after a step: ids and slots mixed
    t.inject(x[:P // 2], up[:P // 2], d[:P // 2])
    U = torch.from_numpy(w.field()).cuda().to(t.field_dtype)
    t.step(U, 2e-4)
    t.inject(x[P // 2:], up[P // 2:], d[P // 2:])
    for _ in range(6):
        t.step(U, 5e-4)
    return t, w


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("P", [RECORDS_MIN - 1, RECORDS_MIN, RECORDS_MIN + 257])
def test_particles_by_records(form, P):
    import torch
    t, _ = _moved(P, form, capacity=P if P % 2 else P + 1000)
    a = t.particles()
    torch.cuda.synchronize()
    # from another stream than the steps' the read-out is the direct one
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        b = t.particles()
    side.synchronize()
    assert torch.equal(a["id"], torch.arange(P, device="cuda"))
    for k in a:
        assert torch.equal(a[k], b[k]), k
    # again after more steps (a re-bin may have used the records' memory)
    t.inject(*(v[:100].cpu().numpy() for v in (a["x"], a["up"], a["d"]))) if P % 2 == 0 else None
    c = t.particles()
    for k in a:
        assert torch.equal(a[k], c[k][:P]), k
    t.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("edge", [2, 4, 8])
def test_sources_any_alignment(form, edge):
    import torch
    import paper_2603_26691_amd._native as N
    t, w = _moved(3000, form, edge=edge)
    n = int(np.prod(t.field_shape))
    S = t.sources()
    buf = torch.full((n + 1,), float("nan"), dtype=torch.float64, device="cuda")
    for off in (0, 1):
        view = buf[off:off + n]
        N.check(N.lib().st_get_sources(t.ctx, ctypes.c_void_p(view.data_ptr()), off, 1,
                                       ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)),
                t.ctx)
        assert torch.equal(view.reshape(t.field_shape), S), off
    assert float(t.sources().abs().max()) == 0.0    # the second call cleared them
    assert float(S.abs().max()) > 0.0
    t.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("n,edge,P", [((24, 16, 40), 8, 3000), ((40, 16, 16), 4, 20000),
                                      ((6, 10, 36), 2, 2000), ((16, 16, 16), 8, 60000)])
def test_sources_cleared_between_steps(form, n, edge, P):
    """Sources read and cleared after every step (a reset only marks a chunk;
    empty chunks, chunks that droplets enter and leave, and chunks of several
    containers) add up to those left to accumulate, and a read-out without a
    reset changes nothing."""
    import torch
    w = workload("plume256", n=n, L=tuple(0.1 * v / 32 for v in n), P=P, plumes=1, noise=0.3,
                 plume_sigma=0.08, chunk_edge=edge)
    x, up, d = w.particles()
    a, b = tracker(w, form, capacity=2 * P), tracker(w, form, capacity=2 * P)
    U = torch.from_numpy(w.field()).cuda().to(a.field_dtype)
    total = torch.zeros(a.field_shape, dtype=torch.float64, device="cuda")
    size = torch.zeros_like(total)
    for t in (a, b):
        t.inject(x, up, d)
    assert float(a.sources(reset=True).abs().max()) == 0.0
    for k in range(12):
        a.step(U, 1e-3)
        b.step(U, 1e-3)
        if k == 5:     # more containers: half the droplets again, in one chunk
            for t in (a, b):
                t.inject(x[: P // 2] * 0.2, up[: P // 2], d[: P // 2])
        S = a.sources()
        assert torch.equal(a.sources(reset=k % 4 != 3), S)
        if k % 4 != 3:
            assert float(a.sources().abs().max()) == 0.0
            total += S
            size += S.abs()
    total += a.sources(reset=True)
    size += total.abs()
    eps = 2.0 ** -22 if form == "fp32" else 2.0 ** -50
    # sums of the same terms in another order: at most P roundings of the sum
    # of their sizes in one cell, and far fewer in all but the fullest
    assert float((total - b.sources()).abs().max()) <= 64 * eps * float(size.max())
    a.close()
    b.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("per_part", [1, 7, 700, 20001])
def test_boxes_of_scattered_partitions(form, per_part):
    import torch
    P = 20000
    t, _ = _moved(P, form)
    nparts = (P + per_part - 1) // per_part + 2     # the last ones are empty
    box = t.bounding_boxes(0, per_part, nparts).cpu().numpy()
    x = t.particles()["x"].cpu().numpy()
    want = np.empty((nparts, 6))
    for p in range(nparts):
        q = x[p * per_part:(p + 1) * per_part]
        want[p, :3] = q.min(0) if len(q) else np.inf
        want[p, 3:] = q.max(0) if len(q) else -np.inf
    assert np.array_equal(box, want)
    # from another stream than the steps' (the atomic updates), and for an id
    # range that starts and ends inside the droplets
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        again = t.bounding_boxes(0, per_part, nparts)
        part = t.bounding_boxes(per_part // 2, per_part, 3)
    side.synchronize()
    assert np.array_equal(again.cpu().numpy(), want)
    assert torch.equal(part, t.bounding_boxes(per_part // 2, per_part, 3))
    t.close()


def test_boxes_of_more_partitions_than_one_table():
    """Partition counts around one and several LDS tables' worth."""
    import torch
    P = 400000
    t, _ = _moved(P, "fp32_local", n=(40, 40, 40), capacity=6_000_000)
    x = t.particles()["x"]
    for nparts in (3328, 3329, 6657, 13312, 13313):
        per = P // nparts + 1
        at = (torch.arange(P, device="cuda") // per)[:, None].expand(-1, 3)
        inf = float("inf")
        lo = torch.full((nparts, 3), inf, dtype=torch.float64, device="cuda")
        lo = lo.scatter_reduce(0, at, x, "amin")
        hi = torch.full((nparts, 3), -inf, dtype=torch.float64, device="cuda")
        hi = hi.scatter_reduce(0, at, x, "amax")
        assert torch.equal(t.bounding_boxes(0, per, nparts), torch.cat([lo, hi], 1)), nparts
    t.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("P,nparts,edge,tables", [
    (15, 1, 8, False), (16, 1, 8, True), (774, 100, 8, False), (775, 100, 8, True),
    (121, 1, 2, False), (122, 1, 2, True), (5918, 100, 2, False), (5919, 100, 2, True),
    (15_000, 100, 8, True), (131_072, 4000, 8, False), (21_300, 1000, 2, False)])
def test_boxes_where_their_way_changes(form, P, nparts, edge, tables):
    """Particles, particles per box and chunks per workgroup on either side of
    where tables take over from updates in memory."""
    import torch
    t, _ = _moved(P, form, edge=edge, capacity=600_000)
    names = _kernels(lambda: t.bounding_boxes(0, -(-P // nparts), nparts))
    assert ("k_bbox_tables" in names) == tables, names
    x = t.particles()["x"]
    per = -(-P // nparts)
    at = (torch.arange(P, device="cuda") // per)[:, None].expand(-1, 3)
    inf = float("inf")
    lo = torch.full((nparts, 3), inf, dtype=torch.float64, device="cuda")
    hi = torch.full((nparts, 3), -inf, dtype=torch.float64, device="cuda")
    want = torch.cat([lo.scatter_reduce(0, at, x, "amin"), hi.scatter_reduce(0, at, x, "amax")], 1)
    assert torch.equal(t.bounding_boxes(0, per, nparts), want)
    t.close()


# (64-bit divisions from 65536 segments, or where per_seg times a segment's
# voxels reaches 2^32)
@pytest.mark.parametrize("order,nseg,seg_begin,seg_end,per_seg", [
    (6, 65535, 100, 30100, 1), (6, 65536, 65000, 65536, 3), (7, 70001, 0, 5000, 3),
    (7, 1, 0, 1, 2047), (7, 1, 0, 1, 2048), (7, 3, 1, 3, 700), (1, 8, 0, 8, 129)])
def test_hilbert_division_widths(order, nseg, seg_begin, seg_end, per_seg):
    import torch
    orc = load_oracle()
    w = workload("tg32", n=(16, 16, 16), L=(0.1, 0.06, 0.05), P=16)
    t = tracker(w, "fp64")
    n = (seg_end - seg_begin) * per_seg
    u = np.random.default_rng(order + nseg).random((n, 3))
    got = t.hilbert_positions(order, nseg, seg_begin, seg_end, per_seg,
                              torch.from_numpy(u).cuda()).cpu().numpy()
    assert np.array_equal(got, orc.hilbert_positions(order, nseg, seg_begin, seg_end, per_seg,
                                                     w.L, u))
    t.close()


def test_hilbert_large_per_segment():
    """per_seg (v1 - v0) beyond 2^32: the same particles as placed with the
    narrow divisions where both apply (particle k of per_seg lies in voxel
    floor(k nv / per_seg), so every 4th of 4 per_seg is particle k of per_seg)."""
    import torch
    w = workload("tg32", n=(16, 16, 16), L=(0.1, 0.06, 0.05), P=16)
    t = tracker(w, "fp64")
    order, nseg, per = 6, 8, 40000          # nv = 32768: 40000 x 32768 < 2^32 <= 160000 x 32768
    u = torch.zeros((per, 3), dtype=torch.float64, device="cuda")
    a = t.hilbert_positions(order, nseg, 3, 4, per, u)
    v = torch.zeros((4 * per, 3), dtype=torch.float64, device="cuda")
    b = t.hilbert_positions(order, nseg, 3, 4, 4 * per, v)
    assert torch.equal(a, b[::4])
    t.close()


@pytest.mark.parametrize("form", FORMS)
@pytest.mark.parametrize("P", [65_535, 65_536, 163_839, 163_840])
def test_read_out_where_its_way_changes(form, P):
    """The two ways of the read-out give the same droplets as another stream's,
    which is always direct."""
    import torch
    t, _ = _moved(P, form)
    names = _kernels(lambda: t.particles())
    assert ("k_records_out" in names) == (P >= 65_536), names
    mine = t.particles()
    torch.cuda.synchronize()
    with torch.cuda.stream(torch.cuda.Stream()):
        other = t.particles()
    torch.cuda.synchronize()
    assert torch.equal(mine["id"], torch.arange(P, device="cuda"))
    for k in mine:
        assert torch.equal(mine[k], other[k]), k
    t.close()


def _kernels(call):
    """Names of the kernels that run during call()."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CUDA]) as p:
        call()
        torch.cuda.synchronize()
    return " ".join(e.name for e in p.events())


def test_read_out_beside_captures():
    """Steps and read-outs captured in graphs leave the way of other read-outs
    alone; a captured read-out takes the fast way (through the second store) where its
    own capture stepped first, and only there."""
    import torch
    P = 200_000
    w = workload("tg32", P=P, noise=0.3)
    a, b = tracker(w, "fp32_local"), tracker(w, "fp32_local")
    U = fields(w, "fp32_local")[0]
    for t in (a, b):
        t.inject(*w.particles())
        t.step(U, 1e-3)
    fast = ("k_records_out", "k_bbox_tables")
    got = {}

    def read(t):
        got["s"] = t.particles()
        got["box"] = t.bounding_boxes(0, 1000, 100)

    names = _kernels(lambda: read(a))
    assert all(k in names for k in fast), names
    torch.cuda.synchronize()
    step, both, only = (torch.cuda.CUDAGraph() for _ in range(3))
    with torch.cuda.graph(step):
        a.step(U, 1e-3)
    with torch.cuda.graph(both):
        a.step(U, 1e-3)
        read(a)
    in_both = got.copy()
    with torch.cuda.graph(only):
        read(a)
    in_only = got.copy()
    torch.cuda.synchronize()

    def same(out):
        want = {}
        want["s"], want["box"] = b.particles(), b.bounding_boxes(0, 1000, 100)
        for k in want["s"]:
            assert torch.equal(out["s"][k], want["s"][k]), k
        assert torch.equal(out["box"], want["box"])

    for k in range(3):
        step.replay()
        b.step(U, 1e-3)
        names = _kernels(lambda: read(a))
        assert all(n in names for n in fast), names
        same(got)
        names = _kernels(both.replay)
        b.step(U, 1e-3)
        assert all(n in names for n in fast), names
        same(in_both)
        names = _kernels(only.replay)
        assert not any(n in names for n in fast) and "k_get_particles" in names, names
        same(in_only)
    a.close()
    b.close()
