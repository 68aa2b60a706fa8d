"""Device memory that closed trackers leave for new ones, on the GPU: a tracker
on kept memory gives what one on fresh memory gives, from several threads and
streams, and what is kept is bounded."""
import threading

import numpy as np
import pytest

from gpu_helpers import fields, state, tracker, workload

pytestmark = pytest.mark.gpu

KEEP = 512 << 20     # bytes kept at most


def _run(w, form, U):
    """State, sources and gradients of a short taped run on a new tracker."""
    x, up, d = w.particles()
    t = tracker(w, form)
    t.inject(x, up, d)
    t.sources(reset=True)
    for _ in range(5):
        t.step(U, 5e-4, tape=2)
    S = t.sources()
    dU, dd = t.backward(S)
    s = state(t)
    out = [s[k] for k in ("x", "up", "cell")] + [v.cpu().numpy() for v in (S, dU, dd)]
    t.close()
    return out


@pytest.mark.parametrize("form", ["fp64", "fp32_local"])
def test_trackers_on_kept_memory(form):
    import torch
    cases = [workload("tg32", P=P, n=n, noise=0.2, seed=k)
             for k, (P, n) in enumerate([(20000, (32, 32, 32)), (3000, (16, 16, 16)),
                                         (21000, (32, 32, 32)), (60000, (40, 24, 16))])]
    Us = [fields(w, form)[0] for w in cases]
    first = [_run(w, form, U) for w, U in zip(cases, Us)]
    errors = []

    def work(k):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for j in range(6):
                    i = (k + j) % len(cases)
                    got = _run(cases[i], form, Us[i])
                    for n, (a, b) in enumerate(zip(got[:3], first[i][:3])):
                        assert np.array_equal(a, b), (i, n)
                    for a, b in zip(got[3:], first[i][3:]):   # sums ordered by atomics
                        assert np.linalg.norm(a - b) <= 1e-6 * np.linalg.norm(b), i
        except BaseException as e:  # noqa: BLE001 (shown below, in the test's own thread)
            errors.append(e)

    threads = [threading.Thread(target=work, args=(k,)) for k in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors


def test_kept_memory_is_bounded():
    import torch
    w = workload("tg32", P=1, n=(16, 16, 16))
    torch.cuda.synchronize()
    free0 = torch.cuda.mem_get_info()[0]
    for capacity in [10_000, 3_000_000, 500_000, 8_000_000, 1_000_000, 20_000_000, 2_000_000]:
        tracker(w, "fp32_local", capacity=capacity).close()
    free1 = torch.cuda.mem_get_info()[0]
    assert free0 - free1 <= KEEP + (64 << 20), (free0, free1)
