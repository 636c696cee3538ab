"""A batch that is refused for its problems leaves the HIP error of the calls
before it as it was, with and without a GPU."""
import ctypes
import threading

import pytest

import paper_1502_02389_amd as L
from paper_1502_02389_amd import lift as B


@pytest.mark.parametrize("storage", [L.LIFT_F32, L.LIFT_BF16])
@pytest.mark.parametrize("knobs", [None, B.knobs()])
def test_refused_batches_report_no_hip_error(storage, knobs):
    got = []

    def refused():     # a thread of its own: the error is kept per thread
        p = (L.lift_problem * 1)()
        p[0].kind, p[0].n, p[0].a, p[0].out = L.LIFT_KIND_ASUM, -1, 1 << 20, 1 << 21
        h = ctypes.c_void_p()
        got.append(L.lift_batch_create(p, 1, storage, L.ACC["f32"], L.LIFT_F32, knobs, h))
        got.append(L.lift_last_hip_error())

    t = threading.Thread(target=refused)
    t.start()
    t.join()
    assert got == [L.LIFT_EINVAL, 0]
