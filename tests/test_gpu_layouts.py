"""GPU: workspaces that hold only the smaller layout of the kernels over
bitmap rows.  The choice belongs to the workspace that is bound, in every
order of binds, through pccl_set_workspace and pccl_synthesize_static;
schedules against the CPU oracle (integers, so equality is exact)."""

import numpy as np
import pytest

from oracle import oracle as O
from paper_2606_07019_amd import workloads as W
from tests.test_gpu_neighbour import _digraph, _generic
from tests.test_zz_no_alloc import _context, _schedule, _status

pytestmark = pytest.mark.gpu

# collectives whose layout over columns is the larger one: 102,400 polled
# entries; a 64-bit mask per limited switch and chunk against a 32-bit count
CASES = {
    "plain": (lambda: _generic("digraph400", _digraph(400, 16, 3), 4200, 20000, 2, 3), "neighbour", "windowed"),
    "switch": (lambda: W.Workload("rail9", W.with_switch_model(W.switch2level(9, 5), 7, 1),
                                  W.a2a_k_bitmaps(45, 5, 9000), 8), "switch columns", "switch rows"),
}


def _smallest(lo, hi, ok):
    """The smallest multiple of 256 in (lo, hi] that passes, hi passing."""
    lo, hi = lo // 256, hi // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if ok(mid * 256) else (mid, hi)
    return hi * 256


@pytest.mark.parametrize("name", sorted(CASES))
def test_the_bound_workspace_picks_the_layout(name):
    import torch
    from paper_2606_07019_amd import pccl as P
    make, columns, rows = CASES[name]
    wl = make()
    print(f"[layouts] {name}: {wl.name}", flush=True)
    ref = O.run_workload(wl)
    assert ref.status == 0, ref.message
    n, stream = len(ref.sends), torch.cuda.current_stream(0).cuda_stream
    h = _context(wl)
    try:
        full = P.pccl_workspace_bytes(h, n)
        ws = torch.empty(full, dtype=torch.uint8, device="cuda:0")

        def bind(size):
            return _status(P.pccl_set_workspace, h, ws.data_ptr(), size, n, stream)

        def check(got, kernel):
            assert got == (n, ref.collective_time)
            np.testing.assert_array_equal(_schedule(h, n), ref.sends)
            assert P.pccl_get_kernel(h)[0] == kernel
            assert P.pccl_workspace_bytes(h, n) == full

        least = _smallest(0, full, lambda b: bind(b) == "OK")
        assert least < full
        for size, kernel in ((full, columns), (least, rows), (full - 256, rows), (full, columns)):
            assert bind(size) == "OK"
            for _ in range(2):
                check(P.pccl_synthesize(h), kernel)
        assert bind(least - 256) == "ENOMEM"
        # the static scratch, with a bound for which only the rows fit, with the exact one, and with the first again
        scratch = P.PCCL_STATIC_SCRATCH_BYTES
        lo, hi = n, scratch // 16
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (lo, mid) if P.pccl_workspace_bytes(h, mid) > scratch else (mid, hi)
        for bound, kernel in ((hi, rows), (n, columns), (hi, rows), (hi, rows)):
            check(P.pccl_synthesize_static(h, bound, stream), kernel)
        assert bind(full) == "OK"
        check(P.pccl_synthesize(h), columns)
    finally:
        P.pccl_destroy(h)
