"""Run calls of few iterations on grids that take one sweep: a call with fewer
than two one-sweep iterations runs the separate sweeps (it would have to copy
its iterate home after one), longer ones sweep, and every way to split a run
into calls gives the same bits."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# iterations of the calls, sweep launches in each
SPLITS = [([1, 1, 1, 1], [0, 0, 0, 0]), ([2, 1, 2, 3], [2, 0, 0, 2]), ([3, 1, 4], [3, 0, 4]), ([5, 5, 2], [5, 4, 2]),
          ([0, 9, 2, 21], [0, 9, 0, 20])]


def _inst(n, seed=92):
    return dotgen.tiny_instance(len(n) - 1, n, seed=seed, floor=0.02)


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
@pytest.mark.parametrize("n", [(31, 150, 150), (700, 1200)])
def test_short_calls(n, prec):
    print(f"[case] short calls {n} precision={prec}", flush=True)
    inst = _inst(n)
    plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)
    w = plan.info.off_w
    a, b = G.GpuState(plan), G.GpuState(plan)
    for calls, sweeps in SPLITS:
        a.reset()
        a.run(sum(calls))
        B.dot_profile_select(plan, B.KERNEL_CLASSES["sweep"])
        b.reset()
        for k, count in zip(calls, sweeps):
            b.run(k)
            assert B.dot_profile_read(plan)[1] == count, (calls, k)
        B.dot_profile_select(plan, -1)
        assert np.array_equal(G.host(a.buf)[:w], G.host(b.buf)[:w]), calls
    plan.close()


def test_short_calls_of_a_batch():
    torch = G.torch_mod()
    batch = B.dot_batch_create([_inst(n, 93 + k) for k, n in enumerate([(40, 120, 150), (31, 130, 140), (60, 90, 70)])],
                               tol=-1.0, max_iter=10 ** 6)
    st = G.stream_handle()
    a = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
    b = torch.zeros_like(a)
    for calls, sweeps in SPLITS:
        B.dot_batch_reset(batch, a.data_ptr(), st)
        B.dot_batch_run(batch, a.data_ptr(), sum(calls), st)
        B.dot_batch_reset(batch, b.data_ptr(), st)
        B.dot_batch_profile_select(batch, B.KERNEL_CLASSES["sweep"])
        for k, count in zip(calls, sweeps):
            B.dot_batch_run(batch, b.data_ptr(), k, st)
            assert B.dot_batch_profile_read(batch)[1] == count, (calls, k)
        B.dot_batch_profile_select(batch, -1)
        for i in range(3):
            (ra, ma), (rb, mb) = (B.dot_batch_extract(batch, s.data_ptr(), i, st) for s in (a, b))
            assert np.array_equal(ra, rb) and all(np.array_equal(x, y) for x, y in zip(ma, mb)), (calls, i)
    batch.close()
