"""Device memory that only speed depends on: pivots of long lines held for what
runs and no longer, and every path without the pivots or the one-sweep buffer."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

LINES = (24, 100, 900)  # 2525 lines of 901 nodes: 18 MB of pivots
PIVOTS = 25 * 101 * 901 * 8


def _inst(n, seed=111):
    return dotgen.tiny_instance(len(n) - 1, n, seed=seed, floor=0.02)


def _plan(inst, **kw):
    kw = {"tol": -1.0, "max_iter": 10 ** 6, **kw}
    return B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, **kw)


def _used():
    torch = G.torch_mod()
    torch.cuda.synchronize()
    free, total = torch.cuda.mem_get_info()
    return total - free


def _solve(inst, its, **kw):
    plan = _plan(inst, **kw)
    s = G.GpuState(plan)
    s.reset()
    r = s.run(its)
    rho, m = s.extract()
    plan.close()
    return r, rho, m


def test_requests_hold_pivots_while_they_run():
    inst = _inst(LINES)
    kw = dict(tol=-1.0, max_iter=80)
    one = B.dot_footprint_bytes(2, LINES, B.DOT_FP64)
    ctx = B.dot_ctx_create(2, B.DOT_FP64, 2 * one + (1 << 20), 2)
    st = G.stream_handle()
    B.dot_ctx_submit(ctx, _inst((6, 9, 700)), **kw)  # first use of the kernels
    while sum(B.dot_ctx_step(ctx, 40, st)):
        pass
    base = _used()
    tickets = [B.dot_ctx_submit(ctx, inst, **kw) for _ in range(6)]
    queued = _used() - base
    assert queued < 6 * PIVOTS // 2, queued
    most = 0
    while sum(B.dot_ctx_step(ctx, 20, st)):
        most = max(most, _used() - base)
    assert most < queued + 3 * PIVOTS, (queued, most)
    r, rho, m = _solve(inst, 80)
    for t in tickets:
        rc, rhoc, mc = B.dot_ctx_fetch(ctx, t)
        assert (rc.iters, rc.eta_dot, rc.objective) == (r.iters, r.eta_dot, r.objective)
        assert np.array_equal(rho, rhoc) and all(np.array_equal(x, y) for x, y in zip(m, mc))
    ctx.close()


def test_batch_of_too_many_lines_holds_no_pivots():
    torch = G.torch_mod()
    st = G.stream_handle()
    insts = [_inst(LINES, 112 + k) for k in range(4)]
    warm = B.dot_batch_create([_inst((6, 9, 700))] * 2, tol=-1.0, max_iter=10)
    base = _used()
    # together the lines take the chunked solve; the last two alone do not
    tols = [1e3, 1e3, -1.0, 1e3]
    batch = B.dot_batch_create(insts, per_instance=[dict(tol=t) for t in tols], max_iter=10 ** 6)
    assert _used() - base < 4 * PIVOTS // 2
    ws = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
    B.dot_batch_reset(batch, ws.data_ptr(), st)
    res = B.dot_batch_run(batch, ws.data_ptr(), 90, st)
    assert [r.iters for r in res] == [5, 5, 90, 5] and B.dot_batch_laid_out(batch) == 1
    for i in (1, 2):
        r, rho, m = _solve(insts[i], 90, tol=tols[i])
        rb, mb = B.dot_batch_extract(batch, ws.data_ptr(), i, st)
        assert (res[i].iters, res[i].eta_dot) == (r.iters, r.eta_dot)
        assert np.array_equal(rho, rb) and all(np.array_equal(x, y) for x, y in zip(m, mb))
    B.dot_batch_reset(batch, ws.data_ptr(), st)  # all members again, then another layout
    res = B.dot_batch_run(batch, ws.data_ptr(), 90, st)
    assert [r.iters for r in res] == [5, 5, 90, 5]
    batch.close()
    warm.close()


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
@pytest.mark.parametrize("n", [(31, 150, 150), (9, 30, 700), LINES])
def test_without_scratch_memory(n, prec):
    """One sweep, whole lines, and both: the same bits without them, and the
    sweep back in the first call that gets its memory."""
    print(f"[case] no scratch {n} precision={prec}", flush=True)
    inst = _inst(n)
    r, rho, m = _solve(inst, 75, precision=prec)
    big = int(np.prod([k + 1 for k in n])) > 1 << 19
    B.dot_test_fail_scratch(1 << 20)
    try:
        plan = _plan(inst, precision=prec)
        s = G.GpuState(plan)
        s.reset()
        B.dot_profile_select(plan, B.KERNEL_CLASSES["sweep"])
        s.run(15)
        assert B.dot_profile_read(plan)[1] == 0
        B.dot_test_fail_scratch(0)
        s.run(5)  # from an odd count: the first iteration is a separate one
        assert B.dot_profile_read(plan)[1] == (4 if big else 0)
        B.dot_profile_select(plan, -1)
        r2 = s.run(55)
    finally:
        B.dot_test_fail_scratch(0)
    rho2, m2 = s.extract()
    assert (r2.iters, r2.eta_dot, r2.objective) == (r.iters, r.eta_dot, r.objective)
    assert np.array_equal(rho, rho2) and all(np.array_equal(x, y) for x, y in zip(m, m2))
    plan.close()


def test_batch_and_requests_without_scratch_memory():
    torch = G.torch_mod()
    st = G.stream_handle()
    insts = [_inst(n, 120 + k) for k, n in enumerate([(31, 150, 150), (9, 30, 700), LINES])]
    alone = [_solve(i, 80) for i in insts]
    for fail in (1 << 20, 1):  # all of them, or only the first
        B.dot_test_fail_scratch(fail)
        try:
            batch = B.dot_batch_create(insts, tol=-1.0, max_iter=10 ** 6)
            ws = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
            B.dot_batch_reset(batch, ws.data_ptr(), st)
            res = B.dot_batch_run(batch, ws.data_ptr(), 80, st)
            B.dot_test_fail_scratch(fail)
            ctx = B.dot_ctx_create(2, B.DOT_FP64, sum(B.dot_footprint_bytes(2, i.n, B.DOT_FP64) + 256 for i in insts), 3)
            tickets = [B.dot_ctx_submit(ctx, i, tol=-1.0, max_iter=80) for i in insts]
            while sum(B.dot_ctx_step(ctx, 40, st)):
                pass
        finally:
            B.dot_test_fail_scratch(0)
        for k, (r, rho, m) in enumerate(alone):
            rb, mb = B.dot_batch_extract(batch, ws.data_ptr(), k, st)
            rc, rhoc, mc = B.dot_ctx_fetch(ctx, tickets[k])
            for got, rr, mm in ((res[k], rb, mb), (rc, rhoc, mc)):
                assert (got.iters, got.eta_dot, got.objective) == (r.iters, r.eta_dot, r.objective), (fail, k)
                assert np.array_equal(rho, rr) and all(np.array_equal(x, y) for x, y in zip(m, mm)), (fail, k)
        batch.close()
        ctx.close()
    with pytest.raises(B.DotError):
        B.dot_test_fail_scratch(-1)
