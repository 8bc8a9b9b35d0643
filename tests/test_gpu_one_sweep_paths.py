"""The one-sweep iteration on the paths that the other files do not reach, each
against the separate sweeps and bitwise: beside the chunked elimination of long
lines (its checkpoints then lie in a buffer of their own), alone and in a batch
whose members follow each other in that buffer; with boxes of few and of many
waves; at other check cadences, without graphs, after a time limit, entered in
the middle of a captured run; and promoted or exported after an odd count."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

PRECS = [B.DOT_FP64, B.DOT_MIXED]


def _inst(n, seed=94, masked=False):
    return dotgen.tiny_instance(len(n) - 1, n, seed=seed, floor=0.01, masked=masked)


def _plan(inst, prec, **kw):
    kw = {"tol": -1.0, "max_iter": 10 ** 6, **kw}
    return B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, **kw)


def _select(plan, name):
    B.dot_profile_select(plan, B.KERNEL_CLASSES[name] if name else -1)


def _sweeps(plan, s):
    """Sweep launches of two iterations of a plan."""
    _select(plan, "sweep")
    s.reset()
    s.run(2)
    n = B.dot_profile_read(plan)[1]
    _select(plan, None)
    s.reset()
    return n


def _separate(plan, its):
    s = G.GpuState(plan)
    s.reset()
    _select(plan, "cone")
    r = s.run(its)
    _select(plan, None)
    return r, s


def _iterate(s):
    return s.buf[:s.plan.info.off_w]


def _same(a, b):
    return G.torch_mod().equal(_iterate(a), _iterate(b))


# the last: too many lines for the whole-line elimination
LONG = [(70, 1, 3999), (400, 1400), (20, 380, 600)]


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n", LONG, ids=["x".join(map(str, n)) for n in LONG])
def test_chunked_elimination(n, prec):
    print(f"[case] chunked {n} precision={prec}", flush=True)
    plan = _plan(_inst(n), prec)
    s = B.dot_plan_get_schedule(plan)
    B.dot_plan_set_schedule(plan, s["cw"], s["waves"])  # written out: the chunked elimination
    a = G.GpuState(plan)
    assert _sweeps(plan, a) == 2
    for k in (7, 13, 55):
        ra = a.run(k)
    rb, b = _separate(plan, 75)
    assert (ra.iters, ra.eta_dot, ra.sigma) == (rb.iters, rb.eta_dot, rb.sigma) and np.isfinite(ra.eta_dot)
    assert _same(a, b)
    plan.close()


@pytest.mark.parametrize("prec", PRECS)
def test_chunked_elimination_in_a_batch(prec):
    torch = G.torch_mod()
    insts = [_inst(n, 95 + i) for i, n in enumerate([(70, 1, 3999), (12, 90, 1000), (9, 30, 50), (30, 40, 800)])]
    batch = B.dot_batch_create(insts, tol=-1.0, max_iter=10 ** 6, precision=prec)
    s = B.dot_batch_get_schedule(batch)
    B.dot_batch_set_schedule(batch, s["cw"], s["waves"])
    ws = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
    st = G.stream_handle()
    B.dot_batch_reset(batch, ws.data_ptr(), st)
    B.dot_batch_profile_select(batch, B.KERNEL_CLASSES["sweep"])
    B.dot_batch_run(batch, ws.data_ptr(), 2, st)
    assert B.dot_batch_profile_read(batch)[1] == 2
    B.dot_batch_profile_select(batch, -1)
    B.dot_batch_run(batch, ws.data_ptr(), 5, st)
    res = B.dot_batch_run(batch, ws.data_ptr(), 50, st)
    for i, inst in enumerate(insts):
        print(f"[case] member {i} {inst.n}", flush=True)
        plan = _plan(inst, prec)
        r, b = _separate(plan, 57)
        assert (res[i].iters, res[i].eta_dot, res[i].objective) == (r.iters, r.eta_dot, r.objective)
        (ra, ma), (rb, mb) = B.dot_batch_extract(batch, ws.data_ptr(), i, st), b.extract()
        assert np.array_equal(ra, rb) and all(np.array_equal(x, y) for x, y in zip(ma, mb))
        plan.close()
    batch.close()


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("n", [(36, 120, 120), (28, 152, 124), (250, 75, 35), (162, 4000)])
def test_boxes_by_precision(n, prec):
    print(f"[case] boxes {n} precision={prec}", flush=True)
    plan = _plan(_inst(n, masked=len(n) > 2), prec)
    a = G.GpuState(plan)
    assert _sweeps(plan, a) == 2
    ra = a.run(55)
    rb, b = _separate(plan, 55)
    assert ra.eta_dot == rb.eta_dot and np.isfinite(ra.eta_dot) and _same(a, b)
    plan.close()


BIG = (31, 150, 150)


@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("every", [1, 3, 4])
def test_other_cadences(every, prec):
    print(f"[case] cadence {every} precision={prec}", flush=True)
    plan = _plan(_inst(BIG), prec, check_every=every)
    a = G.GpuState(plan)
    assert _sweeps(plan, a) == 2
    for k in (3, 2, 20):
        ra = a.run(k)
    rb, b = _separate(plan, 25)
    assert (ra.checks, ra.eta_dot, ra.sigma) == (rb.checks, rb.eta_dot, rb.sigma) and _same(a, b)
    plan.close()


@pytest.mark.parametrize("prec", PRECS)
def test_without_graphs_and_into_captured_runs(prec):
    plan = _plan(_inst(BIG), prec)
    a = G.GpuState(plan)
    assert _sweeps(plan, a) == 2
    B.dot_plan_set_graphs(plan, False)
    a.run(95)
    B.dot_plan_set_graphs(plan, True)
    a.run(2)
    a.run(63)  # from an odd count, after a call that swept nothing
    _, b = _separate(plan, 160)
    assert _same(a, b)
    # separate sweeps first, so that the first sweep of the plan is a captured one
    c = G.GpuState(plan)
    c.reset()
    _select(plan, "cone")
    c.run(10)
    _select(plan, None)
    c.run(150)
    assert _same(c, b)
    plan.close()


@pytest.mark.parametrize("prec", PRECS)
def test_after_a_time_limit(prec):
    """A budget that the first poll exceeds ends the call there, at an even
    count and resumable."""
    inst = _inst(BIG)
    plan = _plan(inst, prec, time_limit_s=1e-9)
    free = _plan(inst, prec)
    for start, at in ((0, 40), (3, 50)):  # the second: 7 iterations to a multiple of 10, then blocks of 10
        a = G.GpuState(plan)
        assert _sweeps(free, G.GpuState(free)) == 2
        a.reset()
        if start:
            a.run(start)
        r = a.run(1000)
        assert B.TERM_NAMES[r.term] == "timeout" and r.iters == at
        _, b = _separate(free, at)
        assert _same(a, b)
    plan.close()
    free.close()


def test_promoted_and_exported_after_an_odd_count():
    inst = _inst(BIG)
    st = G.stream_handle()
    plan, full = _plan(inst, B.DOT_MIXED), _plan(inst, B.DOT_FP64)
    a = G.GpuState(plan)
    assert _sweeps(plan, a) == 2
    a.run(35)
    _, b = _separate(plan, 35)
    for x, y in zip(B.dot_state_export(plan, a.ptr, st), B.dot_state_export(plan, b.ptr, st)):
        assert np.array_equal(x, y)
    f, g = G.GpuState(full), G.GpuState(full)
    B.dot_state_promote(plan, a.ptr, full, f.ptr, st)
    B.dot_state_promote(plan, b.ptr, full, g.ptr, st)
    rf = f.run(22)
    _select(full, "cone")
    rg = g.run(22)
    _select(full, None)
    assert rf.iters == rg.iters == 57 and rf.eta_dot == rg.eta_dot and _same(f, g)
    plan.close()
    full.close()
