"""The one-lane elimination of few long lines with the plan's pivots
(tri_line_body), against the chunked one (a schedule written out selects it):
bitwise the same iterates, at line lengths around its blocks of 16 nodes, line
counts around its workgroups, on the longest lines and in a batch with shorter
ones."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRIDS = [(1, 576), (3, 591), (64, 1000), (2, 4096), (5, 60, 606), (27, 17, 577), (11, 100, 700), (2, 3, 4, 640)]


def _solve(plan, its, chunked):
    if chunked:
        s = B.dot_plan_get_schedule(plan)
        B.dot_plan_set_schedule(plan, s["cw"], s["waves"])
    s = G.GpuState(plan)
    s.reset()
    r = s.run(its)
    h, i = G.host(s.buf), plan.info
    return r, np.concatenate([h[i.off_phi:i.off_scratch], h[i.off_q:i.off_w]])


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
@pytest.mark.parametrize("n", GRIDS, ids=["x".join(map(str, n)) for n in GRIDS])
def test_long_lines_give_the_chunked_bits(n, prec):
    print(f"[case] long lines {n} precision={prec}", flush=True)
    inst = dotgen.tiny_instance(len(n) - 1, n, seed=23, floor=0.0, masked=len(n) > 2)
    plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)
    ra, a = _solve(plan, 57, False)
    rb, b = _solve(plan, 57, True)
    assert ra.iters == rb.iters == 57 and ra.eta_dot == rb.eta_dot and np.isfinite(ra.eta_dot)
    assert np.array_equal(a, b)
    plan.close()


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
def test_long_lines_in_a_batch(prec):
    torch = G.torch_mod()
    insts = [dotgen.tiny_instance(2, n, seed=60 + i, floor=0.02)
             for i, n in enumerate([(4, 9, 610), (6, 12, 300), (3, 20, 900), (8, 16, 40)])]
    tols = [1e-2, 2e-3, 5e-3, 1e-3]
    batch = B.dot_batch_create(insts, per_instance=[dict(tol=t) for t in tols], max_iter=10 ** 6, precision=prec)
    ws = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
    B.dot_batch_reset(batch, ws.data_ptr(), G.stream_handle())
    res = B.dot_batch_run(batch, ws.data_ptr(), 400, G.stream_handle())
    for i, inst in enumerate(insts):
        plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, tol=tols[i], max_iter=10 ** 6,
                                 precision=prec)
        r, _ = _solve(plan, 400, True)
        assert (res[i].term, res[i].iters, res[i].eta_dot, res[i].objective) == (r.term, r.iters, r.eta_dot, r.objective)
        plan.close()
    batch.close()
