"""The plane solve (kernels_plane.hpp), which small grids take, against the
transform passes (a schedule written out selects them): bitwise the same
iterates, at axis lengths around its 16-row blocks, its 4-wide k-steps and its
longest axes, and in a batch."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

GRIDS = [(1, 1), (63, 63), (71, 40), (2, 71), (64, 64), (30, 31), (5, 15, 16), (3, 63, 1), (9, 32, 64), (511, 6, 9),
         (4, 3, 17, 47), (2, 2, 71, 62), (12, 40, 27, 31)]


def _solve(plan, its, passes):
    if passes:
        s = B.dot_plan_get_schedule(plan)
        B.dot_plan_set_schedule(plan, s["cw"], s["waves"])
    s = G.GpuState(plan)
    s.reset()
    r = s.run(its)
    h, i = G.host(s.buf), plan.info
    return r, np.concatenate([h[i.off_phi:i.off_scratch], h[i.off_q:i.off_w]])


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
@pytest.mark.parametrize("n", GRIDS, ids=["x".join(map(str, n)) for n in GRIDS])
def test_plane_solve_gives_the_passes_bits(n, prec):
    print(f"[case] plane solve {n} precision={prec}", flush=True)
    inst = dotgen.tiny_instance(len(n) - 1, n, seed=17, floor=0.0, masked=n[-1] > 8)
    plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)
    ra, a = _solve(plan, 57, False)
    rb, b = _solve(plan, 57, True)
    assert ra.iters == rb.iters == 57 and ra.eta_dot == rb.eta_dot and np.isfinite(ra.eta_dot)
    assert np.array_equal(a, b)
    plan.close()


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
def test_plane_solve_in_a_batch(prec):
    torch = G.torch_mod()
    insts = [dotgen.tiny_instance(2, n, seed=40 + i, floor=0.02, masked=i == 1)
             for i, n in enumerate([(5, 15, 20), (12, 33, 16), (7, 40, 63)])]
    tols = [1e-2, 2e-3, 5e-4]
    batch = B.dot_batch_create(insts, per_instance=[dict(tol=t) for t in tols], max_iter=10 ** 6, precision=prec)
    ws = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
    B.dot_batch_reset(batch, ws.data_ptr(), G.stream_handle())
    res = B.dot_batch_run(batch, ws.data_ptr(), 3000, G.stream_handle())
    for i, inst in enumerate(insts):
        plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, tol=tols[i], max_iter=10 ** 6,
                                 precision=prec)
        r, _ = _solve(plan, 3000, True)
        assert B.TERM_NAMES[res[i].term] == "converged"
        assert (res[i].iters, res[i].eta_dot, res[i].objective) == (r.iters, r.eta_dot, r.objective)
        plan.close()
    batch.close()
