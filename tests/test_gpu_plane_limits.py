"""The plane solve at the last sizes that take it, against the transform passes
bitwise, with its launches counted; and the first sizes past them, which run
the passes."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

D64, MIX = B.DOT_FP64, B.DOT_MIXED
# grid, precision, taken?
CASES = [((63, 63), D64, True), ((71, 31), D64, True), ((17, 65), D64, True), ((4, 71, 31), D64, True),
         ((2, 2, 24, 71), D64, True), ((511, 6, 9), D64, True), ((15, 31, 20, 9), D64, True),
         # two line blocks in a wave
         ((63, 68, 50), D64, True), ((7, 7, 60, 66), D64, True), ((63, 64, 61), D64, True),
         ((62, 68, 50), D64, False), ((6, 8, 60, 66), D64, False), ((66, 55), D64, False), ((64, 62), D64, False),
         ((64, 64), MIX, True), ((5, 71, 63), MIX, True), ((511, 4, 6), MIX, True), ((1023, 25, 25), MIX, True),
         ((30, 32, 40, 16), MIX, True),
         ((100, 64, 64), D64, False), ((2, 2, 71, 62), D64, False), ((512, 6, 9), D64, False),
         ((3, 72, 20), D64, False), ((12, 40, 27, 31), D64, False), ((72, 40), MIX, False), ((5, 71, 64), MIX, False),
         ((1024, 25, 25), MIX, False), ((512, 4, 6), MIX, False)]


def _run(plan, its):
    s = G.GpuState(plan)
    s.reset()
    r = s.run(its)
    h, i = G.host(s.buf), plan.info
    return r, np.concatenate([h[i.off_phi:i.off_scratch], h[i.off_q:i.off_w]])


@pytest.mark.parametrize("n,prec,taken", CASES, ids=["x".join(map(str, c[0])) + "-" + "dm"[c[1]] for c in CASES])
def test_plane_limits(n, prec, taken):
    print(f"[case] plane limit {n} precision={prec}", flush=True)
    inst = dotgen.tiny_instance(len(n) - 1, n, seed=18, floor=0.0, masked=n[-1] > 8)
    plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)
    B.dot_profile_select(plan, B.KERNEL_CLASSES["plane"])
    _run(plan, 3)
    assert B.dot_profile_read(plan)[1] == (3 if taken else 0)
    B.dot_profile_select(plan, -1)
    ra, a = _run(plan, 37)
    s = B.dot_plan_get_schedule(plan)
    B.dot_plan_set_schedule(plan, s["cw"], s["waves"])  # written out: the passes
    rb, b = _run(plan, 37)
    assert ra.iters == rb.iters == 37 and ra.eta_dot == rb.eta_dot and np.isfinite(ra.eta_dot)
    assert np.array_equal(a, b)
    plan.close()
