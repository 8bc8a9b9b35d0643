"""Schedules that set the waves of an axis and leave its tile width to the rule:
every count is taken that some tile up to the rule's width holds, whatever
width the rule has for the grid, with the rule's bits."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

ITEMS = {B.DOT_FP64: 3, B.DOT_MIXED: 5}  # work items of a wave on tiles of 32 or 64 lines, twice that on 16


def _fewest(L, prec):
    """Waves that hold an axis of L points on the narrowest tile."""
    rows = ((L - L // 2) + 15) // 16 + (L // 2 + 15) // 16
    return -(-rows // (2 * ITEMS[prec]))


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
@pytest.mark.parametrize("n", [(48, 150, 131), (32, 200, 180), (16, 48, 50), (40, 120, 70)])
def test_waves_alone(n, prec):
    print(f"[case] waves alone {n} precision={prec}", flush=True)
    inst = dotgen.tiny_instance(2, n, seed=66, floor=0.02)
    plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)
    s = G.GpuState(plan)
    s.reset()
    s.run(10)
    ref = G.host(s.buf)[:plan.info.off_w]
    rule = B.dot_plan_get_schedule(plan)
    for a in range(3):
        few = _fewest(n[a] + 1, prec)
        for w in range(1, 17):
            waves = [w if d == a else 0 for d in range(3)]
            if w < few:
                with pytest.raises(B.DotError):
                    B.dot_plan_set_schedule(plan, waves=waves)
                continue
            B.dot_plan_set_schedule(plan, waves=waves)
            got = B.dot_plan_get_schedule(plan)
            assert got["waves"][a] == w and got["cw"][a] <= rule["cw"][a]
            if w in (few, 16):
                s.reset()
                s.run(10)
                assert np.array_equal(G.host(s.buf)[:plan.info.off_w], ref), (a, w)
    plan.close()
