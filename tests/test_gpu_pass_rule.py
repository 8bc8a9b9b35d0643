"""The rule for the tile widths and waves of the transform passes, at both sides
of its limits: short axes take a middle width below 256 tiles only beside a
neighbour that has it, and five FP32 waves only where three workgroups share a
CU. Widths and waves change no bit."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

D64, MIX = B.DOT_FP64, B.DOT_MIXED
# grid, precision, axis -> tile width
WIDTHS = [((46, 24, 153), D64, {0: 16, 1: 16}), ((46, 24, 153), MIX, {0: 16, 1: 32}),
          ((96, 63, 58), D64, {0: 16, 1: 16}), ((96, 64, 58), D64, {0: 16, 1: 32}), ((53, 49, 31, 1), MIX, {1: 16, 2: 16}),
          ((30, 42, 22, 4), MIX, {0: 16, 1: 16, 2: 16}), ((28, 57, 18, 3), D64, {2: 16}),
          ((48, 150, 131), D64, {0: 32, 1: 32, 2: 32}), ((13, 41, 47, 11), MIX, {0: 32, 1: 32, 2: 32}),
          ((22, 26, 256), D64, {0: 32, 1: 32}), ((40, 120, 70), D64, {0: 32, 1: 16, 2: 32})]
# grid, precision, axis, waves
WAVES = [((64, 128, 128), MIX, 0, 5), ((75, 126, 143), MIX, 0, 5), ((64, 30, 30, 30), MIX, 0, 4),
         ((139, 102, 123), MIX, 1, 4), ((64, 128, 128), D64, 0, 4)]


def _plan(n, prec):
    inst = dotgen.tiny_instance(len(n) - 1, n, seed=67, floor=0.02)
    return B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)


def _state(plan):
    s = G.GpuState(plan)
    s.reset()
    s.run(10)
    return s.buf[:plan.info.off_w]


@pytest.mark.parametrize("n,prec,widths", WIDTHS, ids=["x".join(map(str, c[0])) + "-" + "dm"[c[1]] for c in WIDTHS])
def test_widths(n, prec, widths):
    print(f"[case] widths {n} precision={prec}", flush=True)
    plan = _plan(n, prec)
    cw = B.dot_plan_get_schedule(plan)["cw"]
    assert {a: cw[a] for a in widths} == widths
    a = _state(plan)
    flip = [48 - cw[d] if d in widths else 0 for d in range(len(n))]  # 16 for 32 and 32 for 16
    B.dot_plan_set_schedule(plan, cw=flip)
    assert G.torch_mod().equal(a, _state(plan))
    plan.close()


@pytest.mark.parametrize("n,prec,a,waves", WAVES, ids=["x".join(map(str, c[0])) + "-" + "dm"[c[1]] for c in WAVES])
def test_waves(n, prec, a, waves):
    plan = _plan(n, prec)
    assert B.dot_plan_get_schedule(plan)["waves"][a] == waves
    plan.close()


def test_widths_of_a_batch():
    """Members count together: alone each has narrow tiles."""
    insts = [dotgen.tiny_instance(2, (30, 33, 36), seed=68 + k, floor=0.02) for k in range(6)]
    one = B.dot_batch_create(insts[:1], tol=-1.0, max_iter=10)
    six = B.dot_batch_create(insts, tol=-1.0, max_iter=10)
    assert B.dot_batch_get_schedule(one)["cw"] == [16, 16, 16]
    assert B.dot_batch_get_schedule(six)["cw"] == [32, 32, 32]
    one.close()
    six.close()
