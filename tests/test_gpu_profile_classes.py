"""Kernel classes: the one-sweep iteration and the plane solve are recorded as
runs launch them, the ten classes of the separate launches each by themselves,
and what is recorded changes no bit of the iterates."""
import re
import os

import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from paper_2505_05424_amd import perfmodel as PM
from tests import gpu_util as G

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_the_binding_names_the_headers_classes():
    src = open(os.path.join(ROOT, "include", "dotsocp.h")).read()
    ids = {int(v) for v in re.findall(r"DOT_K_[A-Z_]+ = (-?\d+)", src)}
    assert ids == set(B.KERNEL_CLASSES.values()) | {-1}


@pytest.mark.parametrize("D,n", [(1, (16, 32)), (2, (8, 20, 24)), (3, (4, 6, 8, 10))])
def test_every_class_has_its_bytes(D, n):
    for w in (4, 8):
        kb, lp = PM.kernel_bytes(D, n, w), PM.launches_per_iteration(D)
        for name in B.KERNEL_CLASSES:
            assert kb[name] >= 0 and (name in lp or name in ("resid", "final")), name


def _recorded(plan, name, its=20):
    """Launches of one class in `its` iterations from zero, and the state."""
    B.dot_profile_select(plan, B.KERNEL_CLASSES[name] if name else -1)
    s = G.GpuState(plan)
    s.reset()
    s.run(its)
    launches = B.dot_profile_read(plan)[1]
    B.dot_profile_select(plan, -1)
    return launches, G.host(s.buf)[:plan.info.off_w]


# grid, precision, one sweep?, plane solve?
CASES = [("2d-large", (31, 130, 140), B.DOT_FP64, True, False), ("1d-large", (600, 900), B.DOT_MIXED, True, False),
         ("2d-small", (8, 20, 24), B.DOT_MIXED, False, True), ("1d-small", (16, 32), B.DOT_FP64, False, True),
         ("3d", (12, 40, 27, 31), B.DOT_FP64, False, False)]


@pytest.mark.gpu
@pytest.mark.parametrize("name,n,prec,sweep,plane", CASES, ids=[c[0] for c in CASES])
def test_classes_record_what_runs_launch(name, n, prec, sweep, plane):
    print(f"[case] classes {name}", flush=True)
    inst = dotgen.tiny_instance(len(n) - 1, n, seed=5, floor=0.02)
    plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)
    none, ref = _recorded(plan, None)
    assert none == 0
    expect = {"sweep": 20 if sweep else 0, "plane": 20 if plane else 0, "cone": 20, "qd": 20, "beta": 20, "rhs": 20}
    for cls, count in expect.items():
        launches, state = _recorded(plan, cls)
        assert launches == count, cls
        assert np.array_equal(state, ref), cls
    with pytest.raises(B.DotError):
        B.dot_profile_select(plan, max(B.KERNEL_CLASSES.values()) + 1)
    plan.close()
