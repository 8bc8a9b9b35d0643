"""The one-sweep iteration on paths that the other files do not reach, each
against the separate sweeps and bitwise: with boxes of few and of many waves."""
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
