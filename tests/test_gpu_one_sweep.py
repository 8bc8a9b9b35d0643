"""The one-sweep iteration (kernels_fused.hpp), which large plans and batches
run, against the separate sweeps (a kernel class being timed selects them):
bitwise the same iterates, at grids that cut the workgroups' boxes and time
runs unevenly, through run calls that start and end at odd iteration counts,
and in batches whose members stop at different counts."""
import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

# all above the sizes from which runs take one sweep
GRIDS = [
    ("2d-one-time-segment", (1, 520, 520), False),
    ("2d-odd-masked", (7, 260, 262), True),
    ("2d-many-times", (155, 37, 90), True),
    ("2d-two-node-axis-long-last", (70, 1, 3999), False),
    ("2d-narrow-last", (300, 900, 2), False),
    ("1d-long-last", (400, 1400), False),
    ("1d-many-times", (1000, 540), False),
]


def _plan(n, masked, prec):
    inst = dotgen.tiny_instance(len(n) - 1, n, seed=91, floor=0.0 if masked else 0.01, masked=masked)
    return B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, precision=prec, tol=-1.0,
                             max_iter=10 ** 6)


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
@pytest.mark.parametrize("name,n,masked", GRIDS, ids=[g[0] for g in GRIDS])
def test_one_sweep_gives_the_separate_sweeps_bits(name, n, masked, prec):
    print(f"[case] one sweep {name} precision={prec}", flush=True)
    plan = _plan(n, masked, prec)
    a, b = G.GpuState(plan), G.GpuState(plan)
    a.reset()
    for k in (7, 13, 1, 1, 58):  # odd and even starts and ends, plain launches and graphs
        ra = a.run(k)
    B.dot_profile_select(plan, B.KERNEL_CLASSES["cone"])
    b.reset()
    rb = b.run(80)
    B.dot_profile_select(plan, -1)
    for f in ("objective", "dual_objective", "eta_dot", "eta_p_soc", "eta_d_soc", "sigma", "iters", "checks"):
        assert getattr(ra, f) == getattr(rb, f), f
    w = plan.info.off_w
    assert np.array_equal(G.host(a.buf)[:w], G.host(b.buf)[:w])
    assert np.isfinite(ra.eta_dot)
    plan.close()


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
def test_batch_members_stop_in_one_sweep_iterations(prec):
    """Members together above the size from which a batch takes one sweep (in
    mixed precision each alone runs separate sweeps); they stop at checks of
    even and odd iteration counts, and the layout shrinks around them until
    the rest runs separate sweeps again."""
    torch = G.torch_mod()
    sizes = [(40, 80, 90), (32, 100, 90), (48, 70, 88), (36, 120, 66), (60, 64, 76), (24, 110, 110), (50, 72, 80)]
    insts = [dotgen.tiny_instance(2, n, seed=70 + i, floor=0.02, masked=i % 2 == 1) for i, n in enumerate(sizes)]
    tols = [3e-2, 1e-2, 2e-3, 1e-3, 5e-3, 3e-3, 4e-4]
    kw = [dict(tol=t) for t in tols]
    batch = B.dot_batch_create(insts, per_instance=kw, max_iter=10 ** 6, precision=prec)
    ws = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
    st = G.stream_handle()
    B.dot_batch_reset(batch, ws.data_ptr(), st)
    B.dot_batch_run(batch, ws.data_ptr(), 35, st)
    res = B.dot_batch_run(batch, ws.data_ptr(), 3000, st)
    odd = 0
    for i, inst in enumerate(insts):
        print(f"[case] member {i} {inst.n} iters={res[i].iters}", flush=True)
        assert B.TERM_NAMES[res[i].term] == "converged"
        odd += res[i].iters % 2
        plan = B.dot_plan_create(inst.D, inst.n, inst.rho0, inst.rho1, inst.mask, tol=tols[i], max_iter=10 ** 6,
                                 precision=prec)
        s = G.GpuState(plan)
        s.reset()
        r = s.run(3035)
        for f in ("iters", "checks", "objective", "eta_dot", "sigma"):
            assert getattr(res[i], f) == getattr(r, f), (i, f)
        rho, m = s.extract()
        rb, mb = B.dot_batch_extract(batch, ws.data_ptr(), i, st)
        assert np.array_equal(rb, rho), i
        for x, y in zip(mb, m):
            assert np.array_equal(x, y), i
        plan.close()
    assert 0 < odd < len(insts)  # both kinds of stop were met
