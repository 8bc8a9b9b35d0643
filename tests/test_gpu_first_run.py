"""The first run on a large grid allocates the buffer of the one-sweep
iterations: beside another thread's graph capture and another stream's work,
which it neither breaks nor waits for, and whatever the memory held before."""
import threading

import numpy as np
import pytest

import dotgen
from paper_2505_05424_amd import binding as B
from tests import gpu_util as G

pytestmark = pytest.mark.gpu

BIG = (31, 150, 150)


def _insts(count):
    return [dotgen.tiny_instance(2, BIG, seed=101 + k, floor=0.02) for k in range(count)]


def _plan(prec=B.DOT_FP64):
    i = _insts(1)[0]
    return B.dot_plan_create(i.D, i.n, i.rho0, i.rho1, i.mask, precision=prec, tol=-1.0, max_iter=10 ** 6)


@pytest.mark.parametrize("kind", ["plan", "batch"])
def test_first_run_beside_a_capture(kind):
    torch = G.torch_mod()
    if kind == "plan":
        plan = _plan()
        s = G.GpuState(plan)
        s.reset()
        first = lambda st: B.dot_run(plan, s.ptr, 4, st).iters  # noqa: E731
    else:
        batch = B.dot_batch_create(_insts(2), tol=-1.0, max_iter=10 ** 6)
        ws = torch.zeros(int(batch.workspace_bytes), dtype=torch.uint8, device="cuda")
        B.dot_batch_reset(batch, ws.data_ptr(), G.stream_handle())
        first = lambda st: B.dot_batch_run(batch, ws.data_ptr(), 4, st)[0].iters  # noqa: E731
    x = torch.ones(1 << 16, device="cuda")
    y = torch.zeros_like(x)
    torch.add(x, 1.0, out=y)
    own = torch.cuda.Stream()
    torch.cuda.synchronize()
    got = []
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, capture_error_mode="thread_local"):
        torch.add(x, 1.0, out=y)
        t = threading.Thread(target=lambda: got.append(first(own.cuda_stream)))
        t.start()
        t.join()
    assert got == [4]
    for k in range(3):
        x.fill_(k)
        graph.replay()
        torch.cuda.synchronize()
        assert bool((y == k + 1).all())


def test_first_run_does_not_wait_for_other_streams():
    torch = G.torch_mod()
    plan = _plan()
    s = G.GpuState(plan)
    s.reset()
    mine, other = torch.cuda.Stream(), torch.cuda.Stream()
    with torch.cuda.stream(other):
        torch.cuda._sleep(1 << 10)
    torch.cuda.synchronize()
    done = torch.cuda.Event()
    with torch.cuda.stream(other):
        torch.cuda._sleep(1 << 30)  # of the order of a second; the run takes a millisecond
        done.record()
    B.dot_run(plan, s.ptr, 4, mine.cuda_stream)
    running = not done.query()
    torch.cuda.synchronize()
    assert running
    plan.close()


@pytest.mark.parametrize("prec", [B.DOT_FP64, B.DOT_MIXED])
def test_first_run_in_memory_that_held_nans(prec):
    torch = G.torch_mod()
    a, b = _plan(prec), _plan(prec)
    s, t = G.GpuState(a), G.GpuState(b)
    s.reset()
    t.reset()
    B.dot_profile_select(b, B.KERNEL_CLASSES["cone"])
    t.run(35)
    B.dot_profile_select(b, -1)
    junk = torch.full((3 << 30,), 255, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    del junk
    torch.cuda.empty_cache()
    s.run(35)  # ends at an odd count: copied home from the buffer
    assert torch.equal(s.buf[:a.info.off_w], t.buf[:b.info.off_w])
    alpha = G.host(s.buf)[a.info.off_alpha:a.info.off_beta].view(np.float64).reshape((3,) + tuple(k + 1 for k in BIG))
    assert not alpha[0, -1].any() and not alpha[1, :, -1].any() and not alpha[2, :, :, -1].any()
    a.close()
    b.close()
