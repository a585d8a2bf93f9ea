"""A context whose stream is held up by work of its caller's does not hold up
another one through the side stream they share: its step waits for that work
before it puts anything there."""
import threading
import time

import pytest

from paper_1710_09421_amd import workloads

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ek():
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1710_09421_amd import ek as binding
    binding.lib()
    return binding


def make(ek, seed, stream):
    wl = workloads.pore_system((80, 72, 72), 10, 5, 0.01, 0.01, -0.01, 8, seed,
                               bead_q=workloads.STABLE_BEAD_CHARGE)   # 414,720 sites
    with torch.cuda.stream(stream):
        ctx = ek.from_workload(wl, precision=ek.EK_FP32, poisson_method=ek.EK_POISSON_MG,
                               poisson_tol=1e-8)
        ctx.step(2)
    return ctx


def hold(stream, cycles):
    with torch.cuda.stream(stream):
        torch.cuda._sleep(cycles)


def test_a_held_stream_holds_no_other_context(ek):
    ours = torch.cuda.Stream()
    a = make(ek, 84, ours)
    hold(ours, 1000)
    ours.synchronize()
    cycles, t = 20_000_000, time.perf_counter()
    hold(ours, cycles)
    ours.synchronize()
    cycles = int(cycles * 0.5 / (time.perf_counter() - t))   # half a second

    def timed_steps():
        t = time.perf_counter()
        a.step(2)
        return time.perf_counter() - t

    for _ in range(6):                 # a stream that shares no hardware queue with ours
        theirs = torch.cuda.Stream()
        hold(theirs, cycles)
        free = timed_steps()
        theirs.synchronize()
        if free < 0.1:
            break
    else:
        pytest.skip("every stream shares a hardware queue with the context's")
    b = make(ek, 85, theirs)
    hold(theirs, cycles)
    t0 = time.perf_counter()
    other = threading.Thread(target=b.step, args=(1,))
    other.start()
    time.sleep(0.05)                   # its step has enqueued what it can
    took = timed_steps()
    other.join(timeout=30)
    print(f"alone {free:.4f} s, beside the held context {took:.4f} s, held {time.perf_counter() - t0:.2f} s")
    assert time.perf_counter() - t0 > 0.3
    assert took < 0.1
    a.close()
    b.close()
