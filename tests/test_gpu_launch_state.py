"""What one launch leaves for the next: the reduction words after an adaptive run, after a launch
that the caller captured and replayed, and after a cancelled one; a cancelled launch ends at
its start.  Bit for bit against models that only made the calls compared."""
import sys
import time

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


def _say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def nb():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    import paper_1912_10596_amd as nb
    nb.lib()
    return nb


def _state(m):
    return m.get_state().cpu().numpy()


def _stepped(nb, d, *steps):
    m = nb.Model(d)
    for n in steps:
        m.step(n)
    return _state(m)


@pytest.mark.parametrize("nf,n_u", [(2, 3), (2, 40), (3, 40), (3, 4)])
def test_fixed_steps_after_adaptive_runs(nb, nf, n_u):
    """An adaptive run leaves its sums in the reduction words that the fixed steps use: the next
    stepping launch clears them, the one after it finds them clear.  Grids of one and of many
    blocks; runs that end well and runs that end at the attempt limit."""
    d = workloads.small_params(n_flavor=nf, n_energy=37, n_u=n_u, n_steps=40, r_start_km=600.0,
                               r_end_km=602.0)
    want = _stepped(nb, d, 5, 7)
    ref = nb.Model(d, adaptive=True)
    ref_st = ref.run_adaptive(1e-7)
    ref_x = _state(ref)
    m = nb.Model(d, adaptive=True)
    for i in range(2):
        _say(f"{nf} flavours, {2 * n_u} rows: adaptive run {i}, then fixed steps")
        assert m.run_adaptive(1e-7) == ref_st
        np.testing.assert_array_equal(_state(m), ref_x)
        m.reset()
        m.step(5)
        m.step(7)
        assert m.step_index() == 12
        np.testing.assert_array_equal(_state(m), want)
        m.reset()
        with pytest.raises(nb.NubulbError) as e:     # one attempt is not enough
            m.run_adaptive(1e-7, max_attempts=1)
        assert e.value.code == nb.NB_ESTEP
        m.step(5)                                    # from the initial state it is reset to
        m.step(7)
        np.testing.assert_array_equal(_state(m), want)
        m.reset()


@pytest.mark.parametrize("case", ["2f", "3f", "mixed", "batch"])
def test_eager_steps_between_replays_of_a_captured_call(nb, case):
    """A stepping call captured by the caller, replayed, with eager calls of the same model between
    the replays: each starts from clear reduction words, whichever came before."""
    import torch
    kw = {}
    if case == "batch":
        d = [workloads.small_params(n_energy=ne, n_u=nu, n_steps=60) for ne, nu in ((20, 30), (70, 4), (9, 25))]
    else:
        d = workloads.small_params(n_flavor=2 if case == "2f" else 3, n_energy=70, n_u=30, n_steps=60)
    if case == "mixed":
        d.update(r_start_km=460.0, r_end_km=463.0)
        kw = dict(precision=1)
    ref = nb.Model(d, **kw)
    ref.step(5)
    want = _state(ref)
    s = torch.cuda.Stream()
    m = nb.Model(d, stream=s, **kw)
    ref.reset()
    x0 = ref.get_state()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):
        m.step(5)
    torch.cuda.synchronize()
    for i in range(4):
        _say(f"{case}: replay {i}, then eager")
        m.set_state(x0, 0)
        with torch.cuda.stream(s):
            g.replay()
        torch.cuda.synchronize()
        np.testing.assert_array_equal(_state(m), want)
        m.set_state(x0, 0)
        m.step(2)
        m.step(3)
        assert m.step_index() == 5
        np.testing.assert_array_equal(_state(m), want)
    # a cancelled replay: the next eager call reports it, the one after it is as ever
    m.set_state(x0, 0)
    m.cancel(True)
    with torch.cuda.stream(s):
        g.replay()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(_state(m), x0.cpu().numpy())
    m.cancel(False)
    with pytest.raises(nb.NubulbError) as e:
        m.step(1)
    assert e.value.code == nb.NB_ETIMEOUT
    m.set_state(x0, 0)
    m.step(5)
    np.testing.assert_array_equal(_state(m), want)
    m.set_state(x0, 0)
    with torch.cuda.stream(s):
        g.replay()
    torch.cuda.synchronize()
    np.testing.assert_array_equal(_state(m), want)


def test_cancelled_launch_ends_at_its_start(nb):
    """Every block of a cancelled model's launch returns before it streams its beams: on a model
    whose stages take hundreds of microseconds the cancelled call takes less than half a stage
    (launch, report and clear of a call are 0.1 ms)."""
    import torch
    d = dict(workloads.extended_paper(n_u=40000))    # 80M beams
    m = nb.Model(d)
    m.step(1)

    def seconds(fn):
        torch.cuda.synchronize()
        t = time.perf_counter()
        fn()
        return time.perf_counter() - t

    stage = min(seconds(lambda: m.step(1)) for _ in range(5)) / 4
    m.cancel(True)

    def cancelled():
        with pytest.raises(nb.NubulbError) as e:
            m.step(1)
        assert e.value.code == nb.NB_ETIMEOUT

    t = min(seconds(cancelled) for _ in range(10))
    _say(f"stage {stage * 1e6:.0f} us, cancelled call {t * 1e6:.0f} us")
    assert m.step_index() == 6
    assert t < 0.5 * stage
    m.cancel(False)
    m.step(1)
    assert m.step_index() == 7


@pytest.mark.parametrize("nf", [2, 3])
def test_cancel_while_other_work_is_queued(nb, nf):
    """A cancel between the call and the launch's start, behind the caller's own work on the
    stream: the launch leaves state and step as they were."""
    import threading

    import torch
    d = workloads.small_params(n_flavor=nf, n_energy=70, n_u=30, n_steps=60)
    s = torch.cuda.Stream()
    m = nb.Model(d, stream=s)
    m.step(3)
    before = _state(m)
    got = []

    def call():
        try:
            m.step(4)
            got.append(None)
        except nb.NubulbError as e:
            got.append(e.code)

    with torch.cuda.stream(s):
        torch.cuda._sleep(200_000_000)      # about 0.1 s of spinning
    t = threading.Thread(target=call)
    t.start()
    time.sleep(0.02)
    m.cancel(True)
    t.join()
    assert got == [nb.NB_ETIMEOUT]
    assert m.step_index() == 3
    np.testing.assert_array_equal(_state(m), before)
    m.cancel(False)
    m.step(4)
    np.testing.assert_array_equal(_state(m), _stepped(nb, d, 3, 4))
