"""A launch of a cancelled model ends at its start."""
import sys
import time

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
