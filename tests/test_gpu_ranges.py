"""The rotation and the 3x3 exponential over the exponents their in-range square roots and
divisions accept and over those that take the general forms (tiny and zero angles, states
with vanishing parts), against the oracle, whose operations are the IEEE ones: bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hooks():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no HIP device visible")
    import paper_1912_10596_amd  # noqa: F401
    from paper_1912_10596_amd import testhooks
    testhooks.lib()
    return testhooks


def _dev(a):
    import torch
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("lo,hi", [(-300, -160), (-160, -100), (-100, 0), (0, 15)])
def test_rotation_exponents(hooks, oracle, lo, hi):
    rng = np.random.default_rng(7 - lo)
    n = 4000
    x = rng.standard_normal((n, 3)) * 10.0 ** rng.uniform(lo, hi, (n, 1))
    x[::50] = 0.0
    x[1::7, 1] = 0.0
    p = rng.standard_normal((n, 3))
    p /= np.linalg.norm(p, axis=1, keepdims=True)
    p[::11] = [0.0, 0.0, 1.0]
    got = hooks.test_rotate(_dev(x), _dev(p)).cpu().numpy()
    want = np.stack([oracle.rotate(x[i], p[i]) for i in range(n)])
    np.testing.assert_array_equal(got, want)


@pytest.mark.parametrize("lo,hi", [(-29, -10), (-10, 1), (1, 14)])
@pytest.mark.parametrize("mix", [0, -12, -60, -120, -200])
def test_exponential_exponents(hooks, oracle, lo, hi, mix):
    """mix: decimal exponent of the off-diagonal entries against the diagonal ones, so that
    states on the axes have parts as small, or (mix = 0 with zeroed rows) none at all."""
    rng = np.random.default_rng(11 - lo - mix)
    n = 1500
    k = rng.standard_normal((n, 9)) * 10.0 ** rng.uniform(lo, hi, (n, 1))
    k[:, 3:] *= 10.0 ** mix
    k[::9, 3:5] = 0.0
    k[::9, 7:] = 0.0
    k[1::9, 3:] = 0.0
    p = np.zeros((n, 6))
    p[np.arange(n), 2 * rng.integers(0, 3, n)] = 1.0
    q = rng.standard_normal((n, 6))
    q /= np.linalg.norm(q, axis=1, keepdims=True)
    p[::3] = q[::3]
    got = hooks.test_exp3(_dev(k), _dev(p)).cpu().numpy()
    want = np.stack([oracle.exp3_apply(k[i], p[i]) for i in range(n)])
    np.testing.assert_array_equal(got, want)
