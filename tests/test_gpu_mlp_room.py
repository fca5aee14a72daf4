"""The predictor's arrays through its pinned room (4 Mi floats: from 25891 rows on
in pieces) and, on a handle's first call, without it: the same results."""
import numpy as np
import pytest

from oracle import mlp_ref as R
from paper_2210_16998_amd import tpg
from tests.gpu_util import say

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [(1, 48, 1), (25890, 25891, 40), (65000, 3, 140001)])
def test_arrays_in_pieces(sizes):
    rng = np.random.default_rng(sizes[0])
    m = tpg.MLP(seed=6)
    p = m.params()
    for n in sizes:
        say("case", n)
        x = rng.normal(0, 2, (n, R.IN)).astype(np.float32)
        t = rng.normal(0, 1, (n, R.OUT)).astype(np.float32)
        y = m.forward(x)
        assert np.array_equal(y, tpg.MLP(seed=6).forward(x))
        for lo in (0, n // 2, max(0, n - 77)):  # rows are independent
            assert np.array_equal(y[lo:lo + 77], m.forward(x[lo:lo + 77])), lo
        g, loss = m.gradients(x, t)
        g1, loss1 = tpg.MLP(seed=6).gradients(x, t)
        assert np.array_equal(g, g1) and loss == loss1
        g2, loss2 = m.gradients(x, t)
        assert np.array_equal(g, g2) and loss == loss2
        a, b = tpg.MLP(seed=6), tpg.MLP(seed=6)
        b.forward(x[:1])  # b's arrays go through the room, a's first ones do not
        for _ in range(3):
            la, lb = a.train_step(x, t, 1e-3), b.train_step(x, t, 1e-3)
            assert la == lb
        assert np.array_equal(a.params(), b.params())
    assert np.array_equal(m.params(), p)


def test_steps_without_a_loss():
    """A step that returns no loss does not wait; the next one's arrays take the
    same room."""
    rng = np.random.default_rng(9)
    a, b = tpg.MLP(seed=2), tpg.MLP(seed=2)
    for k in range(12):
        n = (64, 30000, 1, 4000)[k % 4]
        x = rng.normal(0, 2, (n, R.IN)).astype(np.float32)
        t = rng.normal(0, 1, (n, R.OUT)).astype(np.float32)
        tpg._check(tpg.lib().tpg_mlp_train_step(a._h, x.ctypes.data, t.ctypes.data, n, 1e-3, None))
        x0, t0 = x.copy(), t.copy()
        x[:], t[:] = 0, 0  # the caller's arrays are its own again
        b.train_step(x0, t0, 1e-3)
    assert np.array_equal(a.params(), b.params())


def test_parameters_set_after_a_step_without_a_loss():
    """The step is still at work when the parameters and the normalizer change:
    it takes the old ones and leaves the new ones alone."""
    rng = np.random.default_rng(11)
    n = 60000
    x = rng.normal(0, 2, (n, R.IN)).astype(np.float32)
    t = rng.normal(0, 1, (n, R.OUT)).astype(np.float32)
    a, b = tpg.MLP(seed=3), tpg.MLP(seed=4)
    for _ in range(5):
        tpg._check(tpg.lib().tpg_mlp_train_step(a._h, x.ctypes.data, t.ctypes.data, n, 0.5, None))
        a.set_params(b.params())
        a.set_normalizer(np.zeros(R.IN, np.float32), np.ones(R.IN, np.float32))
        assert np.array_equal(a.params(), b.params())
        assert np.array_equal(a.forward(x[:99]), b.forward(x[:99]))
