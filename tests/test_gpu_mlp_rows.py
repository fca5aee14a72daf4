"""Row counts around the predictor kernels' tiles (16 rows a workgroup, steps
of 32 and splits of at least 128 rows for the weight gradients), on one model
in growing and shrinking order: what a larger call left in the padding must not
show in a smaller one."""
import numpy as np
import pytest

from oracle import mlp_ref as R
from paper_2210_16998_amd import tpg
from tests.gpu_util import say

pytestmark = pytest.mark.gpu

# bf16 roundings of three layers (2^-8 relative each) on the propagated
# absolute-term sums forward; twice that through the backward products
FWD_TOL, GRAD_TOL = 2.0 ** -6, 2.0 ** -5


@pytest.mark.parametrize("sizes", [(1, 15, 16, 17, 31, 32, 33), (2049, 65, 1),
                                   (127, 128, 129, 160, 161), (2080, 4097, 2047, 300)])
def test_row_counts_on_one_model(sizes):
    rng = np.random.default_rng(sizes[0])
    m = tpg.MLP(seed=4)
    p = m.params().astype(np.float64)
    mean = rng.normal(0, 1, R.IN).astype(np.float32)
    std = (rng.random(R.IN) + 0.5).astype(np.float32)
    m.set_normalizer(mean, std)
    for n in sizes:
        say("case mlp rows", n)
        x = rng.normal(0, 2, (n, R.IN)).astype(np.float32)
        t = rng.normal(0, 1, (n, R.OUT)).astype(np.float32)
        bound = FWD_TOL * R.abs_terms_forward(p, mean, std, x) + 1e-6
        assert np.all(np.abs(m.forward(x) - R.forward(p, mean, std, x, True)["y"]) <= bound), n
        g, loss = m.gradients(x, t)
        lref, gref = R.loss_and_grads(p, mean, std, x, t, True)
        assert abs(loss - lref) <= FWD_TOL * lref, n
        q = 0
        for name, shape in R.SHAPES:
            k = int(np.prod(shape))
            a, b = g[q:q + k].astype(np.float64), gref[q:q + k]
            assert np.max(np.abs(a - b)) <= GRAD_TOL * (np.max(np.abs(b)) + 1e-12), (n, name)
            q += k
        g2, loss2 = m.gradients(x, t)
        assert np.array_equal(g, g2) and loss == loss2, n
