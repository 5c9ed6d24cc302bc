"""The training pass at the edges of its division into tiles of 16 samples and
256 workgroups (several tiles each beyond 4096 samples): gradient and loss
against the float64 oracle, and the same bits from a second call."""
import numpy as np
import pytest

from oracle import mlp as Mo
from tests.test_gpu_mlp import data, normalised

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [2, 15, 16, 17, 33, 4095, 4096, 4097, 9001])
def test_gradient_over_tiles(n):
    from paper_2401_07965_amd import pa
    X, y, xm, xs, ym, ys = data(n, n)
    p = Mo.init_params(6)
    m = pa.PAMlp(p, xm, xs, ym, ys, max_samples=n + 3)
    m.set_data(X, y)
    print(f"[mlp] n={n}", flush=True)
    g, loss = m.gradient()
    Xn, yn = normalised(X, y, xm, xs, ym, ys)
    lo, go = Mo.loss_and_grad(p.astype(np.float64), Xn, yn)
    # float32 products and sums: relative errors of a few 1e-7 per operation
    assert abs(loss - lo) <= 1e-5 * lo
    assert np.linalg.norm(g - go) <= 1e-4 * np.linalg.norm(go)
    g2, loss2 = m.gradient()
    assert np.array_equal(g, g2) and loss == loss2
    m.close()
