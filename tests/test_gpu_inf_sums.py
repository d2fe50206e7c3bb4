"""A sum that overflows float32: infinite without compensation (as plain additions give it), whichever
way the splits' and segments' partials are added; the other queries do not see it."""
import numpy as np
import pytest

from tests.helpers import cuda, host, unit_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("beta", [0.0, 2.3])
@pytest.mark.parametrize("n", [60, 3000])
@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_an_infinite_partial_stays_infinite(n, beta, sign):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(n)
    P = rng.uniform(-1, 1, (3, n)).astype(np.float32)
    N = unit_rows(rng, n)
    area = np.full(n, 1.0 / n, np.float32)
    P[:, 7], N[:, 7], area[7] = (5.0, 0.0, 0.0), (sign, 0.0, 0.0), 1e30
    Q = P[:, :20].copy()
    Q[:, 7] = (4.5, 0.0, 0.0)
    Q[:, 3] = (5.0 - 2.0 ** -20, 0.0, 0.0)  # a / (4 pi r^2) = 8e40
    w = host(dwg.gwn(cuda(P), cuda(N), cuda(area), None, cuda(Q), dwg.Params(beta=beta, compensated=False))[0])
    v = host(dwg.gwn(cuda(P), cuda(N), cuda(area), None, cuda(Q), dwg.Params(beta=beta, compensated=False), grad=False))
    for x in (w, v):
        assert x[3] == sign * np.inf
        assert np.isfinite(np.delete(x, 3)).all()
