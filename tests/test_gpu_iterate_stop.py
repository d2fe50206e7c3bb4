"""Nothing runs behind the iteration that ends a solve, though further ones are launched before its
statistics are read: the workspace is then left as by a call of that many iterations, byte for byte, but
for the clock's stamps (16 bytes an iteration) and, above 16,384 points, the order of the gathered angles."""
import numpy as np
import pytest
import torch

from paper_2405_13839_amd import synth
from tests.helpers import cuda, unit_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,beta", [(700, 0.0), (700, 2.3), (16_000, 2.3), (20_011, 0.0), (20_011, 2.3)])
@pytest.mark.parametrize("later", [False, True])
def test_no_work_behind_the_last_iteration(n, beta, later):
    from paper_2405_13839_amd import dwg
    c = synth.torus_ellipsoids(n, seed=n)
    P, area, prm = cuda(c.P), cuda(c.area), dwg.Params(lam=4.0, beta=beta)
    rng = np.random.default_rng(n)
    N0 = cuda(unit_rows(rng, c.n) * 0.5 + c.N_true)
    N0 = (N0 / N0.norm(dim=0)).contiguous()
    d = dwg.delta_anchor_mean(P)
    top = dwg.iterate(P, area, d, N0.clone(), prm, max_iters=24, fixed_iters=True)[1][:, 1].tolist()
    # a solve to the angle of its first iteration, or to that of a later one that is below all before it
    ends = next(t for t in range(24) if (t > 0) == later and all(top[t] < x for x in top[:t])) + 1
    left = []
    for its in (ends, 24):
        ws = torch.full((dwg.workspace_bytes(c.n, c.n, prm),), 0x5A, dtype=torch.uint8, device="cuda")
        N = N0.clone()
        _, st = dwg.iterate(P, area, d, N, prm, max_iters=its, fixed_iters=its == ends, eps_deg=top[ends - 1], ws=ws)
        torch.cuda.synchronize()
        assert st.shape[0] == ends
        left.append((ws, N))
    assert torch.equal(left[0][1], left[1][1])
    assert int((left[0][0] != left[1][0]).sum()) <= 16 * ends + (4096 if n > 16_384 else 0)
