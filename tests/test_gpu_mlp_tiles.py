"""The MLP kernels at the edges of their tiles: 32 rows per wavefront, 512 per block of the forward
pass, 128 per block of the training step, one mask count per 8,192 rows; rows that start at any
float; and the learned normals' own feature path against the features it stands for."""
import numpy as np
import pytest
import torch

from oracle import mlp as om
from paper_2405_13839_amd import mlp_init, synth
from tests.helpers import cuda, host

pytestmark = pytest.mark.gpu


def _blob(seed):
    rng = np.random.default_rng(seed)
    return (mlp_init.init_params(seed) + 0.05 * rng.standard_normal(om.N_PARAMS)).astype(np.float32)


def _rel(a, b):
    return float(np.linalg.norm(np.asarray(a, np.float64) - b) / max(np.linalg.norm(b), 1e-30))


@pytest.mark.parametrize("B", [1, 16, 31, 32, 33, 511, 513, 8193, 8225])
def test_forward_tiles(B):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(B)
    blob, X = _blob(2), rng.standard_normal((B, 48)).astype(np.float32)
    buf = torch.empty(B * 48 + 1, device="cuda")
    for off in (0, 1):  # rows aligned to 16 bytes, then to 4
        Xc = buf[off:off + B * 48].view(B, 48)
        Xc.copy_(cuda(X))
        Y = host(dwg.mlp_infer(cuda(blob), Xc))
        # tolerance of a few one-ulp BF16 flips among a row's 256 activations
        assert _rel(Y, om.forward(blob, X)[1]) < 1e-3


@pytest.mark.parametrize("B,masked", [(1, False), (31, True), (127, True), (128, False), (129, True), (300, True),
                                      (20_001, True)])
def test_train_tiles(B, masked):
    from paper_2405_13839_amd import dwg
    rng = np.random.default_rng(B)
    blob, X = _blob(4), rng.standard_normal((B, 48)).astype(np.float32)
    T = rng.standard_normal((B, 3))
    T = (T / np.linalg.norm(T, axis=1, keepdims=True)).astype(np.float32)
    mask = (rng.uniform(size=B) < 0.8).astype(np.uint8)
    mask[0] = 1
    p = cuda(blob)
    m, v = torch.zeros_like(p), torch.zeros_like(p)
    loss, g = dwg.mlp_train_step(p, m, v, 1, 1e-3, cuda(X), cuda(T), cuda(mask, torch.uint8) if masked else None,
                                 want_grad=True)
    rl, rg = om.loss_and_grad(blob, X, T, mask if masked else np.ones(B, np.uint8))
    assert abs(host(loss)[0] - rl) <= 1e-4 * max(1.0, abs(rl))
    off = 0
    for name, shp in om.SHAPES:
        k = int(np.prod(shp))
        # at one row, a one-ulp flip of f of 128 values moves the gradient by 2^-8 sqrt(f / 128): f = 8
        assert _rel(host(g)[off:off + k], rg[off:off + k]) < 2e-3, name
        off += k
    np.testing.assert_allclose(host(m), 0.1 * host(g), rtol=1e-5, atol=0)


def test_train_step_with_no_kept_row():
    from paper_2405_13839_amd import dwg
    p = cuda(_blob(4))
    before, m, v = p.clone(), torch.zeros_like(p), torch.zeros_like(p)
    X, T = torch.randn(70, 48, device="cuda"), torch.zeros(70, 3, device="cuda")
    loss, g = dwg.mlp_train_step(p, m, v, 1, 1e-3, X, T, torch.zeros(70, dtype=torch.uint8, device="cuda"),
                                 want_grad=True)
    assert float(loss) == 0.0 and not g.any() and torch.equal(p, before)


@pytest.mark.parametrize("n", [18, 33, 4097, 20_003])
def test_learned_normals_equal_the_mlp_of_the_features(n):
    from paper_2405_13839_amd import dwg
    P = cuda(synth.torus_ellipsoids(max(n, 64), seed=6).P[:, :n])
    blob = cuda(_blob(8))
    assert torch.equal(dwg.mlp_normals(P, blob).T.contiguous(), dwg.mlp_infer(blob, dwg.features(P, 4096)))
