"""The gradient kernel's tiles (64 samples per wavefront, 4 wavefronts per
workgroup, at most 256 workgroups) at the batch sizes where they end, against
the oracle."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from oracle import mlp  # noqa: E402
from paper_1207_3392_amd import hydro  # noqa: E402
from test_gpu_learned import _abs_gradient, random_params  # noqa: E402


@pytest.mark.parametrize("batch", [1, 15, 16, 63, 64, 65, 255, 257, 65536, 65600 + 3])
def test_gradient_at_the_ends_of_tiles(batch):
    rng = np.random.default_rng(batch)
    P = random_params(5)
    n = 4096
    X = rng.uniform(-1, 1, size=(n, 4)).astype(np.float32)
    T = rng.normal(scale=0.5, size=n).astype(np.float32)
    idx = rng.integers(0, n, size=batch).astype(np.int32)
    tr = hydro.Trainer(P)
    g, loss = tr.gradient(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), torch.from_numpy(idx).cuda())
    again, _ = tr.gradient(torch.from_numpy(X).cuda(), torch.from_numpy(T).cuda(), torch.from_numpy(idx).cuda())
    tr.close()
    assert np.array_equal(g, again)  # sums in a fixed order
    Xb, Tb = X[idx].astype(np.float64), T[idx].astype(np.float64)
    lref, gref = mlp.loss_and_grad(P.astype(np.float64), Xb, Tb, bf16=True)
    # a few roundings to bfloat16 (2^-9 each) per term of the sum over the
    # batch: 2^-6 of the sum of the terms' magnitudes.  The loss: each residual
    # is off by an FP32 sum's rounding or one bfloat16 unit of an activation.
    A = _abs_gradient(P.astype(np.float64), Xb, Tb)
    assert np.all(np.abs(g - gref) <= 2.0 ** -6 * A + 1e-7 * np.abs(gref).max())
    assert loss == pytest.approx(lref, rel=2.0 ** -6)
