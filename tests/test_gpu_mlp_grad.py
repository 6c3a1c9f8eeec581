"""The surrogate's loss and gradient at the edges of their 16-sample groups, 32-sample steps and
256-sample chunks, against the oracle, with the tolerances of tests/test_gpu_mlp.py."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2609_17661_amd import pic1d

from .test_gpu_mlp import GRAD_TOL, _box_inputs, _params, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 33, 255, 256, 257, 2049])
def test_gradient_at_chunk_edges(n):
    torch = _torch()
    print("gradient", n, flush=True)
    p = _params(71, 1.5).astype(np.float32).astype(np.float64)
    X = _box_inputs(72 + n, n)
    T = np.random.default_rng(73).standard_normal((n, 3)).astype(np.float32)
    loss, g = pic1d.mlp_loss_grad(torch.from_numpy(p.astype(np.float32)).cuda(), torch.from_numpy(X).cuda(),
                                  torch.from_numpy(T).cuda())
    L, gref = omlp.loss_and_grad(p, omlp.normalize_inputs(X.astype(np.float64)), T.astype(np.float64))
    g = g.cpu().numpy().astype(np.float64)
    assert abs(loss - L) <= 1e-5 * L
    k = 0
    for o, i in omlp.LAYERS:
        for size in (o * i, o):
            a, b = g[k:k + size], gref[k:k + size]
            assert np.linalg.norm(a - b) <= GRAD_TOL * np.linalg.norm(b), (o, i, size)
            k += size
