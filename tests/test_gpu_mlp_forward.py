"""The surrogate's forward pass on both sides of its small-batch and its large-batch kernel: group
edges, and parameters that are not 16-byte aligned (the packing path), against the oracle."""
import numpy as np
import pytest

from oracle import mlp as omlp
from paper_2609_17661_amd import pic1d

from .test_gpu_mlp import OUT_TOL, _box_inputs, _params, _torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,shift", [(1, 0), (17, 0), (4095, 0), (4096, 0), (4097, 0), (33, 1), (4096, 3), (262143, 0),
                                     (262149, 1)])
def test_forward_at_small_batch_edges(n, shift):
    torch = _torch()
    print("forward", n, shift, flush=True)
    p = _params(81, 1.5).astype(np.float32)
    X = _box_inputs(82, n)
    buf = torch.zeros(p.size + 4, dtype=torch.float32, device="cuda")
    buf[shift:shift + p.size] = torch.from_numpy(p).cuda()
    out = pic1d.mlp_forward(buf[shift:shift + p.size], torch.from_numpy(X).cuda()).cpu().numpy().astype(np.float64)
    ref, _ = omlp.forward(p.astype(np.float64), omlp.normalize_inputs(X.astype(np.float64)))
    assert np.all(np.abs(out - ref) <= OUT_TOL * np.maximum(1.0, np.abs(ref)))
