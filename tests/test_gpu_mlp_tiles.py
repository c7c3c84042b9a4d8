"""Network training at the edges of the gradient kernel: sample counts around a
tile (16), a workgroup (64) and a full round (4096) against the CPU reference's
bounds, and the operand copies that an Adam step writes: after training, the
gradient equals, bit for bit, that of a fresh model given the same parameters."""
from __future__ import annotations

import numpy as np
import pytest

from oracle import mlp
from test_gpu_mlp import bf16_bits, dev, features, model_with, params

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 15, 17, 63, 65, 1025, 4095, 4097, 8257])
def test_gradient_tiles(n):
    flat = params(n)
    X = features(n, n)
    t = np.random.default_rng(n).uniform(0.0, 1.0, n).astype(np.float32).astype(np.float64)
    feat, tgt = dev(bf16_bits(X), torch.int16), dev(t, torch.float32)
    M = model_with(flat)
    g = M.grad(feat, tgt).cpu().numpy().astype(np.float64)
    ge, _ = mlp.backward(flat, X, t, True)
    assert np.all(np.abs(g - ge) <= mlp.backward_bound(flat, X, t))
    M.train(feat, tgt, steps=5, batch=n, lr=1e-3, seed=n)
    after = M.get_params()
    F = model_with(after.astype(np.float64))
    np.testing.assert_array_equal(M.grad(feat, tgt).cpu().numpy(), F.grad(feat, tgt).cpu().numpy())
    assert not np.array_equal(after, flat.astype(np.float32))
