"""The training kernels at batch sizes around their tiles (16 samples a
forward wave, 64 a backward chunk, at most 128 partial gradients) and on
operands that are not 16-byte aligned, against the FP64 reference: logits
within one BF16 unit of the hidden layer's terms, gradients within BF16
rounding (2^-6) of the sum of the magnitudes of their terms."""
import numpy as np
import pytest

from oracle import mlp
from tests.test_gpu_learned import _abs_gradient, _params

pytestmark = pytest.mark.gpu


def _at(a, offset):
    """`a` on the GPU, its first element `offset` elements past an allocation."""
    import torch
    buf = torch.empty(a.numel() + offset, dtype=a.dtype, device="cuda")
    out = buf[offset:].view(a.shape)
    out.copy_(a)
    return out


@pytest.mark.parametrize("batch,offset", [(1, 0), (15, 0), (16, 1), (17, 0), (63, 0), (64, 4), (65, 1), (130, 0), (8257, 0)])
def test_batch_sizes(batch, offset):
    import torch
    from paper_2201_12193_amd.mrhweno import MLP_PARAMS, mlp_backward, mlp_cache_bytes, mlp_forward
    print(f"mlp: batch={batch} offset={offset}", flush=True)
    rng = np.random.default_rng(batch)
    X = torch.from_numpy(0.5 * rng.standard_normal((batch, 320))).to(torch.bfloat16)
    X[:, 301:] = 0
    P = _params(4, b3=0.05)
    Xd = _at(X, offset)
    Pd = _at(torch.from_numpy(np.asarray(P, dtype=np.float32)).to(torch.bfloat16), offset)
    y = (rng.random(batch) < 0.5).astype(np.float32)
    cache = torch.empty(mlp_cache_bytes(batch), dtype=torch.uint8, device="cuda")
    z, loss = torch.empty(batch, device="cuda"), torch.empty(batch, device="cuda")
    grads = torch.full((MLP_PARAMS,), 7.0, device="cuda")
    again = torch.empty_like(grads)
    yd = torch.from_numpy(y).cuda()
    mlp_forward(Xd, Pd, cache, z)
    mlp_backward(Xd, Pd, cache, yd, grads, loss)
    mlp_backward(Xd, Pd, cache, yd, again, loss)
    torch.cuda.synchronize()
    assert torch.equal(grads, again)
    X64 = X.float().numpy().astype(np.float64)
    w = mlp.unpack(P)
    zr, a = mlp.forward(X64, P, bf16_hidden=True)
    zg = z.cpu().numpy().astype(np.float64)
    # FP32 sums may move a hidden value across a BF16 rounding boundary
    bound = 2.0 ** -7 * (np.abs(a["h1"]) @ (np.abs(w["W2"]).T @ np.abs(w["W3"])))
    assert np.all(np.abs(zg - zr) <= 1e-4 * (np.abs(zr).mean() + 1e-3) + bound)
    assert np.allclose(loss.cpu().numpy(), mlp.bce(zg, y), rtol=1e-5, atol=1e-6)
    gr = mlp.gradient(X64, P, y, bf16_hidden=True)
    gabs = _abs_gradient(X64, P, y)
    gdz = _abs_gradient(X64, P, y, dz=np.full(batch, 0.25 * np.abs(zg - zr).max() / batch))
    gg = grads.cpu().numpy().astype(np.float64)
    assert np.all(np.abs(gg - gr) <= 2.0 ** -6 * gabs + 2.0 * gdz + 1e-12)
    assert np.all(gg[mlp.OFF["b3"] + 1:] == 0.0)
