"""The training step's kernels at ragged row counts and unaligned arrays.

Bars: the loss is a sum of squares accumulated in FP64 and rounded once to
fp32 (2^-23); dy is two fp32 roundings (2^-22); dw sums at most n products of
bf16 factors split exactly, with fp32 accumulation over 32-row chunks and
slots: 2e-6 of its norm, as for the row counts tested elsewhere.
"""
import numpy as np
import pytest
import torch

from paper_1611_09322_amd import precond

pytestmark = pytest.mark.gpu


def _at(a, shift, dtype):
    """A device copy of `a` starting `shift` elements past an aligned start."""
    t = torch.empty(a.size + shift, dtype=dtype, device="cuda")
    t[shift:].copy_(torch.as_tensor(a.reshape(-1)).to(dtype))
    return t[shift:]


# one row; around a 4-value piece of 9 n values, a 32-row chunk and one
# 4096-value block of dy; more 32-row chunks than the 256 wavefronts
@pytest.mark.parametrize("n", [1, 3, 31, 33, 455, 456, 8225])
@pytest.mark.parametrize("shift", [0, 1])
def test_loss_and_backward(gpu_lib, n, shift):
    r = np.random.default_rng(n)
    y, t = (r.standard_normal((n, 9)).astype(np.float32) for _ in range(2))
    yd, td, dy = _at(y, shift, torch.float32), _at(t, shift, torch.float32), _at(np.zeros((n, 9)), shift, torch.float32)
    loss = torch.full((1,), 7.0, device="cuda")
    gpu_lib.pse_mlp_loss_grad(yd.data_ptr(), td.data_ptr(), n, dy.data_ptr(), loss.data_ptr())
    torch.cuda.synchronize()
    d = (y - t).astype(np.float64)
    assert abs(float(loss[0]) / ((d**2).sum() / n) - 1) < 2.0**-23
    ref = 2.0 / n * d
    got = dy.cpu().numpy().reshape(n, 9)
    assert np.max(np.abs(got - ref)) <= 2.0**-22 * np.max(np.abs(ref))
    # dy written over y: the same values, and the loss of the original y
    gpu_lib.pse_mlp_loss_grad(yd.data_ptr(), td.data_ptr(), n, yd.data_ptr(), loss.data_ptr())
    torch.cuda.synchronize()
    assert abs(float(loss[0]) / ((d**2).sum() / n) - 1) < 2.0**-23
    assert np.array_equal(yd.cpu().numpy().reshape(n, 9), got)
    # backward pass with x and the activations at the same offset
    w = precond.init_weights(3)
    w["W3"] = 0.1 * r.standard_normal((9, 64))
    wb = torch.as_tensor(precond.pack(w)).to(torch.bfloat16).cuda()
    x = torch.as_tensor(r.standard_normal((n, 24))).to(torch.bfloat16)
    xa = x.cuda().contiguous()
    out, cache = torch.empty((n, 9), device="cuda"), torch.empty((n, 128), dtype=torch.bfloat16, device="cuda")
    gpu_lib.pse_mlp_forward(wb.data_ptr(), xa.data_ptr(), n, out.data_ptr(), cache.data_ptr())
    xs = _at(x.double().numpy(), shift, torch.bfloat16)
    cs = _at(cache.double().cpu().numpy(), shift, torch.bfloat16)
    nbytes = gpu_lib.pse_mlp_backward_workspace(n)
    work, dw = torch.empty(nbytes // 4, device="cuda"), torch.zeros(7312, device="cuda")
    gpu_lib.pse_mlp_backward(wb.data_ptr(), xs.data_ptr(), cs.data_ptr(), dy.data_ptr(), n, dw.data_ptr(),
                             work.data_ptr(), nbytes)
    torch.cuda.synchronize()
    f = wb.double().cpu().numpy()
    W2, W3 = f[2112:6208].reshape(64, 64), f[6272:7296].reshape(16, 64)[:9]
    h = cache.double().cpu().numpy()
    h1, h2, g = h[:, :64], h[:, 64:], dy.double().cpu().numpy().reshape(n, 9)
    d2 = (g @ W3) * (h2 > 0)
    d1 = (d2 @ W2) * (h1 > 0)
    ref = np.zeros(7312)
    ref[:2048].reshape(64, 32)[:, :24] = d1.T @ x.double().numpy()
    ref[2048:2112], ref[2112:6208], ref[6208:6272] = d1.sum(0), (d2.T @ h1).ravel(), d2.sum(0)
    ref[6272:7296].reshape(16, 64)[:9] = g.T @ h2
    ref[7296:7305] = g.sum(0)
    e = np.linalg.norm(dw.double().cpu().numpy() - ref) / np.linalg.norm(ref)
    print(f"dw n={n} shift={shift}: {e:.1e}", flush=True)
    assert e <= 2e-6
