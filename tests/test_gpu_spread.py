"""Spreading on the matrix cores: a tile's particles are listed in rounds and
summed in batches of 128, so crowded tiles are checked at counts around a
batch, at several batches with a remainder and over more than one listing
round, together with tiles that hold nothing."""
import numpy as np
import pytest

import synth
from oracle import ewald
from parity import check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 127, 128, 129, 400, 1500])
def test_crowded_tiles(gpu_lib, n):
    """n particles within a sphere of diameter 3 (a few grid nodes) about a
    tile corner next to the box boundary, at every tile depth, against the
    direct Fourier sums (the bar of the other wave-space tests: the window's
    truncation at 8 nodes)."""
    import torch

    L, M, xi = 40.0, 128, 0.5
    rng = np.random.default_rng(3100 + n)
    d = rng.standard_normal((n, 3))
    d *= (1.5 * rng.random((n, 1)) ** (1 / 3)) / np.linalg.norm(d, axis=1, keepdims=True)
    x = (np.array([0.2, 0.2, 5.0]) + d) % L
    F = synth.normals(3200 + n, (n, 3))
    ref = ewald.wave_apply_direct(x, F, M, L, 1.0, 1.0, xi)
    s = gpu_lib.Sampler(n, L, xi=xi, rcut=8.0, grid=M, support=8, tol=1e-6, precision="fp32")
    s.set_positions(torch.as_tensor(x, dtype=torch.float32, device="cuda"))
    Fd = torch.as_tensor(F, dtype=torch.float32, device="cuda")
    for depth in (8, 16, 32):
        s.set_launch_shape(depth, 0, 0)
        u = s.wave_apply(Fd)
        torch.cuda.synchronize()
        check(u.double().cpu().numpy(), ref, 1e-4, f"n={n}, tile depth {depth}")
    s.close()
