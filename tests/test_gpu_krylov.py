"""The Krylov square root of the near-field block against its dense root.

Bars: the stopping rule bounds the last change of the iterate by tol, and
with condition numbers below about 20 (convergence factor
(sqrt(kappa) - 1) / (sqrt(kappa) + 1) < 0.64) the remaining error is at most
1 / (1 - 0.64) < 3 times that; the storage type adds its own rounding (the
product's bar in FP32, 1e-12 in FP64).
"""
import numpy as np
import pytest
import torch

import synth
from oracle import lanczos, rpy
from parity import FP32_NEAR_BAR_DENSE, check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def boxes():
    """n -> (positions with overlaps, L, dense M_r at eta = 1)."""
    made = {}

    def get(n):
        if n not in made:
            L = 22.0
            x = synth.uniform_positions(n, L, seed=70 + n)
            made[n] = (x, L, rpy.real_block_dense(x, L, 1.0, 1.0, 0.45, 7.0))
        return made[n]

    return get


@pytest.mark.parametrize("n", [2, 321])
@pytest.mark.parametrize("eta", [1.0, 3e-11, 5e10])
@pytest.mark.parametrize("precision,tol", [("fp64", 1e-3), ("fp64", 1e-12), ("mixed", 1e-5), ("fp32", 1e-3)])
def test_root_over_iterations_and_units(gpu_lib, boxes, precision, tol, eta, n):
    """From a few Krylov iterations to several tens, and with mobilities far
    from 1 (the tridiagonal solve scales its matrix)."""
    x, L, Mr = boxes(n)
    s = gpu_lib.Sampler(n, L, eta=eta, xi=0.45, rcut=7.0, grid=32, support=6, tol=tol, precision=precision)
    s.set_positions(torch.as_tensor(x, dtype=s.dtype, device="cuda"))
    z = synth.normals(11, (n, 3))
    y, st = s.real_sample(torch.as_tensor(z, dtype=s.dtype, device="cuda"))
    ref = lanczos.sqrt_apply(Mr, z.ravel()) / np.sqrt(eta)
    bar = 3 * tol + (1e-12 if precision == "fp64" else FP32_NEAR_BAR_DENSE)
    assert st.converged == 1
    check(y.double().cpu().numpy(), ref, bar, f"root n={n} {precision} eta={eta:g} iters {st.lanczos_iters}")
    s.close()
