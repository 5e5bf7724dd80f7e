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


# around the bound up to which one workgroup does an iteration's vector work
# (4096 particles)
@pytest.mark.parametrize("n", [4095, 4096, 4097])
@pytest.mark.parametrize("precision", ["mixed", "fp32", "fp64"])
def test_vector_work_by_size(gpu_lib, n, precision):
    """M_r^{1/2} applied twice is M_r: both products of one context, so the
    bar is the Krylov tolerance's and the storage type's alone."""
    L = (4 * np.pi * n / 0.6) ** (1 / 3)  # phi = 0.2
    x = synth.uniform_positions(n, L, seed=5)
    tol = 1e-10 if precision == "fp64" else 1e-5
    s = gpu_lib.Sampler(n, L, xi=0.7, rcut=4.5, grid=64, support=6, tol=tol, precision=precision)
    s.set_positions(torch.as_tensor(x, dtype=s.dtype, device="cuda"))
    z = torch.as_tensor(synth.normals(12, (n, 3)), dtype=s.dtype, device="cuda")
    y, st = s.real_sample(z)
    assert st.converged == 1
    again, _ = s.real_sample(y.clone())
    ref = s.real_matvec(z)
    # two roots: each 3 tol (see above) and the storage type's rounding
    bar = 6 * tol + (1e-12 if precision == "fp64" else 2 * FP32_NEAR_BAR_DENSE)
    check(again.double().cpu().numpy(), ref.double().cpu().numpy(), bar,
          f"root twice n={n} {precision} iters {st.lanczos_iters}")
    s.close()


@pytest.mark.parametrize("n", [321, 4097])
@pytest.mark.parametrize("eta,power", [(5e10, -55), (3e-11, 50)])
def test_start_vector_of_any_magnitude(gpu_lib, eta, power, n):
    """The FP32 sample of 2^k z is 2^k times that of z, bit for bit, wherever
    |z|^2 is in range: scaling by powers of two is exact.  |z|^2 mu0 leaves
    the range of FP32 here (mu0 = 1e-12 and 1.8e9)."""
    L = (4 * np.pi * n / 0.6) ** (1 / 3)  # phi = 0.2
    x = synth.uniform_positions(n, L, seed=6)
    s = gpu_lib.Sampler(n, L, eta=eta, xi=0.7, rcut=4.5, grid=64, support=6, tol=1e-3, precision="fp32")
    s.set_positions(torch.as_tensor(x, dtype=s.dtype, device="cuda"))
    z = torch.as_tensor(synth.normals(13, (n, 3)), dtype=s.dtype, device="cuda")
    y, st = s.real_sample(z)
    y2, st2 = s.real_sample(z * 2.0**power)
    print(f"n={n} eta={eta:g}: iterations {st.lanczos_iters}, of the scaled vector {st2.lanczos_iters}", flush=True)
    assert st.converged == st2.converged == 1 and st.lanczos_iters == st2.lanczos_iters
    assert torch.equal(y * 2.0**power, y2)
    s.close()


@pytest.mark.parametrize("precision,tol", [("mixed", 1e-5), ("fp32", 1e-5)])
def test_vector_work_over_many_particles(gpu_lib, precision, tol):
    """More than the 1024 workgroups of the vector kernels take at once (256
    particles each): the root applied twice, as above, on a lattice with a
    jitter of 0.15a that leaves spheres 2.1a apart (no nearly coincident ones,
    whose slow modes a 2-norm rule does not bound row by row)."""
    g = 67
    L = 2.4 * g
    x = 2.4 * np.stack(np.meshgrid(*[np.arange(g)] * 3, indexing="ij"), -1).reshape(-1, 3)
    n = len(x)
    assert n > 1024 * 256
    x = x + 0.15 * (2.0 * synth.uniform_positions(n, 1.0, seed=14) - 1.0)
    s = gpu_lib.Sampler(n, L, xi=0.7, rcut=4.5, grid=192, support=6, tol=tol, precision=precision)
    s.set_positions(torch.as_tensor(x, dtype=s.dtype, device="cuda"))
    z = torch.as_tensor(synth.normals(15, (n, 3)), dtype=s.dtype, device="cuda")
    y, st = s.real_sample(z)
    assert st.converged == 1
    again, _ = s.real_sample(y.clone())
    ref = s.real_matvec(z)
    check(again.double().cpu().numpy(), ref.double().cpu().numpy(), 6 * tol + 2 * FP32_NEAR_BAR_DENSE,
          f"root twice n={n} {precision} iters {st.lanczos_iters}")
    s.close()
