"""Near-field list and product over box sizes and row lengths, against dense
M_r of the oracle.

Bars: 1e-12 in FP64 (sums of at most some hundred terms of order 1 at
2.2e-16 each); in FP32 storage the table and coordinate bar of the parity
tests for dense boxes.
"""
import numpy as np
import pytest
import torch

import synth
from oracle import rpy
from parity import FP32_NEAR_BAR_DENSE, check, cutoff_rows

pytestmark = pytest.mark.gpu

BAR = {"fp64": 1e-12, "fp32": FP32_NEAR_BAR_DENSE, "mixed": FP32_NEAR_BAR_DENSE}


def dev(x, s):
    return torch.as_tensor(np.ascontiguousarray(x), dtype=s.dtype, device="cuda")


# cells per side 2 (no LDS block: rows of global indices), 3, 4, 5 and 6
# (blocks of 1 to 4 cells, halos that wrap and halos that do not); rows
# around the 16 entries one pass of a row's lanes takes
@pytest.mark.parametrize("nc", [2, 3, 4, 5, 6])
@pytest.mark.parametrize("n", [1, 2, 17, 40, 333])
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_product_by_box_and_row_length(gpu_lib, precision, n, nc):
    rc = 4.6
    L = (nc + 0.05) * rc
    x = synth.uniform_positions(n, L, seed=31 * n + nc)
    x[0] = [L, -0.25 * L, 1.5 * L]  # on the face, below and above the box
    s = gpu_lib.Sampler(n, L, xi=0.7, rcut=rc, grid=64, support=6, precision=precision)
    s.set_positions(dev(x, s))
    v = synth.normals(3, (n, 3))
    ref = rpy.real_block_dense(x, L, 1.0, 1.0, 0.7, rc) @ v.ravel()
    w = s.real_matvec(dev(v, s)).double().cpu().numpy()
    check(w, ref, BAR[precision], f"M_r v n={n} cells {nc} {precision}")
    s.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
def test_rows_grow_past_their_capacity(gpu_lib, precision):
    """All spheres within one cutoff of each other: rows far above the mean
    density's estimate, so the list is reallocated and built again."""
    n, L, rc = 300, 30.0, 4.6
    x = synth.uniform_positions(n, L, seed=8)
    s = gpu_lib.Sampler(n, L, xi=0.7, rcut=rc, grid=64, support=6, precision=precision)
    s.set_positions(dev(x, s))
    y = 13.0 + 2.6 * synth.uniform_positions(n, 1.0, seed=9)
    s.set_positions(dev(y, s))
    v = synth.normals(4, (n, 3))
    ref = rpy.real_block_dense(y, L, 1.0, 1.0, 0.7, rc) @ v.ravel()
    check(s.real_matvec(dev(v, s)).double().cpu().numpy(), ref, BAR[precision], f"clustered M_r v {precision}")
    s.close()


def _pairs(x, L, rc):
    d = x[:, None, :] - x[None, :, :]
    d -= L * np.rint(d / L)
    r2 = (d * d).sum(-1)
    np.fill_diagonal(r2, np.inf)
    return r2


# runs of one segment (128 candidates) and of several, targets that stage more
# hits than a round takes, tiles of 1 to 16 targets, empty columns
@pytest.mark.parametrize("n,L,spread", [(5, 40.0, 40.0), (900, 40.0, 40.0), (4000, 32.0, 32.0), (1500, 40.0, 9.0),
                                         (700, 40.0, 3.0)])
@pytest.mark.parametrize("krep", [0.0, 3.0])
def test_list_counts(gpu_lib, n, L, spread, krep):
    """Pair count and largest row of the LDS list against all pairs of the same
    FP32 positions.  A pair may fall on either side only if its distance is
    within the rounding of the staged coordinates (a few cells, L/2 at most:
    4 L 2^-24 covers the two roundings of each coordinate difference)."""
    rc = 5.0
    x = (0.3 * L + spread * synth.uniform_positions(n, 1.0, seed=n)).astype(np.float32)
    s = gpu_lib.Sampler(n, L, xi=0.65, rcut=rc, grid=64, support=6, precision="fp32", tol=1e-3, kT=0.0)
    pos = torch.as_tensor(x, device="cuda")
    st = s.bd_step(pos, 1, 1, 1e-6, krep=krep)
    w = np.mod(x.astype(np.float64), L)
    r2 = _pairs(w, L, rc)
    eps = 4 * L * 2.0**-24
    lo, hi = r2 <= (rc - eps) ** 2, r2 <= (rc + eps) ** 2
    print(f"n={n} spread={spread}: pairs {st.neighbor_pairs}, {lo.sum()} to {hi.sum()}; largest row "
          f"{st.max_neighbors}, {lo.sum(1).max()} to {hi.sum(1).max()}; block edge {st.lds_block_edge}", flush=True)
    assert st.lds_block_edge > 0
    assert lo.sum() <= st.neighbor_pairs <= hi.sum()
    assert lo.sum(1).max() <= st.max_neighbors <= hi.sum(1).max()
    s.close()


@pytest.mark.parametrize("corner", [0.0, 1.0])
def test_largest_halo_in_first_or_last_block(gpu_lib, corner):
    """The halo capacity is the largest over all blocks: a cluster in the
    first or in the last of 2197 blocks of a nearly empty box (more blocks
    than the wavefronts that walk them), rows of M_r v against brute force."""
    rc, L, xi = 4.0, 209.0, 0.56
    g = np.arange(7) * 2.05
    c = np.stack(np.meshgrid(g, g, g, indexing="ij"), -1).reshape(-1, 3)
    c = 0.5 + c if corner == 0.0 else L - 0.5 - c
    rest = np.random.default_rng(3300).uniform(0.2 * L, 0.8 * L, (40, 3))
    x = np.concatenate([rest, c])
    n = len(x)
    s = gpu_lib.Sampler(n, L, xi=xi, rcut=rc, grid=256, support=8, tol=1e-6, precision="fp32")
    s.set_positions(dev(x, s))
    v = synth.normals(3301, (n, 3))
    w = s.real_matvec(dev(v, s)).double().cpu().numpy()
    rows = np.arange(n)
    check(w, rpy.real_matvec_rows(x, v, rows, L, 1.0, 1.0, xi, rc), FP32_NEAR_BAR_DENSE, f"corner {corner}",
          skip_rows=cutoff_rows(x, L, rc, rows))
    s.close()


def test_list_follows_changing_halos(gpu_lib):
    """One sampler given positions whose largest halo stays, grows past the
    room kept for it (a quarter of the spheres drawn together), shrinks again
    and, in between, holds a position that is not finite: rows of M_r v
    against brute force each time, the refusal as such, and the first
    positions' product reproduced bit for bit."""
    n, rc, L, xi = 3000, 4.6, 46.5, 0.7
    x0 = synth.uniform_positions(n, L, seed=3400)
    x1 = x0 + 0.3 * synth.normals(3401, (n, 3))
    x2 = x0.copy()
    x2[: n // 4] *= 0.25
    s = gpu_lib.Sampler(n, L, xi=xi, rcut=rc, grid=64, support=6, tol=1e-6, precision="fp32")
    v = synth.normals(3402, (n, 3))
    rows = np.arange(0, n, 7)
    first = None
    for k, x in enumerate([x0, x1, x2, None, x2, x0, x0]):
        if x is None:
            bad = x0.copy()
            bad[5, 1] = np.nan
            with pytest.raises(gpu_lib.PSEError):
                s.set_positions(dev(bad, s))
            continue
        s.set_positions(dev(x, s))
        w = s.real_matvec(dev(v, s)).double().cpu().numpy()
        check(w[rows], rpy.real_matvec_rows(x, v, rows, L, 1.0, 1.0, xi, rc), FP32_NEAR_BAR_DENSE, f"positions {k}",
              skip_rows=cutoff_rows(x, L, rc, rows))
        if k == 5:
            first = w
    assert np.array_equal(w, first)
    s.close()
