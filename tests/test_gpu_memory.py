"""Contexts on a nearly full GPU: the FP64 pair coefficients are optional."""
import time

import numpy as np
import pytest
import torch

import synth
from parity import check

# A process that ran other GPU tests and then this one ended with a GPU fault
# whose cause is not known; the allocation order itself is tested without a GPU
# (test_context_memory.py).
pytestmark = [pytest.mark.gpu, pytest.mark.skip(reason="fills the GPU's memory; one of the tests of a process that "
                                                       "ended with a GPU fault of unknown cause")]

def test_fp64_context_without_room_for_coefficients(gpu_lib):
    """With room for everything but the FP64 pair coefficients a context is
    created without them, and its product agrees with that of a context that
    has them (the same closed forms, summed in the same order)."""
    n, L, rc = 30000, 60.0, 12.0
    x = torch.as_tensor(synth.uniform_positions(n, L, seed=41), device="cuda")
    v = torch.as_tensor(synth.normals(42, (n, 3)), device="cuda")

    def free():
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        return torch.cuda.mem_get_info()[0]

    def settled():  # (freed memory comes back some time after the call)
        last = -1
        for _ in range(100):
            f = free()
            if f == last:
                return f
            last = f
            time.sleep(0.05)
        return last

    def make():
        return gpu_lib.Sampler(n, L, xi=0.4, rcut=rc, grid=64, support=8, tol=1e-4, precision="fp64")

    s = make()  # (the first context of a process also brings up the library)
    s.close()
    before = settled()
    s = make()
    used = before - settled()
    s.set_positions(x)
    ref = s.real_matvec(v).cpu().numpy()
    s.close()
    slots = n * int(1.6 * n / L**3 * 4.18879 * rc**3 + 48)  # the library's estimate
    coef, rest = 16 * slots, used - 20 * slots  # 4 bytes per slot: the list itself
    assert coef > 300 << 20 and 20 << 20 < rest < coef
    # one array of that room, all other memory, then the room alone
    hold = torch.empty(used - rest // 2, dtype=torch.uint8, device="cuda")
    blockers = []
    for size in (1 << 34, 1 << 30, 1 << 26, 1 << 23):
        try:
            while True:
                blockers.append(torch.empty(size, dtype=torch.uint8, device="cuda"))
        except torch.OutOfMemoryError:
            pass
    print(f"context {used >> 20} MiB, coefficients {coef >> 20} MiB, room {hold.numel() >> 20} MiB, "
          f"free beside it {free() >> 20} MiB", flush=True)
    del hold
    settled()
    s = make()
    s.set_positions(x)
    got = s.real_matvec(v).cpu().numpy()
    s.close()
    del blockers
    torch.cuda.empty_cache()
    assert np.all(np.isfinite(got))
    check(got, ref, 1e-14, "M_r v without stored coefficients")
