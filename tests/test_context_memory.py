"""What a context allocates, and in which order, on a stand-in for the HIP
runtime's memory calls with a fixed budget (host only, no GPU): the FP64 pair
coefficients are optional and must never take the room of a required buffer."""
import json
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

STAND_IN = r"""
#include <cstdlib>
#include <cstring>
#include <cstdint>
// 64 bytes before each block hold its size; memory is never written past them
static size_t used = 0, budget = 0;
extern "C" {
void set_budget(size_t b) { budget = b; }
size_t get_used() { return used; }
int hipMalloc(void **p, size_t n) {
  if (used + n > budget) return 2;
  char *q = (char *)std::malloc(n + 64);
  if (!q) return 2;
  std::memcpy(q, &n, sizeof n);
  used += n;
  *p = q + 64;
  return 0;
}
int hipFree(void *p) {
  if (!p) return 0;
  size_t n;
  std::memcpy(&n, (char *)p - 64, sizeof n);
  used -= n;
  std::free((char *)p - 64);
  return 0;
}
int hipMemGetInfo(size_t *f, size_t *t) { *f = budget - used; *t = budget; return 0; }
int hipHostMalloc(void **p, size_t n, unsigned) { *p = std::malloc(n); return *p ? 0 : 2; }
int hipHostFree(void *p) { std::free(p); return 0; }
int hipMemcpy(void *d, const void *s, size_t n, int) { std::memcpy(d, s, n); return 0; }
int hipMemset(void *d, int v, size_t n) { std::memset(d, v, n); return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int *d) { *d = 0; return 0; }
int hipSetDevice(int) { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipStreamCreateWithFlags(void **s, unsigned) { *s = (void *)8; return 0; }
int hipStreamDestroy(void *) { return 0; }
int hipEventCreate(void **e) { *e = (void *)8; return 0; }
int hipEventCreateWithFlags(void **e, unsigned) { *e = (void *)8; return 0; }
int hipEventDestroy(void *) { return 0; }
}
"""

# (status, bytes held) of a context, or of a batch of `replicas`, at a budget
DRIVER = r"""
import ctypes, json, sys
shim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)  # before the library: its calls go here
sys.path.insert(0, sys.argv[2])
import paper_1611_09322_amd as pse
lib = ctypes.CDLL(pse.LIB_PATH)
shim.get_used.restype = ctypes.c_size_t
VP = ctypes.c_void_p
out = []
for budget, replicas, kw in json.loads(sys.argv[3]):
    shim.set_budget(ctypes.c_size_t(budget))
    p = (pse.Params * max(replicas, 1))(*[pse.make_params(**kw)] * max(replicas, 1))
    h = VP()
    if replicas:
        st = lib.pse_batch_create(p, replicas, None, ctypes.byref(h))
    else:
        st = lib.pse_create(p, None, ctypes.byref(h))
    held = shim.get_used()
    if st == 0:
        (lib.pse_batch_destroy if replicas else lib.pse_destroy)(h)
    out.append((st, held, shim.get_used()))
print(json.dumps(out))
"""

N, L, RC = 3000, 28.0, 12.0
KW = dict(n=N, box=L, xi=0.4, rcut=RC, grid=32, support=8, precision="fp64")
HUGE = 1 << 40
OOM = -2


@pytest.fixture(scope="module")
def create(tmp_path_factory):
    d = tmp_path_factory.mktemp("standin")
    src, so = d / "standin.cpp", d / "standin.so"
    src.write_text(STAND_IN)
    subprocess.check_call(["g++", "-O1", "-shared", "-fPIC", "-o", str(so), str(src)])

    def run(*cases):
        r = subprocess.run([sys.executable, "-c", DRIVER, str(so), ROOT, json.dumps(cases)], capture_output=True,
                           text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        got = json.loads(r.stdout.splitlines()[-1])
        assert all(left == 0 for _, _, left in got)  # destroyed, or refused without a trace
        return [(st, held) for st, held, _ in got]

    return run


def coef_bytes():
    expect = N / L**3 * 4.18879020478639 * RC**3
    cap = (min(int(1.6 * expect + 48), N) + 7) & ~7
    return 16 * cap * N


def test_coefficients_come_last(create):
    coef = coef_bytes()
    (st, full), = create((HUGE, 0, KW))
    need = full - coef
    assert st == 0 and need > 0
    # required buffers alone; one byte less; room for the coefficients but one byte; up to half of the rest
    cases = [need, need - 1, need + coef - 1, need + coef, need + 2 * coef - 1, need + 2 * coef]
    got = create(*[(b, 0, KW) for b in cases])
    assert got == [(0, need), (OOM, 0), (0, need), (0, need), (0, need), (0, full)]


def test_batch_takes_them_after_all_replicas(create):
    coef = coef_bytes()
    (_, full), = create((HUGE, 0, KW))
    need = full - coef
    got = create((3 * need, 3, KW), (3 * need - 1, 3, KW), (3 * need + 2 * coef, 3, KW), (HUGE, 3, KW))
    assert got == [(0, 3 * need), (OOM, 0), (0, 3 * need + coef), (0, 3 * full)]


@pytest.mark.parametrize("precision", ["fp32", "mixed"])
def test_no_coefficients_in_fp32_storage(create, precision):
    kw = dict(KW, precision=precision)
    (st, full), = create((HUGE, 0, kw))
    assert st == 0
    assert create((full, 0, kw), (full - 1, 0, kw)) == [(0, full), (OOM, 0)]
