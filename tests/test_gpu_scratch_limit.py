"""Sign step where device memory ends: what the Newton iteration alone can do is done.

A child process whose hipMalloc refuses whatever would take the process above a limit (a
library of a few lines in front of the runtime's) solves a tridiagonal sign of size 400: its
Newton matrices take 20.5 MB, the larger pole set of the rational step 52.4 MB.  Limits: the
Newton matrices fit and the pole set does not; the pole set fits, is refused by its estimate,
and leaves no room beside it.
"""
import os
import subprocess
import sys

import pytest

from gpu_util import say

pytestmark = pytest.mark.gpu

LIMITER = r"""
#define _GNU_SOURCE
#include <dlfcn.h>
#include <pthread.h>
#include <stddef.h>
static size_t limit = (size_t)-1, used;
static struct { void* p; size_t n; } held[65536];
static pthread_mutex_t mu = PTHREAD_MUTEX_INITIALIZER;
static void* real(const char* name) {
    void* h = dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD);
    return h ? dlsym(h, name) : NULL;
}
size_t limiter_used(void) { return used; }
void limiter_set(size_t n) { limit = n; }
int hipMalloc(void** p, size_t n) {
    static int (*f)(void**, size_t);
    pthread_mutex_lock(&mu);
    if (!f) f = (int (*)(void**, size_t))real("hipMalloc");
    int e = !f || used + n > limit ? 2 : f(p, n);
    for (int i = 0; e == 0 && i < 65536; ++i)
        if (!held[i].p) { held[i].p = *p; held[i].n = n; used += n; break; }
    pthread_mutex_unlock(&mu);
    return e;
}
int hipFree(void* p) {
    static int (*f)(void*);
    pthread_mutex_lock(&mu);
    if (!f) f = (int (*)(void*))real("hipFree");
    for (int i = 0; p && i < 65536; ++i)
        if (held[i].p == p) { used -= held[i].n; held[i].p = NULL; break; }
    int e = f ? f(p) : 1;
    pthread_mutex_unlock(&mu);
    return e;
}
"""

CHILD = r"""
import ctypes, sys
lim = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
lim.limiter_used.restype = ctypes.c_size_t
lim.limiter_set.argtypes = [ctypes.c_size_t]
sys.path[:0] = sys.argv[2:4]
import numpy as np
from gpu_util import host, rel
from oracle.sign import sign_schur
from paper_1604_08057_amd import Context
from test_gpu_rational_sign import _tridiagonal
k, gap, room = 400, float(sys.argv[4]), float(sys.argv[5])
ctx = Context((2, 2, 2, 2), -2.0, 0.0)
a, b = _tridiagonal(k, 0.1, np.random.default_rng(1))
_, info = ctx.tridiag_sign(a + 0.3j, b, b)     # the first pole set and the workspace are held
assert info.newton_iters == 1 and lim.limiter_used() > 6e6
a, b = _tridiagonal(k, gap, np.random.default_rng(2))
lim.limiter_set(lim.limiter_used() + int(room * 1e6))
c, info = ctx.tridiag_sign(a + 0.3j, b, b)
T = np.diag(a + 0.3j) + np.diag(b, -1) + np.diag(b, 1)
e = rel(host(c), sign_schur(T)[:, 0])
print(f"err {e:.2e} (tol {10 * k * 2.2e-16 * 2 * np.linalg.norm(T, 2) / gap:.1e}), steps {info.newton_iters}")
assert e < 10 * k * 2.2e-16 * 2 * np.linalg.norm(T, 2) / gap
assert info.newton_iters > 2
"""


@pytest.mark.parametrize("gap,room_mb", [(0.006, 16), (1e-5, 48)])
def test_sign_step_at_memory_limit(gap, room_mb, tmp_path):
    here = os.path.dirname(os.path.abspath(__file__))
    src, lib, child = tmp_path / "limiter.c", tmp_path / "liblimiter.so", tmp_path / "child.py"
    src.write_text(LIMITER)
    child.write_text(CHILD)
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", "-o", str(lib), str(src), "-ldl", "-lpthread"], check=True)
    r = subprocess.run([sys.executable, str(child), str(lib), os.path.dirname(here), here, str(gap), str(room_mb)],
                       capture_output=True, text=True, timeout=100)
    say(f"memory limit gap={gap}: {r.stdout.strip()} {r.stderr.strip()[-300:]}")
    assert r.returncode == 0
