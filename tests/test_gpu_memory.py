"""Builds on the device when memory runs out.  A child process puts a hipMalloc of its own in front of the
runtime's (a shared object loaded before the library): it notes every size and, for the calls asked for, lets the
runtime fail a request of 2^60 bytes instead, so that the runtime's own error is left behind as in a real
shortage."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HOOK = r"""
#include <dlfcn.h>
#include <stddef.h>
long hook_calls, hook_fail_from = -1, hook_fail_to = -1;
size_t hook_sizes[256];
int hipMalloc(void **p, size_t n)
{
    static int (*real)(void **, size_t);
    if (!real) real = (int (*)(void **, size_t))dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY), "hipMalloc");
    long i = hook_calls++;
    if (i < 256) hook_sizes[i] = n;
    return real(p, i >= hook_fail_from && i < hook_fail_to ? (size_t)1 << 60 : n);
}
"""

CHILD = r"""
import ctypes as C, sys
hook = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
import paper_1803_11385_amd as hch
calls, first, last = (C.c_long.in_dll(hook, k) for k in ("hook_calls", "hook_fail_from", "hook_fail_to"))
sizes = (C.c_size_t * 256).in_dll(hook, "hook_sizes")

def batch(u, n, models=2):
    rng = np.random.default_rng(u + n)
    parts = [np.sort(rng.choice(64 ** 3, n, replace=False)) for _ in range(models)]
    q = np.concatenate(parts)
    return np.stack([q // 4096, q // 64 % 64, q % 64], 1).astype(np.int32) * (u // 64), np.arange(models + 1) * n

def build(args, fail=(), levels=5, call=hch.hch_build_levels_device):
    '''The level set or None where it ends with out of memory, and the sizes asked for.'''
    calls.value, (first.value, last.value) = 0, fail or (-1, -1)
    try:
        lv = call(*args, levels, stream=0)
    except hch.HchError as e:
        assert fail and e.status == 2, e
        lv = None
    assert calls.value > 0, "the hook is not in front of the runtime's function"
    return lv, list(sizes[:calls.value])

def same(a, b):
    for l in range(a.n_levels):
        x, y = a.info(l), b.info(l)
        # the tables depend on which bucket was faster, what they hold does not
        assert np.array_equal(x.N, y.N) and np.array_equal(x.coords_host(), y.coords_host()) and x.nbr_valid == y.nbr_valid

"""


def _child(tmp_path, code):
    src, lib = tmp_path / "hook.c", tmp_path / "hook.so"
    src.write_text(HOOK)
    subprocess.run(["gcc", "-O1", "-shared", "-fPIC", "-o", str(lib), str(src), "-ldl"], check=True)
    run = subprocess.run([sys.executable, "-c", CHILD + code, str(lib), ROOT], capture_output=True, text=True, timeout=100)
    assert run.returncode == 0, (run.stdout + run.stderr)[-3000:]


def test_allocation_failures(tmp_path):
    """Every allocation of a build fails once, alone and with all that follow.  The first one of a build on the device is
    for the checks of the positions: the host does them then.  What was out of memory leaves nothing behind for
    the next call, which succeeds."""
    _child(tmp_path, r"""
for call, n in ((hch.hch_build_levels_device, 30000), (hch.hch_build_levels, 3000)):
    args = (*batch(256, n), 256)
    want, asked = build(args, call=call)
    if call is hch.hch_build_levels_device:
        lv, _ = build(args, (0, 1))
        assert lv is not None, "an allocation that the build can do without"
        same(lv, want)
    for k in range(len(asked)):
        for until in (k + 1, 256):
            build(args, (k, until), call=call)
            same(build(args, call=call)[0], want)
""")
