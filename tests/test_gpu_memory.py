"""Builds on the device when memory runs out.  A child process puts a hipMalloc of its own in front of the
runtime's (a shared object loaded before the library): it notes every size, and what is allocated besides, and, for the
calls asked for, lets the runtime fail a request of 2^60 bytes instead, so that the runtime's own error is left behind as
in a real shortage."""
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
size_t hook_sizes[256], hook_live[256];
static size_t live, size_of[1024];
static void *block[1024];
static void *real(const char *name) { return dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY), name); }
int hipMalloc(void **p, size_t n)
{
    static int (*f)(void **, size_t);
    if (!f) f = (int (*)(void **, size_t))real("hipMalloc");
    long i = hook_calls++;
    if (i < 256) { hook_sizes[i] = n; hook_live[i] = live; }
    int e = f(p, i >= hook_fail_from && i < hook_fail_to ? (size_t)1 << 60 : n);
    for (int k = 0; k < 1024 && !e; ++k)
        if (!block[k]) { block[k] = *p; size_of[k] = n; live += n; break; }
    return e;
}
int hipFree(void *p)
{
    static int (*f)(void *);
    if (!f) f = (int (*)(void *))real("hipFree");
    for (int k = 0; k < 1024 && p; ++k)
        if (block[k] == p) { block[k] = 0; live -= size_of[k]; break; }
    return f(p);
}
"""

CHILD = r"""
import ctypes as C, sys
hook = C.CDLL(sys.argv[1], C.RTLD_GLOBAL)
sys.path.insert(0, sys.argv[2])
import numpy as np
import paper_1803_11385_amd as hch
calls, first, last = (C.c_long.in_dll(hook, k) for k in ("hook_calls", "hook_fail_from", "hook_fail_to"))
sizes, live = ((C.c_size_t * 256).in_dll(hook, k) for k in ("hook_sizes", "hook_live"))

def batch(u, n, models=2):
    rng = np.random.default_rng(u + n)
    parts = [np.sort(rng.choice(64 ** 3, n, replace=False)) for _ in range(models)]
    q = np.concatenate(parts)
    return np.stack([q // 4096, q // 64 % 64, q % 64], 1).astype(np.int32) * (u // 64), np.arange(models + 1) * n

def build(args, fail=(), levels=5, call=hch.hch_build_levels_device):
    '''The level set or None where it ends with out of memory, the sizes asked for and what was allocated then.'''
    calls.value, (first.value, last.value) = 0, fail or (-1, -1)
    try:
        lv = call(*args, levels, stream=0)
    except hch.HchError as e:
        assert fail and e.status == 2, e
        lv = None
    assert calls.value > 0, "the hook is not in front of the runtime's function"
    return lv, sizes[:calls.value], live[:calls.value]

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
    want, asked, _ = build(args, call=call)
    if call is hch.hch_build_levels_device:
        same(build(args, (0, 1))[0], want)
    for k in range(len(asked)):
        for until in (k + 1, 256):
            build(args, (k, until), call=call)
            same(build(args, call=call)[0], want)
""")


def test_memory_of_the_checks(tmp_path):
    """The checks of the positions on the device are no reason to run out of memory: where an allocation fails while
    theirs is held, the build does without it.  It is held until the tables are made, not for what comes after."""
    _child(tmp_path, r"""
args = (*batch(256, 30000), 256)
want, asked, used = build(args)
held = [i for i in range(1, len(asked)) if used[i] >= sum(asked[:i])]        # with everything before them still there
assert held == list(range(1, len(asked) - 2)) and max(used[-2:]) < sum(asked[:-2]) - asked[0], (asked, used)
for k in range(4):           # theirs, the tables, the failed pairs, the first attempt; later ones depend on the attempts
    lv, _, _ = build(args, (k, k + 1))
    assert lv is not None, k
    same(lv, want)
    assert build(args, (k, 256))[0] is None
""")


def test_few_voxels_in_a_large_grid(tmp_path):
    """A bit for each of 2^30 positions is not made for a few hundred voxels.  On both sides of the line (16 KB a voxel and
    4 MB a model: 9107 voxels) the levels are those of the host."""
    _child(tmp_path, r"""
for n in (300, 9106, 9107):
    args = (*batch(1024, n, 1), 1024)
    lv, asked, _ = build(args, levels=6)
    assert (max(asked) > 1 << 27) == (n == 9107), (n, asked)
    same(lv, build(args, levels=6, call=hch.hch_build_levels)[0])
""")
