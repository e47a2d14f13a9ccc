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
long host_made, host_freed, host_fail;
size_t host_live, host_most;
static void *host_block[256];
static size_t host_size[256];
int hipHostMalloc(void **p, size_t n, unsigned flags)
{
    static int (*f)(void **, size_t, unsigned);
    if (!f) f = (int (*)(void **, size_t, unsigned))real("hipHostMalloc");
    int e = f(p, host_fail ? (size_t)1 << 60 : n, flags);
    for (int k = 0; k < 256 && !e; ++k)
        if (!host_block[k]) {
            host_block[k] = *p; host_size[k] = n; host_live += n; ++host_made;
            if (host_live > host_most) host_most = host_live;
            break;
        }
    return e;
}
int hipHostFree(void *p)
{
    static int (*f)(void *);
    if (!f) f = (int (*)(void *))real("hipHostFree");
    for (int k = 0; k < 256 && p; ++k)
        if (host_block[k] == p) { host_block[k] = 0; host_live -= host_size[k]; ++host_freed; break; }
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
for call, u, n, models in ((hch.hch_build_levels_device, 256, 30000, 2), (hch.hch_build_levels_device, 64, 40000, 1), (hch.hch_build_levels, 256, 3000, 2)):
    args = (*batch(u, n, models), u)             # two models: a workgroup per table; one of 40 000 voxels: launches over memory
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
for args, first_ones in (((*batch(256, 30000), 256), 3), ((*batch(64, 40000, 1), 64), 4)):
    want, asked, used = build(args)
    used = [u - used[0] for u in used]
    held = [i for i in range(1, len(asked)) if used[i] >= sum(asked[:i])]        # with everything before them still there
    assert held == list(range(1, len(asked) - 2)) and max(used[-2:]) < sum(asked[:-2]) - asked[0], (asked, used)
    # theirs, the tables, (launches over memory: the failed pairs,) the first attempt; later ones depend on the attempts
    for k in range(first_ones):
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


HOST = r"""
made, freed, refused = (C.c_long.in_dll(hook, k) for k in ("host_made", "host_freed", "host_fail"))
pinned, most = (C.c_size_t.in_dll(hook, k) for k in ("host_live", "host_most"))

def check(lv, coords):
    # the host copies are perfect hashes of the positions (Eq.1)
    assert np.array_equal(lv.info(0).coords_host(), coords)
    for l in range(lv.n_levels):
        i = lv.info(l)
        H, T, Phi, V, pos = i.H_host(), i.T_host(), i.Phi_host().astype(np.int64), i.V_host(), i.coords_host().astype(np.int64)
        for v in range(len(i.mbar)):
            m, r, p = int(i.mbar[v]), int(i.rbar[v]), pos[i.N[v]:i.N[v + 1]]
            s = (p % m + Phi[i.R[v] + ((p[:, 0] % r) * r + p[:, 1] % r) * r + p[:, 2] % r]) % m
            slot = i.M[v] + (s[:, 0] * m + s[:, 1]) * m + s[:, 2]
            assert np.array_equal(H[slot], np.arange(len(p))) and np.array_equal(T[slot], p)
            assert np.all(V[i.M[v]:i.M[v + 1]] == v) and int((H[i.M[v]:i.M[v + 1]] >= 0).sum()) == len(p)
"""


def test_pinned_host_copies(tmp_path):
    """The pinned memory of the host copies passes on from one level set to the next.  Without pinned memory it is ordinary memory, and no
    error is left behind."""
    _child(tmp_path, HOST + r"""
args = (*batch(256, 30000), 256)
new = lambda: hch.hch_build_levels_device(*args, 5, stream=0)
some = [new() for _ in range(2)]
assert made.value == 4                           # two blocks each, the tables' and the offsets'
for lv in some: check(lv, args[0]); lv.free()
for k in range(4):
    lv = new(); check(lv, args[0])
    other = batch(256, 20000)
    lw = hch.hch_build_levels_device(*other, 256, 5, stream=0); check(lw, other[0]); check(lv, args[0])
    assert made.value == 4 and freed.value == 0, (k, made.value)
    lv.free(); lw.free()
refused.value = 1
some = [new() for _ in range(5)]                 # 3 more than there are blocks for
for lv in some: check(lv, args[0]); lv.free()
assert made.value == 4
refused.value = 0
lv = new(); check(lv, args[0]); lv.free()
""")


def test_pinned_host_memory_is_bounded(tmp_path):
    """256 MB of it at most, 128 MB while no level set lives; a level set with more than that takes none for its tables and does not empty the pool."""
    _child(tmp_path, HOST + r"""
args = (*batch(256, 30000, 40), 256)             # some 40 MB
new = lambda: hch.hch_build_levels_device(*args, 4, stream=0)
for k in range(4):
    some = [new() for _ in range(8)]
    assert pinned.value <= 256 << 20
    for lv in some: check(lv, args[0]); lv.free()
    assert pinned.value <= 128 << 20, k
assert most.value > 128 << 20 and freed.value > 0
counts = made.value, freed.value
large = (*batch(256, 30000, 160), 256)
lv = hch.hch_build_levels_device(*large, 4, stream=0); check(lv, large[0]); lv.free()
assert made.value <= counts[0] + 1 and freed.value <= counts[1] + 1, (made.value, freed.value, counts)      # its offsets' own block
""")


def test_host_copies_of_several_threads(tmp_path):
    """Blocks pass between level sets of three threads; nobody reads another's."""
    _child(tmp_path, HOST + r"""
import threading
wrong = []
def work(seed):
    try:
        for k in range(12):
            a = batch(256, 9000 + 4000 * ((seed + k) % 3) + seed)
            lv = hch.hch_build_levels_device(*a, 256, 4, stream=0)
            check(lv, a[0])
            lv.free()
    except BaseException as e:
        wrong.append(repr(e))
threads = [threading.Thread(target=work, args=(s,)) for s in range(3)]
for t in threads: t.start()
for t in threads: t.join()
assert not wrong and made.value > 0, wrong
""")
