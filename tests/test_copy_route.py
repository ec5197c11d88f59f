"""Which calls the host code makes (CPU): the library runs in a process of its
own over counting stand-ins for the HIP calls.

A small window step's copies go as one kernel that writes the pinned arena, or
as a copy call per range.  A copy call checks its range and returns an error;
the kernel's stores are not checked, so it may be chosen only when the whole
arena lies in the one pinned allocation.

A skipped step whose skip the host knows starts no blocks for what it leaves
alone."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

SETUP = r"""
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_set_pinned.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
fake.fake_launches.restype = fake.fake_memcpys.restype = ctypes.c_long
fake.fake_last_grid.restype = ctypes.c_uint
import paper_2511_07035_amd as g

keep = []
def at(nbytes):
    keep.append(np.zeros(nbytes + 4096, np.uint8))
    return (keep[-1].ctypes.data + 4095) // 4096 * 4096
def context(n, ring_bytes=0):
    cfg = g.gockpt_config()
    cfg.n = n
    cfg.master, cfg.exp_avg, cfg.exp_avg_sq, cfg.grad16 = at(4 * n), at(4 * n), at(4 * n), at(2 * n)
    cfg.beta1, cfg.beta2, cfg.eps, cfg.init_scale, cfg.check_overflow = 0.9, 0.999, 1e-8, 1.0, 1
    cfg.workspace, cfg.workspace_bytes = at(g.gockpt_workspace_bytes(n)), g.gockpt_workspace_bytes(n)
    cfg.compute_stream, cfg.copy_stream = 1 << 12, 1 << 13
    if ring_bytes:
        cfg.ring, cfg.ring_bytes = at(ring_bytes), ring_bytes
    return g.gockpt_create(cfg)
def arena_bytes(bounds):
    return int(g.gockpt_arena_layout_ex(len(bounds) - 1, np.asarray(bounds, np.int64), bounds[-1], 0)[0].total)
"""

ROUTES = r"""
bounds = [0, 2048, 4096]
ctx = context(4096)
total = arena_bytes(bounds)
block = at(total + 8192)
for name, start, length in (("whole", 0, total), ("inside", -4096, total + 8192), ("short", 0, total - 1),
                            ("half", 0, total // 2)):
    arena = block + 4096
    fake.fake_set_pinned(arena + start, length)
    c0, l0 = fake.fake_memcpys(), fake.fake_launches()
    g.gockpt_begin_window_ex(ctx, 2, bounds, arena, total)
    for _ in range(2):
        g.gockpt_backward_begin(ctx)
        g.gockpt_step(ctx, 1e-4)
    print(name, fake.fake_memcpys() - c0, fake.fake_launches() - l0, flush=True)
    g.gockpt_abort_window(ctx)
g.gockpt_destroy(ctx)
"""

SKIPS = r"""
bounds = [0, 3000000, 5000000, 6000003]
ring = int(sys.argv[2])
ctx = context(bounds[-1], ring)
total = arena_bytes(bounds)
arena = at(total)
fake.fake_set_pinned(arena, total)
for skip in (0, 1):
    fake.fake_fill_page(skip)  # the control page: the finalize's skip decisions
    g.gockpt_begin_window_ex(ctx, 3, bounds, arena, total, late_plan=g.GOCKPT_RING_HOST_WAIT)
    for s in range(3):
        g.gockpt_backward_begin(ctx)
        l0 = fake.fake_launches()
        g.gockpt_step(ctx, 1e-4)
        print(skip, fake.fake_launches() - l0, fake.fake_last_grid(), flush=True)
    g.gockpt_abort_window(ctx)
g.gockpt_destroy(ctx)
"""


def _drive(tmp_path, script, *args):
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("no C compiler")
    so = str(tmp_path / "fake_hip.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run([cc, "-std=gnu11", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                        os.path.join(ROOT, "tests", "host", "fake_hip.c"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([sys.executable, "-c", SETUP + script, so, *map(str, args)], capture_output=True, text=True,
                       cwd=ROOT, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    return [ln.split() for ln in r.stdout.splitlines()]


def test_kernel_copies_need_the_whole_arena_pinned(tmp_path):
    got = {w[0]: (int(w[1]), int(w[2])) for w in _drive(tmp_path, ROUTES)}
    assert got["whole"] == (0, 4) and got["inside"] == (0, 4), got  # a step and a copy kernel each, no copy call
    for name in ("short", "half"):  # the copy calls get the ranges, and with them their checks
        assert got[name][0] > 0 and got[name][1] == 2, got


def test_known_skip_starts_blocks_for_the_pack_only(tmp_path):
    """HOST_WAIT knows the skip before the update is launched: the launch then
    covers what the step packs of its part: all of it in a ring that holds it,
    64 elements in one of 256 bytes.  Blocks take 256 elements above 4.2e6 and
    1024 up to there."""
    whole = -(-6000003 // 256)
    for ring, packs in ((36 << 20, (3000000, 2000000, 1000003)), (256, (64, 64, 64))):
        rows = [(int(a), int(b), int(c)) for a, b, c in _drive(tmp_path, SKIPS, ring)]
        want = [(0, 3, whole)] * 3 + [(1, 3, -(-k // 1024)) for k in packs]  # prepass, finalize, update
        assert rows == want
