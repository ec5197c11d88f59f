"""Which way a small window step's copies go (CPU): one kernel that writes the
pinned arena, or a copy call per range.  A copy call checks its range and
returns an error; the kernel's stores are not checked, so it may be chosen only
when the whole arena lies in the one pinned allocation.  The library's host
code runs in a process of its own over counting stand-ins for the HIP calls."""
import os
import shutil
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

DRIVER = r"""
import ctypes, sys
import numpy as np
fake = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
fake.fake_set_pinned.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
fake.fake_launches.restype = fake.fake_memcpys.restype = ctypes.c_long
import paper_2511_07035_amd as g

n, bounds = 4096, [0, 2048, 4096]
def at(nbytes):
    keep.append(np.zeros(nbytes + 4096, np.uint8))
    return (keep[-1].ctypes.data + 4095) // 4096 * 4096
keep = []
cfg = g.gockpt_config()
cfg.n = n
cfg.master, cfg.exp_avg, cfg.exp_avg_sq, cfg.grad16 = at(4 * n), at(4 * n), at(4 * n), at(2 * n)
cfg.beta1, cfg.beta2, cfg.eps, cfg.init_scale, cfg.check_overflow = 0.9, 0.999, 1e-8, 1.0, 1
cfg.workspace, cfg.workspace_bytes = at(g.gockpt_workspace_bytes(n)), g.gockpt_workspace_bytes(n)
cfg.compute_stream, cfg.copy_stream = 1 << 12, 1 << 13
ctx = g.gockpt_create(cfg)
lay, _ = g.gockpt_arena_layout_ex(2, np.asarray(bounds, np.int64), n, 0)
total = int(lay.total)
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


def test_kernel_copies_need_the_whole_arena_pinned(tmp_path):
    cc = shutil.which("gcc")
    if cc is None:
        pytest.skip("no C compiler")
    so = str(tmp_path / "fake_hip.so")
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    r = subprocess.run([cc, "-std=gnu11", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", f"-I{rocm}/include",
                        os.path.join(ROOT, "tests", "host", "fake_hip.c"), "-o", so], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([sys.executable, "-c", DRIVER, so], capture_output=True, text=True, cwd=ROOT, timeout=120)
    assert r.returncode == 0, (r.stdout + r.stderr)[-3000:]
    got = {w[0]: (int(w[1]), int(w[2])) for w in map(str.split, r.stdout.splitlines())}
    assert got["whole"] == (0, 4) and got["inside"] == (0, 4), got  # a step and a copy kernel each, no copy call
    for name in ("short", "half"):  # the copy calls get the ranges, and with them their checks
        assert got[name][0] > 0 and got[name][1] == 2, got
