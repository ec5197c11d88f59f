"""What the steps of one context keep in its workspace, by the library's own
header (CPU): a program compiled against it lists the byte ranges a context
over n elements writes in any of its steps, and none may touch another.  A
context mixes launch forms (plain steps, timed and HOST_WAIT windows), so the
ranges of all of them count, and the one-launch step's counters must survive
the partials of a prepass with a finalize of its own."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
#include <stdio.h>
#include <stdlib.h>
#include "gockpt_internal.h"
using namespace gockpt;
int main(int argc, char** argv) {
    printf("bytes %zu limit %lld\n", kWsBytes, static_cast<long long>(kAfterMaxElems));
    for (int k = 1; k < argc; ++k) {
        const long long n = atoll(argv[k]);
        auto put = [&](const char* what, size_t at, size_t len) { printf("%lld %s %zu %zu\n", n, what, at, at + len); };
        put("scaler", kWsScalerOff, sizeof(DevScaler));
        put("records", kWsRecordsOff, (GOCKPT_MAX_K + 1) * sizeof(gockpt_step_record));
        put("partials", kWsPartialsOff, prepass_blocks_for(n) * sizeof(Partial));
        put("scans", kWsScanOff, 2 * kScanSlots * sizeof(Partial));
        if (n <= kAfterMaxElems) {
            put("sync", kWsSyncOff, sizeof(StepSync));
            put("counters", kWsArriveOff, kStepArriveLanes * sizeof(StepArrive));
        }
        if (n <= kStepMaxElems) put("slots", kWsSlotsOff, kWsArriveOff - kWsSlotsOff);
    }
}
"""


def _run(tmp_path, args):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    src, exe = tmp_path / "ws.cpp", tmp_path / "ws"
    src.write_text(PROGRAM)
    r = subprocess.run([cxx, "-std=c++17", "-Wall", f"-I{ROOT}/include", f"-I{ROOT}/paper_2511_07035_amd/csrc",
                        str(src), "-o", str(exe)], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    return subprocess.run([str(exe), *map(str, args)], capture_output=True, text=True, check=True).stdout.splitlines()


def test_ranges_of_one_context_are_disjoint(tmp_path):
    sizes = [1, 2048, 1_048_579, 1_048_580, 2_097_152, 2_383_872, 2_383_880, 3_000_003, 4_194_304, 4_194_305,
             1 << 33]
    head, *lines = _run(tmp_path, sizes)
    total = int(head.split()[1])
    by_n = {}
    for ln in lines:
        n, what, a, b = ln.split()
        by_n.setdefault(int(n), []).append((int(a), int(b), what))
    assert set(by_n) == set(sizes)
    for n, ranges in by_n.items():
        ranges.sort()
        for (a0, b0, w0), (a1, b1, w1) in zip(ranges, ranges[1:]):
            assert b0 <= a1, f"n={n}: {w0} [{a0}, {b0}) runs into {w1} [{a1}, {b1})"
        assert ranges[-1][1] <= total
    assert any(w == "counters" for _, _, w in by_n[4_194_304])
    assert not any(w == "counters" for _, _, w in by_n[4_194_305])


def test_workspace_size_is_the_documented_one():
    from paper_2511_07035_amd import gockpt_workspace_bytes
    for n in (0, 1, 1 << 20, 1 << 33):
        assert gockpt_workspace_bytes(n) == 311808  # 304.5 KiB
