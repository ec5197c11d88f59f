"""The update kernel at the sizes where its launch shape changes, against the
oracle, bit for bit: around the last size of the latency-bound shape (256
threads a block, or one launch for the whole step) and the first of the
bandwidth-bound one (one-wavefront blocks of 256 elements under a residency
limit), with ragged ends, parts that begin inside a tile, a ring that wraps and
spills, and a skipped step; the one-launch step in each of its forms, beside
the separate kernels in one context; and a small window step's copies."""
import pytest

from test_gpu_parity import _run_window

pytestmark = pytest.mark.gpu

SHAPE_EDGE = 2 * 256 * 32 * 256  # elements: two rounds of all wave slots, a quad a lane


@pytest.mark.parametrize("n", [SHAPE_EDGE - 5, SHAPE_EDGE, SHAPE_EDGE + 1, SHAPE_EDGE + 256 + 7,
                               SHAPE_EDGE + 2 * 256 - 4])
@pytest.mark.parametrize("late_plan", [1, 2])
def test_update_shapes_same_bits(n, late_plan):
    """late_plan 1 (HOST_WAIT) keeps the update a launch of its own on both
    sides of the edge; with 2 the step up to the edge is step_kernel's."""
    bounds = [0, 1_000_008, 2_097_152 + 248, n]
    _, stats, _ = _run_window(n, 3, bounds, seed=n % 97, ring_bytes=12 << 20, copy_bytes=4 << 20, dynamic=True,
                              inf_steps=(3,), late_plan=late_plan)
    assert stats.bytes_spilled > 0 and stats.bytes_ring > 0 and stats.skipped == 1


ROW = 256 * 256 * 4  # elements of a one-launch step with one quad a lane


@pytest.mark.parametrize("n", [1, 6, 1024, 1028, ROW, ROW + 1, 2 * ROW, 2 * ROW + 4, 4 * ROW + 3, 4 * ROW + 4])
@pytest.mark.parametrize("grad_dtype", ["bf16", "fp16"])
def test_one_launch_step_same_bits(n, grad_dtype):
    """Small spaces take the whole step in one launch: at the sizes where its
    tiling changes and the first size beyond it, with a skipped step, dynamic
    scaling, a pack into a ring that wraps and spills, and the norm."""
    K = 4 if n >= 64 else 1
    bounds = [0] + [n * k // K // 8 * 8 for k in range(1, K)] + [n]
    ring = max(256, n * 5 // 2 // 256 * 256)
    _, stats, _ = _run_window(n, K, bounds, seed=n % 89, ring_bytes=ring, copy_bytes=1 << 20, dynamic=True,
                              inf_steps=(3,) if K > 1 else (), late_plan=2, grad_dtype=grad_dtype)
    assert stats.skipped == (1 if K > 1 else 0)


@pytest.mark.parametrize("kw", [dict(check_overflow=False, grad_norm=False), dict(check_overflow=False),
                                dict(grad_norm=False, found_inf=[0.0, 1.0, 0.0]), dict(found_inf=[0.0, 1.0, 0.0]),
                                dict(grad_norm=False, with_weight=False)])
def test_one_launch_step_options(kw):
    """The step with and without something to exchange between its blocks."""
    n = 300_005
    _run_window(n, 3, [0, 100_000, 200_008, n], seed=61, ring_bytes=1 << 20, **kw)


@pytest.mark.parametrize("n", [1, 1027, 65_540, ROW + 1, 2 * ROW + 6, 4 * ROW + 3])
@pytest.mark.parametrize("grad_dtype", ["bf16", "fp16"])
def test_blocks_compute_the_partials_they_miss(n, grad_dtype, monkeypatch):
    """Every block of the one-launch step takes all partials for missing once
    and computes them itself: counted in the workspace (the third sync word, 64
    bytes in), with a skipped step, and every bit the oracle's."""
    import torch

    monkeypatch.setenv("GOCKPT_TEST_STEP_AGAIN", "1")
    K = 3 if n >= 64 else 1
    bounds = [0] + [n * k // K // 8 * 8 for k in range(1, K)] + [n]
    sess, stats, _ = _run_window(n, K, bounds, seed=n % 83, ring_bytes=1 << 20, dynamic=True,
                                 inf_steps=(2,) if K > 1 else (), late_plan=2, grad_dtype=grad_dtype)
    assert stats.skipped == (1 if K > 1 else 0)
    tile = 1024 if n // 4 <= ROW // 4 else (2048 if n // 4 <= 2 * ROW // 4 else 4096)
    tiles = max(1, -(-(n // 4 * 4) // tile))
    helped = int(sess.workspace[64:128].view(torch.int32)[2])
    assert helped >= K * tiles * tiles


def test_one_launch_step_beside_a_full_device():
    """The blocks of a one-launch step need not run together: with another
    kernel on all but a few of the device's places, those that run compute the
    partials of those that cannot start yet, and the step ends, with the
    oracle's bits, long before the other kernel does.  Whether a block finds
    one of the places left is the device's choice (its shader engines take
    blocks in turn, and both streams may share a hardware queue), so the bits
    are checked for every number of places, and that the step ran beside the
    other kernel for those where it could.  (That blocks compute each other's
    partials at all does not hang on the device's choice: the test above.)"""
    import time

    import numpy as np
    import torch

    import bench
    import oracle
    import synth
    from gpu_util import assert_bits_equal, load_state, to_device_grad16
    from paper_2511_07035_amd import Session

    n = ROW
    places = 8 * torch.cuda.get_device_properties(0).multi_processor_count  # blocks of four wavefronts
    cfg = oracle.AdamWConfig()
    p0 = synth.master_cpu(n, 71)
    ref = oracle.State(p0)
    L = bench.bench_lib()
    side = torch.cuda.Stream()
    beside = []
    with Session(n, ring_bytes=0) as sess:
        load_state(sess, p0, w=ref.w)
        for k, free_blocks in enumerate((64, 96, 192), 1):
            g = synth.grads_cpu(n, 71, k)
            to_device_grad16(sess, g)
            torch.cuda.synchronize()
            hog_end, step_end = torch.cuda.Event(), torch.cuda.Event()
            assert L.gockpt_bench_hog(side.cuda_stream, 100.0, places - free_blocks) == 0
            hog_end.record(side)
            time.sleep(0.01)  # it holds its places before the step is queued
            sess.step(cfg.lr)
            step_end.record(sess.compute)
            step_end.synchronize()
            beside.append(not hog_end.query())
            oracle.adamw_step(ref, g, cfg)
            torch.cuda.synchronize()
            p, m, v, w = sess.state_to_host()
            assert_bits_equal(p, ref.p, "master")
            assert_bits_equal(m, ref.m, "exp_avg")
            assert_bits_equal(v, ref.v, "exp_avg_sq")
            assert np.array_equal(w, ref.w)
    if not any(beside):
        pytest.skip("the device ran the step after the other kernel each time")


@pytest.mark.parametrize("case", ["ring", "spill", "no_ring", "host_wait"])
def test_small_step_copies_in_one_kernel(case):
    """A window step of at most 1 MiB sends its copies in one kernel, a larger
    one by DMA: a window whose steps pass that size midway, with a ring that
    holds a step, one that wraps and spills, none, and the HOST_WAIT plan with
    a skipped step; odd lengths at the end."""
    n = 262_147
    kw = dict(ring=dict(ring_bytes=4 << 20, late_plan=2), spill=dict(ring_bytes=700 << 10, late_plan=2),
              no_ring=dict(ring_bytes=0), host_wait=dict(ring_bytes=2 << 20, late_plan=1))[case]
    _, stats, _ = _run_window(n, 4, [0, 65_536, 131_072, 196_608, n], seed=83, copy_bytes=64 << 10, dynamic=True,
                              inf_steps=(3,), **kw)
    pieces = -(-stats.bytes_d2h // (64 << 10))
    assert 4 < stats.n_copies < pieces  # some steps as one kernel, some in 64 KiB copies


@pytest.mark.parametrize("kw", [dict(), dict(grad_dtype="fp16"), dict(grad_norm=False, found_inf=[0.0, 1.0, 0.0]),
                                dict(check_overflow=False, grad_norm=False, with_weight=False)])
@pytest.mark.parametrize("n", [5 * ROW - 1, 5 * ROW, 6 * ROW + 3, 6 * ROW + 4, 2_000_003])
def test_step_behind_a_prepass_or_alone(kw, n):
    """From 5 * 2^18 elements to 2^22 the launch that updates also reduces the
    prepass's partials, or has nothing to reduce; its shape changes at 6 * 2^18.
    Just below, the kernels are separate."""
    inf = dict(dynamic=True, inf_steps=(3,)) if kw.get("check_overflow", True) and "found_inf" not in kw else {}
    _, stats, _ = _run_window(n, 3, [0, 600_000, n * 7 // 10 // 8 * 8, n], seed=67, ring_bytes=6 << 20, late_plan=2, **inf, **kw)
    assert stats.skipped == (1 if inf or "found_inf" in kw else 0)


@pytest.mark.parametrize("buckets,n", [(1, 700_003), (7, 700_003), (512, 700_003), (600, 700_003),
                                       (3, 1_200_005)])
def test_step_behind_bucket_scans(buckets, n):
    """Up to 512 partials of bucket scans are reduced by the launch that
    updates, more by a finalize of their own; with a skipped step."""
    ends = [n * k // buckets // 8 * 8 for k in range(buckets)] + [n]
    _, stats, _ = _run_window(n, 4, [0, 200_000, 400_000, 600_000, n], seed=73, ring_bytes=4 << 20, dynamic=True,
                              inf_steps=(3,), scan_buckets=ends, per_step=False)
    assert stats.skipped == 1


@pytest.mark.parametrize("n", [2_383_872, 2_383_880, 3_000_003, 4_194_304])
@pytest.mark.parametrize("scan_first", [False, True])
def test_launch_forms_mixed_in_one_context(n, scan_first):
    """Plain steps end in one launch, HOST_WAIT and timed windows take the
    separate kernels; one context runs both in turn over one workspace.  At
    the sizes where the separate prepass, left to itself, would reach the
    one-launch step's counters: the step count, loss scale and growth tracker,
    the records, the device state and every restored checkpoint are the
    oracle's after each stretch."""
    import numpy as np

    import oracle
    import synth
    from gpu_util import assert_bits_equal, load_state, to_device_grad16
    from paper_2511_07035_amd import Session

    cfg = oracle.AdamWConfig(dynamic_scale=True, init_scale=1024.0, growth_interval=4)
    p0 = synth.master_cpu(n, 91)
    ref = oracle.State(p0, scale=1024.0)
    good = [synth.grads_cpu(n, 91, s, scale=1024.0) for s in (1, 2)]
    inf = synth.grads_cpu(n, 91, 3, scale=1024.0, plant_inf=True)
    K = 3
    bounds = [0, n // 3 // 8 * 8, 2 * n // 3 // 8 * 8, n]
    print(f"[case] n={n} scan_first={scan_first}", flush=True)
    with Session(n, dynamic_scale=True, init_scale=1024.0, growth_interval=4, ring_bytes=24 << 20,
                 timing=True) as sess:
        load_state(sess, p0, w=ref.w)
        steps = 0

        def step(g, scan=False):
            nonlocal steps
            steps += 1
            sess.backward_begin()
            to_device_grad16(sess, g)
            if scan:
                sess.scan_grads(0, n)
            sess.step(cfg.lr)
            return oracle.adamw_step(ref, g, cfg)

        def same(what):
            assert sess.scaler() == (ref.t, ref.scale, ref.tracker), what
            p, m, v, w = sess.state_to_host()
            assert_bits_equal(p, ref.p, f"master after {what}")
            assert_bits_equal(m, ref.m, f"exp_avg after {what}")
            assert_bits_equal(v, ref.v, f"exp_avg_sq after {what}")
            assert np.array_equal(w, ref.w), what

        def window(what, **kw):
            sess.begin_window(bounds, **kw)
            recs = [step(good[s % 2]) for s in range(K)]
            sess.drain()
            got = sess.records()
            for field in ("t", "skip", "scale_used"):
                assert list(got[field]) == [r[field][0] for r in recs], (what, field)
            assert list(got["window_step"]) == [1, 2, 3]
            out = (np.empty(n, np.float32), np.empty(n, np.float32), np.empty(n, np.float32), np.empty(n, np.uint16))
            meta = sess.restore(out=out)
            assert (meta.t, meta.scale, meta.tracker) == (ref.t, ref.scale, ref.tracker), what
            for a, b, name in zip(out, (ref.p, ref.m, ref.v, ref.w), ("master", "exp_avg", "exp_avg_sq", "w")):
                assert_bits_equal(a, b, f"restored {name}, {what}")
            same(what)

        def plain(what):
            for g in (good[0], inf, good[1]):
                step(g, scan=scan_first)
            same(what)

        plain("plain steps")
        window("the HOST_WAIT window", late_plan=1, timing=False)
        plain("plain steps after the HOST_WAIT window")
        window("the timed window", late_plan=2)
        plain("plain steps after the timed window")
        window("the untimed DEVICE_WAIT window", late_plan=2, timing=False)
        plain("plain steps after the untimed window")
    assert steps == 4 * 3 + 3 * K


@pytest.mark.parametrize("n", [1024, 65_536, 4 * ROW])
@pytest.mark.parametrize("kw", [dict(), dict(late_plan=1), dict(again="1")])
def test_norm_keeps_every_bit_of_the_block_sums(n, kw, monkeypatch):
    """Squares that one double holds exactly, 1 and 2^-46 in every tile of up
    to 4096 elements: their sum over one, 64 or 256 blocks is exact too, so
    whatever carries the blocks' sums has to keep all of a double -- also where
    the blocks compute each other's."""
    import numpy as np

    from gpu_util import to_device_grad16
    from paper_2511_07035_amd import Session

    kw = dict(kw)
    if "again" in kw:
        monkeypatch.setenv("GOCKPT_TEST_STEP_AGAIN", kw.pop("again"))
    bits = np.zeros(n, np.uint16)
    bits[0::4096] = 0x3F80  # 1
    bits[1023::4096] = 0x3400  # 2^-23
    with Session(n, ring_bytes=1 << 20) as sess:
        sess.begin_window([0, n], **kw)
        sess.backward_begin()
        to_device_grad16(sess, bits)
        sess.step(1e-4)
        sess.drain()
        ones, small = len(bits[0::4096]), len(bits[1023::4096])
        assert float(sess.records()["gnorm2"][0]) == ones + small * 2.0 ** -46
        sess.abort_window()


FORMS = [dict(late_plan=2), dict(late_plan=1), dict(late_plan=2, timing=True), dict(late_plan=2, knob=("GOCKPT_QUADS", "2")),
         dict(late_plan=2, found_inf=True)]


@pytest.mark.parametrize("n", [50_003, 4 * ROW + 3, 4 * ROW + 4])
def test_norm_of_a_huge_gradient_is_the_same_in_every_launch_form(n, monkeypatch):
    """A gradient whose square leaves fp32: up to the one-launch step's size the
    norm is the fp64 sum, above it the prepass's fp32 squares make it inf,
    whether the step is one launch or several."""
    import numpy as np
    import torch

    import synth
    from gpu_util import to_device_grad16
    from paper_2511_07035_amd import Session

    g = synth.grads_cpu(n, 97, 1)
    g[n // 2] = 0x60AD  # 1e20
    x = (g.astype(np.uint32) << 16).view(np.float32).astype(np.float64)
    want = float(np.sum(x * x))
    for form in FORMS:
        kw = dict(form)
        timing, knob, flag = kw.pop("timing", False), kw.pop("knob", None), kw.pop("found_inf", False)
        fi = torch.zeros(1, dtype=torch.float32, device="cuda") if flag else None
        with monkeypatch.context() as m:
            if knob:
                m.setenv(*knob)
            sess = Session(n, ring_bytes=4 << 20, timing=timing, found_inf=fi)
        with sess:
            sess.begin_window([0, n], **kw)
            sess.backward_begin()
            to_device_grad16(sess, g)
            sess.step(1e-4)
            sess.drain()
            rec = sess.records()[0]
            sess.abort_window()
        assert rec["skip"] == 0
        if n <= 4 * ROW + 3:
            assert abs(float(rec["gnorm2"]) - want) <= 1e-13 * want, form
        else:
            assert np.isinf(rec["gnorm2"]), form
