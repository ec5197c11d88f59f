"""The update kernel at the sizes where its launch shape changes, against the
oracle, bit for bit: around the last size of the latency-bound shape (256
threads a block) and the first of the bandwidth-bound one (one-wavefront
blocks of 256 elements under a residency limit), with ragged ends, parts that
begin inside a tile, a ring that wraps and spills, and a skipped step."""
import pytest

from test_gpu_parity import _run_window

pytestmark = pytest.mark.gpu

SHAPE_EDGE = 2 * 256 * 32 * 256  # elements: two rounds of all wave slots, a quad a lane


@pytest.mark.parametrize("n", [SHAPE_EDGE, SHAPE_EDGE + 1, SHAPE_EDGE + 256 + 7, SHAPE_EDGE + 2 * 256 - 4])
def test_update_shapes_same_bits(n):
    bounds = [0, 1_000_008, 2_097_152 + 248, n]
    _, stats, _ = _run_window(n, 3, bounds, seed=n % 97, ring_bytes=12 << 20, copy_bytes=4 << 20, dynamic=True,
                              inf_steps=(3,), late_plan=2)
    assert stats.bytes_spilled > 0 and stats.bytes_ring > 0 and stats.skipped == 1
