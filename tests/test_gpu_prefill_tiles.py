"""Prefill attention over a bf16 cache: query blocks of 128 / G positions over tiles of 32 keys in a ring of
four stages."""
import pytest

import synth
from tests.test_gpu_edges import _gpu, _run

pytestmark = pytest.mark.gpu


# From one tile to past the ring, calls that end just before, at and past a tile and a query block, blocks
# whose wavefronts see different numbers of tiles (G = 1 and 2) and wavefronts without a row.  Bounds: a
# cached element that lies near the middle of two bf16 values may be rounded to either, 2^-8 of it in one
# of its row's dozens of keys; rms 3.7e-4 and 6.7e-3 in the largest element over the stages' shapes, four
# times that here.
@pytest.mark.parametrize("g, d", [(1, 64), (1, 128), (2, 128), (4, 64), (8, 128)])
def test_calls_around_the_tiles_and_the_ring(g, d):
    _gpu()
    shape = synth.StageShape(f"tiles-g{g}-d{d}", 400 + 10 * g + d // 64, 1, 256, 2 * g, 2, d, 512)
    plan = [("prefill", 31), ("prefill", 2), ("prefill", 31), ("append", 32), ("prefill", 33), ("prefill", 127),
            ("prefill", 129)]
    for name, m in _run(shape, plan, False, 400 + g, 400):
        print(f"\n[{shape.name} {name}] {m}", flush=True)
        assert 1 - m["cos"] <= 1.2e-6 and m["max_abs"] <= 0.03 * m["rms_ref"], (name, m)
