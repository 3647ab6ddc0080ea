"""RMSNorm into operand pairs: rows of 1 to 8 whole 1024s in registers, other widths read twice."""
import pytest

import synth
from tests.test_gpu_edges import _gpu, _run

pytestmark = pytest.mark.gpu


# The bounds are those of the prefill attention's tile test: a cached element near the middle of two bf16
# values may be rounded to either.
@pytest.mark.parametrize("hidden", [1024, 3072, 5120, 6144, 7168, 8192, 1536, 9216])
def test_widths_of_whole_and_broken_1024s(hidden):
    _gpu()
    shape = synth.StageShape(f"norm-h{hidden}", 700 + hidden // 512, 1, hidden, 2, 2, 64, 128)
    for name, m in _run(shape, [("prefill", 5)], False, 700, 16):
        print(f"\n[{shape.name} {name}] {m}", flush=True)
        assert 1 - m["cos"] <= 1.2e-6 and m["max_abs"] <= 0.03 * m["rms_ref"], (name, m)
