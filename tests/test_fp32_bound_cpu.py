"""The bound of the fp32-cache comparisons (harness.fp32_close) separates what the kernels may leave from an
operand pair that lost its lo half, in each projection by itself.  The mistake is planted in the oracle."""
import numpy as np
import pytest

import synth
from oracle import stage_oracle
from tests.harness import fp32_close, fp32_errors, weights_of
from tests.test_gpu_few_rows import CUT_2_2_8, CUT_3_3_4


class _Rounded:
    """x @ this = the product with x rounded to `bits` mantissa bits."""

    def __init__(self, w, bits):
        self.w, self.bits = w, bits
        self.T = self

    def __rmatmul__(self, x):
        m, e = np.frexp(x.numpy())
        s = 2.0 ** self.bits
        return x.new_tensor(np.ldexp(np.round(m * s) / s, e)) @ self.w.T


@pytest.mark.parametrize("shape", [CUT_2_2_8, CUT_3_3_4], ids=["2-2-8", "3-3-4"])
@pytest.mark.parametrize("names", [("wq", "wk", "wv"), ("wo",), ("wg", "wu"), ("wd",)], ids=["qkv", "o", "gate-up", "down"])
def test_a_lost_lo_half_is_outside(monkeypatch, shape, names):
    x = synth.normal_f32(synth.seed_of(0xF4, 1), (24, shape.hidden))
    plain = stage_oracle.LayerWeights

    def forward(bits):
        class Planted(plain):
            def __init__(self, w):
                super().__init__(w)
                for n in names if bits else ():
                    setattr(self, n, _Rounded(getattr(self, n), bits))
        monkeypatch.setattr(stage_oracle, "LayerWeights", Planted)
        return np.asarray(stage_oracle.OracleStage(shape, weights_of(shape), kv_dtype="f32").forward([("s", x)])[0])

    want = forward(0)
    assert fp32_close(forward(16), want), fp32_errors(forward(16), want)      # a pair
    assert not fp32_close(forward(8), want), fp32_errors(forward(8), want)    # its hi half alone
