"""Prefill over an fp32 cache: query blocks of 64 / G positions, tiles of 64 keys in two halves."""
import numpy as np
import pytest

import synth
from tests.harness import compute_stream, weights_of
from tests.test_gpu_edges import _gpu, _run

pytestmark = pytest.mark.gpu


# calls that end just before, at and past a query block and a half tile, with and without keys held
# before them.  What differs from the float64 oracle: fp32 sums (1.2e-7 each, a few hundred of them in
# any order) and the projections' 16-bit operand pairs (2^-17 per factor): below 5e-5 of the row.
@pytest.mark.parametrize("g, d", [(1, 128), (2, 64), (4, 128), (8, 64)])
def test_calls_around_the_tiles(g, d):
    _gpu()
    shape = synth.StageShape(f"f32-g{g}-d{d}", 200 + 10 * g + d // 64, 1, 256, 2 * g, 2, d, 512)
    plan = [("prefill", 2), ("prefill", 29), ("prefill", 33), ("append", 63), ("prefill", 64), ("prefill", 65)]
    for name, m in _run(shape, plan, True, 90 + g, 272):
        print(f"\n[{shape.name} {name}] {m}", flush=True)
        assert 1 - m["cos"] <= 5e-9 and m["max_abs"] <= 5e-4 * m["rms_ref"], (name, m)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_later_token_that_is_not_finite(bad, d):
    """Rows before a token whose K and V are not finite keep their bits; the rows that see it are not finite."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    shape, n, at = synth.StageShape(f"f32-nan-d{d}", 235 + d, 1, 256, 4, 2, d, 512), 70, 40
    w = weights_of(shape)(0)
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xF7, 1), (1, 1, n, shape.hidden)))
    spoilt = x.clone()
    spoilt[0, 0, at, 7] = bad
    out = []
    with compute_stream() as cs:
        cfg = P.config_for(shape, max_microbatches=2, max_batch=1, max_context=80, n_resident_max=1, kv_fp32=True,
                           compute_stream=cs.handle)
        h = P.stage_init(cfg)
        try:
            P.stage_load_layer(h, 0, w, 1)
            for mb, t in enumerate((x, spoilt)):
                xd = t.cuda()
                yd = torch.empty_like(xd)
                torch.cuda.synchronize()
                P.stage_prefill(h, [mb], 1, n, xd, yd)
                P.stage_sync(h)
                out.append(yd.cpu().numpy()[0, 0])
        finally:
            P.stage_destroy(h)
    # (key by key adds in the order in which the matrix instruction takes its two keys)
    assert np.isfinite(out[0]).all() and np.array_equal(out[0][:at], out[1][:at])
    assert not np.isfinite(out[1][at:]).all(1).any()
