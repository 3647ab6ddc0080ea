"""Prefill over an fp32 cache: query blocks of 64 / G positions, tiles of 64 keys in two halves."""
import numpy as np
import pytest

import synth
from tests.harness import compute_stream, fp32_close, fp32_errors, weights_of
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


@pytest.mark.parametrize("held", [0, 230], ids=["one-range", "two-ranges"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_a_later_token_that_is_not_finite(bad, d, held):
    """Rows before a token whose K and V are not finite keep their bits; the rows that see it are not finite."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    shape, n, at = synth.StageShape(f"f32-nan-d{d}", 235 + d, 1, 256, 4, 2, d, 512), 70, 40
    w = weights_of(shape)(0)
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xF7, 1), (1, 1, n, shape.hidden)))
    spoilt = x.clone()
    spoilt[0, 0, at, 7] = bad
    kv = [torch.from_numpy(synth.normal_f32(synth.seed_of(0xF7, i), (1, held, 2, d))) for i in (2, 3)]
    out = []
    with compute_stream() as cs:
        cfg = P.config_for(shape, max_microbatches=2, max_batch=1, max_context=320, n_resident_max=1, kv_fp32=True,
                           compute_stream=cs.handle)
        h = P.stage_init(cfg)
        try:
            P.stage_load_layer(h, 0, w, 1)
            for mb, t in enumerate((x, spoilt)):
                if held:
                    P.stage_kv_append(h, mb, 0, held, *kv)
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


# Few query blocks over a longer context: the keys in ranges of 128, a workgroup each, and their merge.  Calls that
# end just before, at and past a range's end, blocks of which some rows see no key of the last range, and a range
# that begins in the middle of a call.
@pytest.mark.parametrize("g, d", [(1, 128), (2, 64), (4, 128), (8, 64), (8, 128)])
def test_calls_around_the_key_ranges(g, d):
    _gpu()
    shape = synth.StageShape(f"f32-ranges-g{g}-d{d}", 800 + 10 * g + d // 64, 1, 256, 2 * g, 2, d, 512)
    plan = [("append", 250), ("prefill", 5), ("prefill", 2), ("prefill", 29), ("append", 200), ("prefill", 26),
            ("prefill", 2), ("prefill", 40), ("append", 700), ("prefill", 3)]
    for name, m in _run(shape, plan, True, 95 + g, 1264):
        print(f"\n[{shape.name} {name}] {m}", flush=True)
        assert 1 - m["cos"] <= 5e-9 and m["max_abs"] <= 5e-4 * m["rms_ref"], (name, m)


def test_key_ranges_of_several_sequences():
    """Prompts' continuations at 20, 300 and 1000 held tokens, in one call and one by one: the same bits (a row's
    ranges are its own, one range gives o / l itself).  33 such sequences in one call, whose blocks are too many for
    ranges: the same values."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    shape, n, rows = synth.StageShape("f32-ranges-seqs", 899, 1, 256, 4, 2, 64, 512), 8, 33
    w = weights_of(shape)(0)
    held = [(20, 300, 1000)[i % 3] for i in range(rows)]
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xF6, 1), (rows, 1, n, shape.hidden)))
    kv = [torch.from_numpy(synth.normal_f32(synth.seed_of(0xF6, i), (1, 1000, 2, 64))) for i in (2, 3)]

    def run(calls):
        out = {}
        with compute_stream() as cs:
            cfg = P.config_for(shape, max_microbatches=rows, max_batch=1, max_context=1008, n_resident_max=1, kv_fp32=True,
                               compute_stream=cs.handle)
            h = P.stage_init(cfg)
            try:
                P.stage_load_layer(h, 0, w, 1)
                for mb in range(rows):
                    P.stage_kv_append(h, mb, 0, held[mb], *(t[:, :held[mb]].contiguous() for t in kv))
                for ids in calls:
                    xd = x[ids].cuda()
                    yd = torch.empty_like(xd)
                    torch.cuda.synchronize()
                    P.stage_prefill(h, ids, 1, n, xd, yd)
                    P.stage_sync(h)
                    out.update(zip(ids, yd.cpu().numpy()))
            finally:
                P.stage_destroy(h)
        return np.stack([out[i] for i in sorted(out)])

    one, three, all_ = run([[i] for i in range(rows)]), run([list(range(i, i + 3)) for i in range(0, rows, 3)]), run([list(range(rows))])
    assert np.array_equal(one, three)
    assert fp32_close(all_, one), fp32_errors(all_, one)
