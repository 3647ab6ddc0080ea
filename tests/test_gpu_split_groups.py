"""Decode attention with a workgroup per group of four 64-key splits (calls with many partial outputs)
gives the bits of a workgroup per split."""
import numpy as np
import pytest

import synth
from tests.harness import compute_stream, weights_of
from tests.test_gpu_edges import _gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv", [8, 32], ids=["G8", "G2"])
def test_groups_of_splits_give_the_same_bits(hkv):
    """40 rows in one call (5 groups x 64 query heads x 40 rows: grouped) and 20 rows in each of two (half of
    that: not), the projections on the same engine; contexts end at and around the edges of a split and of a
    group, in every part of the last group."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    shape = synth.StageShape(f"groups-{hkv}", 600 + hkv, 1, 256, 64, hkv, 128, 512)
    w = weights_of(shape)(0)
    edges = [64 * u + e for u in range(1, 18) for e in (-1, 0)] + [1, 2, 257, 300, 1099, 1100]
    rows, most = len(edges), 1104
    assert rows == 40
    gen = torch.Generator(device="cuda")
    gen.manual_seed(7)
    kv = torch.empty((2, 1, most, hkv, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xFA, hkv), (rows, shape.hidden))).cuda()
    outs = []
    for parts in (1, 2):
        with compute_stream() as cs:
            cfg = P.config_for(shape, max_microbatches=rows, max_batch=1, max_context=most, n_resident_max=1,
                               compute_stream=cs.handle)
            h = P.stage_init(cfg)
            try:
                P.stage_load_layer(h, 0, w, 1)
                torch.cuda.synchronize()
                for m, n in enumerate(edges):   # with the step's own token n, at least 2
                    k, v = (t[:, :max(n - 1, 1)].contiguous().view(torch.int16) for t in kv)
                    P.stage_kv_append(h, m, 0, k.shape[1], k, v)
                y = torch.empty_like(x)
                torch.cuda.synchronize()
                per = rows // parts
                for i in range(0, rows, per):
                    P.stage_decode(h, list(range(i, i + per)), 1, x[i:i + per], y[i:i + per])
                P.stage_sync(h)
                outs.append(y.cpu().numpy())
            finally:
                P.stage_destroy(h)
    assert np.isfinite(outs[0]).all() and np.array_equal(outs[0], outs[1])


@pytest.mark.parametrize("hkv,rows,held,far", [(32, 2, 300, 2800), (8, 48, 780, 4900)], ids=["splits", "groups"])
def test_cache_reads_past_the_infinity_cache_give_the_same_bits(hkv, rows, held, far):
    """The sequences of a call alone on the stage (their cache is read plainly), and beside others with which
    it holds more than 256 MB (non-temporally); a workgroup per split and per group of splits."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    shape = synth.StageShape(f"stream-{hkv}", 640 + hkv, 1, 256, 64, hkv, 128, 512)
    w = weights_of(shape)(0)
    others = 6
    gen = torch.Generator(device="cuda")
    gen.manual_seed(9)
    k, v = (t.view(torch.int16) for t in torch.empty((2, 1, far, hkv, 128), dtype=torch.bfloat16, device="cuda").normal_(generator=gen))
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xFA, 99), (rows, shape.hidden))).cuda()
    outs = []
    for beside in (False, True):
        per_token = 2 * hkv * 128 * 2
        assert rows * (held + 1) * per_token < 256 << 20 < (rows * (held + 1) + others * far) * per_token
        with compute_stream() as cs:
            cfg = P.config_for(shape, max_microbatches=rows + others, max_batch=1, max_context=far + 16, n_resident_max=1,
                               compute_stream=cs.handle)
            h = P.stage_init(cfg)
            try:
                P.stage_load_layer(h, 0, w, 1)
                torch.cuda.synchronize()
                for m in range(rows):
                    P.stage_kv_append(h, m, 0, held, k[:, :held].contiguous(), v[:, :held].contiguous())
                for m in range(rows, rows + others if beside else rows):
                    P.stage_kv_append(h, m, 0, far, k, v)
                y = torch.empty_like(x)
                torch.cuda.synchronize()
                P.stage_decode(h, list(range(rows)), 1, x, y)
                P.stage_sync(h)
                outs.append(y.cpu().numpy())
            finally:
                P.stage_destroy(h)
    assert np.isfinite(outs[0]).all() and np.array_equal(outs[0], outs[1])
