"""A call of one sequence carries that sequence's place in its kernels' arguments; a call of several
reads them from the metadata in device memory.  Both give a row the same bits."""
import numpy as np
import pytest

import synth
from tests.harness import compute_stream, weights_of
from tests.test_gpu_edges import _gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d, kv_fp32", [(64, False), (128, False), (128, True)])
def test_alone_and_together(d, kv_fp32):
    """Sequences of batch 2 in the second and third micro-batch (slots off 0), of different lengths: prefill
    of one token (the decode kernels) and of several, then decode across a cache block's and a split's edge."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    shape = synth.StageShape(f"one-d{d}", 500 + d, 2, 256, 4, 2, d, 512)
    w = weights_of(shape)
    H, lengths = shape.hidden, (15, 62)
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xF8, d), (2, 3, H)))
    hist = torch.from_numpy(synth.normal_f32(synth.seed_of(0xF9, d), (2, 62, H)))

    def run(together):
        out = []
        with compute_stream() as cs:
            cfg = P.config_for(shape, max_microbatches=3, max_batch=1, max_context=80, n_resident_max=2,
                               kv_fp32=kv_fp32, compute_stream=cs.handle)
            h = P.stage_init(cfg)
            try:
                for layer in range(2):
                    P.stage_load_layer(h, layer, w(layer), 1)
                xd, hd = x.cuda(), hist.cuda()
                torch.cuda.synchronize()
                for m, n in enumerate(lengths):   # alone in both runs: their lengths differ
                    for a, b in ((0, 1), (1, n)):
                        y = torch.empty((1, 1, b - a, H), device="cuda")
                        P.stage_prefill(h, [m + 1], 1, b - a, hd[m, a:b].reshape(1, 1, b - a, H).contiguous(), y)
                        P.stage_sync(h)
                        out.append(y.cpu().numpy().reshape(-1, H))
                for step in range(3):
                    y = torch.empty((2, 1, H), device="cuda")
                    xs = xd[:, step].reshape(2, 1, H).contiguous()
                    torch.cuda.synchronize()
                    if together:
                        P.stage_decode(h, [1, 2], 1, xs, y)
                    else:
                        for m in range(2):
                            P.stage_decode(h, [m + 1], 1, xs[m], y[m])
                    P.stage_sync(h)
                    out.append(y.cpu().numpy().reshape(-1, H))
                y = torch.empty((2, 1, 3, H), device="cuda")
                xs = xd.reshape(2, 1, 3, H).contiguous()
                torch.cuda.synchronize()
                if together:
                    P.stage_prefill(h, [1, 2], 1, 3, xs, y)
                else:
                    for m in range(2):
                        P.stage_prefill(h, [m + 1], 1, 3, xs[m], y[m])
                P.stage_sync(h)
                out.append(y.cpu().numpy().reshape(-1, H))
            finally:
                P.stage_destroy(h)
        return out

    for a, b in zip(run(False), run(True)):
        assert np.isfinite(a).all() and np.array_equal(a, b)
