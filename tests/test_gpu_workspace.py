"""The workspace of the partial products of projections cut in K: a lane has what decode calls need from
the start, and it grows with the rows of the calls."""
import numpy as np
import pytest

import synth
from tests.harness import compute_stream, weights_of
from tests.test_gpu_edges import _gpu

pytestmark = pytest.mark.gpu

WIDE = synth.StageShape("workspace-1L-h4096", 77, 1, 4096, 32, 8, 128, 14336)
GROWN = synth.StageShape("workspace-1L-h1024", 78, 1, 1024, 8, 2, 128, 4096)


def test_lanes_take_what_decode_calls_need():
    """Device memory of three more lanes of an 8B-shaped stage that has run nothing."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    streams = [torch.cuda.Stream().cuda_stream for _ in range(4)]

    def held(n_lanes):
        cfg = P.config_for(WIDE, max_microbatches=1, max_batch=1, max_context=16, n_resident_max=1, n_lanes=n_lanes,
                           compute_stream=streams[0], lane_streams=streams[:n_lanes])
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        h = P.stage_init(cfg)
        try:
            return before - torch.cuda.mem_get_info()[0]
        finally:
            P.stage_destroy(h)

    held(4)   # (what the first stage of a process takes once)
    per_lane = (held(4) - held(1)) / 3
    partials = 8 * 2 * 16 * WIDE.ffn * 4   # 14.7 MB; 101 MB with those of 1024 rows
    assert per_lane <= partials + 8 * 2**20, per_lane


def test_calls_after_the_workspace_grew():
    """Prefills of more and of fewer rows in any order, and a decode, on one stage: the bits of each on a stage
    of its own (8 ranges of the down projection, 8 parts of them up to some 700 rows)."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    w = weights_of(GROWN)(0)
    calls = [37, 65, 700, 130, 1024, 64, 1]
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xFB, 1), (max(calls), GROWN.hidden)))

    def run(which):
        out = []
        with compute_stream() as cs:
            cfg = P.config_for(GROWN, max_microbatches=len(calls), max_batch=1, max_context=1040, n_resident_max=1,
                               compute_stream=cs.handle)
            h = P.stage_init(cfg)
            try:
                P.stage_load_layer(h, 0, w, 1)
                for mb in which:
                    n = calls[mb]
                    xd = x[:n].cuda().reshape(1, 1, n, GROWN.hidden)
                    yd, zd = torch.empty_like(xd), torch.empty((1, 1, GROWN.hidden), device="cuda")
                    torch.cuda.synchronize()
                    P.stage_prefill(h, [mb], 1, n, xd, yd)
                    P.stage_decode(h, [mb], 1, yd[:, :, -1].contiguous(), zd)
                    P.stage_sync(h)
                    out.append((yd.cpu().numpy(), zd.cpu().numpy()))
            finally:
                P.stage_destroy(h)
        return out

    for mb, got in enumerate(run(range(len(calls)))):
        for a, b in zip(got, run([mb])[0]):
            assert np.isfinite(a).all() and np.array_equal(a, b), calls[mb]
