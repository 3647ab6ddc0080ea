"""K/V moves between the paged cache and device buffers: whole 16-byte chunks where the buffers start
on a 16-byte boundary, single elements where they do not, are byte-exact and agree."""
import pytest

import synth
from tests.harness import compute_stream

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kv_fp32", [False, True], ids=["bf16", "fp32"])
@pytest.mark.parametrize("hkv, d, layers, held, n", [
    (2, 64, 1, 1, 1),       # one head vector per chunk group, far less than a workgroup's share
    (3, 128, 2, 33, 17),    # heads that are no power of two, a tail over two cache blocks
    (8, 128, 3, 100, 65),   # a last workgroup that is partly filled
])
def test_device_buffers_of_any_alignment(kv_fp32, hkv, d, layers, held, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2512_21835_amd as P

    shape = synth.StageShape("kv-copy", 298, layers, 256, hkv, hkv, d, 64)
    kind = torch.int32 if kv_fp32 else torch.int16   # bit patterns of the elements

    def buffer(tokens, off):   # [layers][tokens][hkv][d], `off` elements past a 16-byte boundary
        t = torch.zeros(layers * tokens * hkv * d + off, dtype=kind, device="cuda")
        return t[off:].view(layers, tokens, hkv, d)

    with compute_stream() as cs:
        cfg = P.config_for(shape, max_microbatches=2, max_batch=1, max_context=held + 16, n_resident_max=layers,
                           kv_fp32=kv_fp32, compute_stream=cs.handle)
        h = P.stage_init(cfg)
        try:
            src = [torch.randint(-30000, 30000, (layers, held, hkv, d), dtype=kind, device="cuda") for _ in range(2)]
            for seq, off in ((0, 0), (1, 1)):   # one sequence through each path
                k, v = buffer(held, off), buffer(held, off)
                k.copy_(src[0]), v.copy_(src[1])
                torch.cuda.synchronize()
                P.stage_kv_append(h, seq, 0, held, k, v)
            for seq in (0, 1):
                for off in (0, 1):
                    k, v = buffer(n, off), buffer(n, off)
                    torch.cuda.synchronize()
                    P.stage_kv_export_tail(h, seq, 0, n, k, v, False)
                    assert torch.equal(k, src[0][:, held - n:]) and torch.equal(v, src[1][:, held - n:]), (seq, off)
        finally:
            P.stage_destroy(h)
