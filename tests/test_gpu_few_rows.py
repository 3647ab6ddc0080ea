"""GEMMs of few rows, whose K is cut into ranges that run in different workgroups: short prefills, and
decode calls of more rows than the decode GEMVs take at once, against the oracle; and the bits of a
row, which may not depend on how many rows share the call (the cut depends on the matrix only)."""
import numpy as np
import pytest

import synth
from tests.harness import Scenario, compare, compute_stream, fp32_close, fp32_errors, run_gpu, run_oracle, weights_of

pytestmark = pytest.mark.gpu

TOL_ABS = 2e-2
TOL_COS = 0.9995

# Ranges per projection (QKV, O, down): 2, 2, 8; 3, 3, 4 (41 tiles of 64 as 11 + 11 + 11 + 8); 3, 8, 2
# with a QKV wide enough to run its 3 ranges in one workgroup; 4, 8, 8 with an O and a down
# projection that run 4 at a time.
CUT_2_2_8 = synth.StageShape("cut-1L-h1024", 70, 1, 1024, 8, 2, 128, 4096)
CUT_3_3_4 = synth.StageShape("cut-1L-h1536", 71, 1, 1536, 12, 12, 128, 2624)
CUT_WIDE_QKV = synth.StageShape("cut-1L-h2048", 72, 1, 2048, 64, 8, 128, 2048)
CUT_WIDE_O = synth.StageShape("cut-1L-h4096", 73, 1, 4096, 32, 8, 128, 4096)


def _gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _check(tag, sc):
    got, ref = run_gpu(sc), run_oracle(sc)
    m = compare(got.flat_out(), ref.flat_out(), got.flat_in(), ref.flat_in())
    print(f"\n[{tag}] {m}", flush=True)
    assert m["cos"] >= TOL_COS and m["cos_delta"] >= TOL_COS and m["max_abs"] <= TOL_ABS, m
    if sc.kv_fp32:
        assert fp32_close(got.flat_out(), ref.flat_out()), fp32_errors(got.flat_out(), ref.flat_out())


# 17, 32 | 33, 64: the edges of the 32- and 64-row tiles; ragged contexts around one 64-key split
@pytest.mark.parametrize("kv_fp32", [False, True])
@pytest.mark.parametrize("rows", [17, 32, 33, 64])
@pytest.mark.parametrize("shape", [CUT_2_2_8, CUT_3_3_4], ids=["2-2-8", "3-3-4"])
def test_decode_of_more_rows_than_the_gemvs_take(shape, rows, kv_fp32):
    """Decode steps of `rows` sequences in one call, at contexts 63 to 66 (one split, whose output the
    split kernel writes, then two and their merge)."""
    _gpu()
    wl = synth.Workload(f"{shape.name}-{rows}", 170, shape, n_mb=rows, batch=1, prefill=62, decode_steps=4)
    _check(f"{shape.name} {rows} rows fp32={kv_fp32}",
           Scenario(wl, prefill=62, decode_steps=4, kv_fp32=kv_fp32, calls="all"))


@pytest.mark.parametrize("kv_fp32", [False, True])
@pytest.mark.parametrize("tokens", [2, 31, 33, 64, 65, 128, 129, 300, 1024, 1025])
@pytest.mark.parametrize("shape", [CUT_2_2_8, CUT_3_3_4], ids=["2-2-8", "3-3-4"])
def test_short_prefills(shape, tokens, kv_fp32):
    _gpu()
    wl = synth.Workload(f"{shape.name}-p{tokens}", 171, shape, n_mb=1, batch=1, prefill=tokens, decode_steps=1)
    _check(f"{shape.name} prefill {tokens} fp32={kv_fp32}", Scenario(wl, prefill=tokens, decode_steps=1, kv_fp32=kv_fp32))


@pytest.mark.parametrize("shape,n_mb,tokens", [(CUT_WIDE_QKV, 4, 128), (CUT_WIDE_O, 4, 128), (CUT_WIDE_O, 8, 128), (CUT_WIDE_O, 8, 37),
                                               (CUT_3_3_4, 16, 5)],
                         ids=["qkv-3", "o-4", "o-4-wide", "37-rows", "5-rows"])
def test_rows_do_not_depend_on_the_call_they_share(shape, n_mb, tokens):
    """Prompts prefilled one per call (a range per workgroup) and all in one call of up to 512 rows
    (neighbouring ranges in one workgroup) give the same bits, and the oracle's values."""
    _gpu()
    wl = synth.Workload(f"{shape.name}-x{n_mb}", 172, shape, n_mb=n_mb, batch=1, prefill=tokens, decode_steps=1)
    one = run_gpu(Scenario(wl, prefill=tokens, decode_steps=1, calls="one"))
    sc = Scenario(wl, prefill=tokens, decode_steps=1, calls="all")
    together, ref = run_gpu(sc), run_oracle(sc)
    a = np.concatenate([o.reshape(-1, shape.hidden) for o in one.outputs[:n_mb]])
    b = together.outputs[0].reshape(-1, shape.hidden)
    assert np.array_equal(a, b)
    m = compare(b, np.asarray(ref.outputs[0]).reshape(-1, shape.hidden),
                together.inputs[0].reshape(-1, shape.hidden), ref.inputs[0].reshape(-1, shape.hidden))
    assert m["cos"] >= TOL_COS and m["max_abs"] <= TOL_ABS, m


# The two lines at which the order of a row's sums changes with the rows beside it: K is cut up to 1024 rows of
# a call of several tokens, and decode calls run on the GEMVs up to 16 rows and as GEMMs from 19.
@pytest.mark.parametrize("n_mb,tokens,steps", [(2, 600, 0), (24, 30, 2)], ids=["prefill-600-1200", "decode-1-24"])
def test_calls_on_either_side_of_a_line(n_mb, tokens, steps):
    """Micro-batches one per call and all in one call: values that both lie within the fp32 bound of the oracle's."""
    _gpu()
    shape = CUT_2_2_8
    wl = synth.Workload(f"{shape.name}-line{n_mb}", 173, shape, n_mb=n_mb, batch=1, prefill=tokens, decode_steps=max(steps, 1))
    for calls in ("one", "all"):
        sc = Scenario(wl, prefill=tokens, decode_steps=max(steps, 1), kv_fp32=True, calls=calls)
        _check(f"{shape.name} {n_mb} x {tokens}, {calls}", sc)


@pytest.mark.parametrize("zero_copy", [False, True])
def test_noalloc_and_host_weights_give_the_same_rows(zero_copy):
    """A 40-row decode call through stage_decode_noalloc (workspaces in the scratch array), and with
    the weights read in place from host memory, gives stage_decode's bits."""
    _gpu()
    import torch
    import paper_2512_21835_amd as P

    shape, rows = CUT_2_2_8, 40
    w = weights_of(shape)(0)
    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xF1, 1), (rows, shape.hidden)))
    k = torch.from_numpy(synth.normal_bf16(synth.seed_of(0xF2, 1), (1, 70, 2, 128)).view(np.int16))
    v = torch.from_numpy(synth.normal_bf16(synth.seed_of(0xF2, 2), (1, 70, 2, 128)).view(np.int16))

    def run(resident, fn):
        with compute_stream() as cs:
            cfg = P.config_for(shape, max_microbatches=rows, max_batch=1, max_context=80, n_resident_max=1,
                               zero_copy=not resident, compute_stream=cs.handle)
            h = P.stage_init(cfg)
            try:
                P.stage_load_layer(h, 0, w, 1 if resident else 0)
                for m in range(rows):
                    n = 40 + m % 31
                    P.stage_kv_append(h, m, 0, n, k[:, :n].contiguous(), v[:, :n].contiguous())
                xd = x.cuda()
                yd = torch.empty_like(xd)
                outs = []
                for _ in range(2):
                    fn(h, list(range(rows)), 1, xd, yd)
                    P.stage_sync(h)
                    outs.append(yd.cpu().numpy())
                return outs
            finally:
                P.stage_destroy(h)

    import paper_2512_21835_amd as P
    want = run(True, P.stage_decode)
    got = run(not zero_copy, P.stage_decode if zero_copy else P.stage_decode_noalloc)
    for a, b in zip(want, got):
        assert np.array_equal(a, b)


def _decode_calls(shape, w, rows, calls):
    """One decode step of each of `rows` sequences (fp32 cache; 40 to 70 tokens held), as `calls` group them."""
    import torch
    import paper_2512_21835_amd as P

    x = torch.from_numpy(synth.normal_f32(synth.seed_of(0xF3, 1), (rows, shape.hidden)))
    kv = [torch.from_numpy(synth.normal_f32(synth.seed_of(0xF3, i), (1, 70, shape.n_kv_heads, shape.head_dim))) for i in (2, 3)]
    with compute_stream() as cs:
        cfg = P.config_for(shape, max_microbatches=rows, max_batch=1, max_context=80, n_resident_max=1, kv_fp32=True,
                           compute_stream=cs.handle)
        h = P.stage_init(cfg)
        try:
            P.stage_load_layer(h, 0, w, 1)
            for m in range(rows):
                n = 40 + 7 * m % 31
                P.stage_kv_append(h, m, 0, n, *(t[:, :n].contiguous() for t in kv))
            y = {}
            for ids in calls:
                xd = x[ids].cuda()
                yd = torch.empty_like(xd)
                torch.cuda.synchronize()
                P.stage_decode(h, ids, 1, xd, yd)
                P.stage_sync(h)
                y.update(zip(ids, yd.cpu().numpy()))
            return y
        finally:
            P.stage_destroy(h)


# Widths off 128, and an ffn as wide as the hidden size (whose down projection keeps four rows in fp32).
OFF_128 = synth.StageShape("fp32-rows-1L-h192", 75, 1, 192, 3, 3, 64, 320)
SQUARE = synth.StageShape("fp32-rows-1L-h512", 76, 1, 512, 4, 2, 128, 512)


@pytest.mark.parametrize("shape,rows,last", [(CUT_2_2_8, 17, 1), (CUT_2_2_8, 18, 2), (CUT_2_2_8, 33, 1), (CUT_2_2_8, 50, 2),
                                             (SQUARE, 34, 2), (OFF_128, 18, 18), (OFF_128, 33, 33)],
                         ids=lambda p: getattr(p, "name", p))
def test_rows_that_run_in_fp32(shape, rows, last):
    """The rows past a multiple of 16 that the decode GEMVs multiply in fp32 keep their bits (those of the
    row alone) in calls whose other rows run as GEMMs on 16-bit pairs; so does every row of widths off 128."""
    _gpu()
    w = weights_of(shape)(0)
    ids = list(range(rows - last, rows))
    together = _decode_calls(shape, w, rows, [list(range(rows))])
    alone = _decode_calls(shape, w, rows, [[i] for i in ids])
    for i in ids:
        assert np.array_equal(together[i], alone[i]), i


@pytest.mark.parametrize("rows", [19, 20, 35, 36])
def test_square_o_projection_rows_in_fp32(rows):
    """A square O projection keeps the last three and four rows in fp32 as well, the others of their layer on
    pairs: with zero Q, K, V and gate weights the O projection's is the only product that counts."""
    _gpu()
    w = dict(weights_of(CUT_2_2_8)(0))
    for t in ("wq", "wk", "wv", "wg"):
        w[t] = np.zeros_like(w[t])
    ids = list(range(16 * (rows // 16), rows))
    together = _decode_calls(CUT_2_2_8, w, rows, [list(range(rows))])
    alone = _decode_calls(CUT_2_2_8, w, rows, [[i] for i in ids])
    for i in ids:
        assert np.array_equal(together[i], alone[i]), i
