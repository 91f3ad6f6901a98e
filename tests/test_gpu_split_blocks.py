"""Prefill calls with fewer query blocks than CUs: their blocks are cut into
parts of the key range (at least 16 tile visits each) whose states a second
kernel merges.  Checked against the fp64 oracle, and the paged chunk against
the dense one bit for bit (both are cut alike)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2607_07740_amd import api, synth
from parity_util import assert_close, say, to_dev, to_f64

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rescale", [None, 3.0])
@pytest.mark.parametrize("P,n,B,Hkv,g,w_pre,w0", [
    (4000, 64, 1, 1, 4, 1024, 300),    # one block, parts on both sides of the view switch
    (3000, 300, 2, 2, 1, 700, 4000),   # the band covers every key: no remote part
    (2500, 1, 1, 2, 8, 8192, 100),     # one query, G = 1: the vanilla kernel
    (5003, 129, 1, 2, 2, 600, 0),      # ragged ends, w_local = 0
    (0, 4100, 1, 1, 8, 2048, 500),     # a whole prefill whose blocks differ in length
    (1100, 40, 1, 1, 1, 512, 64),      # too short to cut: one part
])
def test_split_blocks(P, n, B, Hkv, g, w_pre, w0, rescale):
    """With the rescale bound lowered to 2^3 every part runs the checked pass,
    whose parts carry different softmax references into the merge."""
    T, Hq, page = P + n, g * Hkv, 64
    q, k, v = synth.prefill_inputs(B, Hq, Hkv, T, 128, seed=T + g, outlier_channels=8)
    pages = (T + page - 1) // page
    pad = [(0, 0), (0, pages * page - T), (0, 0), (0, 0)]
    kp, vp = (np.pad(x, pad, constant_values=0x7FC0) for x in (k, v))  # NaN past the sequence
    kd, vd = to_dev(kp), to_dev(vp)
    table = torch.arange(B * pages, dtype=torch.int32, device="cuda").view(B, pages)
    kw = dict(q_start=P, w_pretrained=w_pre, w_local=w0, want_lse=True)
    old = api.debug_prefill_rescale_log2(rescale) if rescale else None
    try:
        say("split blocks P=%d n=%d g=%d rescale=%s" % (P, n, g, rescale))
        out, lse = api.prefill_chunk(to_dev(q[:, P:]), kd, vd, **kw)
        say("split blocks, paged")
        pg, pl = api.prefill_chunk_paged(to_dev(q[:, P:]), kd.view(-1, page, Hkv, 128),
                                         vd.view(-1, page, Hkv, 128), table, **kw)
        torch.cuda.synchronize()
    finally:
        if rescale:
            api.debug_prefill_rescale_log2(old)
    assert torch.equal(out.view(torch.int16), pg.view(torch.int16))
    assert torch.equal(lse.view(torch.int32), pl.view(torch.int32))
    pos = sorted(set(range(P, T, max(1, n // 40))) | {T - 1})
    rows = np.array([[b, h, x] for b in range(B) for h in range(Hq) for x in pos], dtype=np.int64)
    want, want_lse, _ = O.prefill_rows(q, k, v, rows, theta=1e6, w_pretrained=w_pre, w_local=w0,
                                       want_lse=True)
    assert_close(to_f64(out)[rows[:, 0], rows[:, 2] - P, rows[:, 1]], want, what="split blocks")
    assert np.isfinite(to_f64(out)).all()
    assert_close(lse.cpu().numpy()[rows[:, 0], rows[:, 1], rows[:, 2] - P], want_lse, max_abs=5e-2,
                 mean_abs=5e-3, what="split lse")


@pytest.mark.parametrize("rescale", [None, 3.0])
@pytest.mark.parametrize("P,n,B,Hkv,g,w_pre,w0", [
    (3000, 64, 1, 8, 4, 1024, 300),    # 8 blocks, all cut, one per XCD
    (2900, 130, 3, 8, 4, 1 << 20, 0),  # 72 blocks of three q blocks a group, G = 1
    (9000, 2100, 1, 8, 4, 2048, 500),  # 256 whole blocks and the last wave's 8 in parts
    (6000, 1370, 2, 3, 8, 2048, 500),  # 256 and 2, groups no multiple of the XCDs
])
def test_cut_blocks_in_the_grid(P, n, B, Hkv, g, w_pre, w0, rescale):
    """Whole blocks in front of a cut last wave, and cut blocks in the XCD order
    (kv heads times sequences a multiple of 8): rows of every query block, its
    first and last, against the oracle, over a poisoned output."""
    T, Hq, page, bq = P + n, g * Hkv, 64, 256 // g
    q, k, v = synth.prefill_inputs(B, Hq, Hkv, T, 128, seed=T + g, outlier_channels=8)
    pages = -(-T // page)
    pad = [(0, 0), (0, pages * page - T), (0, 0), (0, 0)]
    kd, vd = (to_dev(np.pad(x, pad, constant_values=0x7FC0)) for x in (k, v))
    qd = to_dev(q[:, P:])
    table = torch.arange(B * pages, dtype=torch.int32, device="cuda").view(B, pages)
    kw = dict(q_start=P, w_pretrained=w_pre, w_local=w0, want_lse=True)
    old = api.debug_prefill_rescale_log2(rescale) if rescale else None
    try:
        say("cut blocks in the grid P=%d n=%d B=%d rescale=%s" % (P, n, B, rescale))
        out, lse = api.prefill_chunk(qd, kd, vd, out=torch.full_like(qd, float("nan")), **kw)
        say("cut blocks in the grid, paged")
        pg, pl = api.prefill_chunk_paged(qd, kd.view(-1, page, Hkv, 128),
                                         vd.view(-1, page, Hkv, 128), table,
                                         out=torch.full_like(qd, float("nan")), **kw)
        torch.cuda.synchronize()
    finally:
        if rescale:
            api.debug_prefill_rescale_log2(old)
    assert torch.equal(out.view(torch.int16), pg.view(torch.int16))
    assert torch.equal(lse.view(torch.int32), pl.view(torch.int32))
    assert bool(torch.isfinite(out.float()).all()) and bool(torch.isfinite(lse).all())
    starts = range(P, T, bq)
    pos = sorted({x for s in starts for x in (s, min(s + bq, T) - 1)})
    rows = np.array([[b, h, x] for b in range(B) for i, x in enumerate(pos)
                     for h in {i % Hq, (i + bq) % Hq, Hq - 1 - i % Hq}], dtype=np.int64)
    want, want_lse, _ = O.prefill_rows(q, k, v, rows, theta=1e6, w_pretrained=w_pre, w_local=w0,
                                       want_lse=True)
    assert_close(to_f64(out)[rows[:, 0], rows[:, 2] - P, rows[:, 1]], want, what="cut in the grid")
    assert_close(lse.cpu().numpy()[rows[:, 0], rows[:, 1], rows[:, 2] - P], want_lse, max_abs=5e-2,
                 mean_abs=5e-3, what="cut lse")


def test_cut_calls_on_two_streams():
    """Cut calls that overlap on two streams, each with its own states, one of
    them growing its scratch while the other runs: the bits of calls made alone."""
    Hq, Hkv, P = 8, 2, 6000
    shapes = [64, 200, 520]  # more parts each: the scratch grows
    q, k, v = (to_dev(x) for x in synth.prefill_inputs(1, Hq, Hkv, P + 520, 128, seed=8))
    chunks = [(q[:, P:P + n].contiguous(), k[:, :P + n].contiguous(), v[:, :P + n].contiguous())
              for n in shapes]
    kw = dict(q_start=P, w_pretrained=2048, w_local=500)
    alone = [api.prefill_chunk(*c, **kw) for c in chunks]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    say("cut chunks on two streams")
    got = []
    for i in range(6):
        for j, st in enumerate(streams):
            m = (i // 2 if j == 0 else 2 - i // 2)  # one grows, the other starts large
            out = torch.empty_like(chunks[m][0])
            api.prefill_chunk(*chunks[m], out=out, stream=st, **kw)
            got.append((m, out))
    torch.cuda.synchronize()
    for m, out in got:
        assert torch.equal(out.view(torch.int16), alone[m].view(torch.int16)), m


def test_cut_call_under_capture_needs_no_allocation():
    """A stream whose calls so far needed no scratch captures a call that would
    be cut: the call runs whole blocks instead of allocating inside the capture.
    After an eager call of that shape the capture cuts as the eager call does,
    and its replays stay good when a larger call replaces the scratch."""
    Hq, Hkv, P, n = 8, 2, 9000, 64
    q, k, v = (to_dev(x) for x in synth.prefill_inputs(1, Hq, Hkv, P + n, 128, seed=3))
    kw = dict(w_pretrained=2048, w_local=500)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    with torch.cuda.stream(side):
        big = torch.randn((8, 4096, 32, 128), device="cuda").to(torch.bfloat16)  # fills the CUs
        kv = big[:, :, :8].contiguous()
        api.bifocal_prefill(big, kv, kv, **kw)
        api.rope_attention_decode(q[:, -1].contiguous(), k, v,  # the RoPE table covers the call
                                  torch.tensor([P + n], dtype=torch.int32, device="cuda"))
        qc, out = q[:, P:].contiguous(), torch.empty_like(q[:, P:].contiguous())
        torch.cuda.synchronize()

        def captured():
            say("cut chunk, captured")
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=side):
                api.prefill_chunk(qc, k, v, q_start=P, out=out, **kw)
            outs = []
            for _ in range(3):
                out.fill_(float("nan"))
                graph.replay()
                torch.cuda.synchronize()
                outs.append(out.clone())
            assert all(torch.equal(o.view(torch.int16), outs[0].view(torch.int16)) for o in outs)
            return graph, outs[0]

        _, whole = captured()
        say("cut chunk, eager")
        eager = api.prefill_chunk(qc, k, v, q_start=P, **kw)
        torch.cuda.synchronize()
        graph, cut = captured()
        say("larger cut chunk, then the graph again")  # its states must not lie in freed memory
        api.prefill_chunk(big[:1, :1000], k, v, q_start=P - 1000, w_pretrained=2048, w_local=500)
        filler = [torch.full((1 << 20,), float("nan"), device="cuda") for _ in range(40)]
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        del filler
        assert torch.equal(out.view(torch.int16), cut.view(torch.int16))
    assert torch.equal(cut.view(torch.int16), eager.view(torch.int16))
    full = api.bifocal_prefill(q, k, v, **kw)[:, P:]
    torch.cuda.synchronize()
    assert_close(to_f64(whole), to_f64(full), what="captured whole blocks")
    assert_close(to_f64(cut), to_f64(full), what="captured parts")
