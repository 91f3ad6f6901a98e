"""Prefill parity: the HIP kernels through the C ABI against the fp64 oracle."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2607_07740_amd import api, synth
from parity_util import (assert_close, prefill_block_q, rows_for, sample_positions, say, to_dev,
                         to_f64)

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _run(bifocal, q, k, v, w, w0, theta=1e6, want_lse=False):
    qd, kd, vd = to_dev(q), to_dev(k), to_dev(v)
    out = torch.full_like(qd, float("nan"))  # poison: every element must be written
    lse = None
    if want_lse:
        lse = torch.full((q.shape[0], q.shape[2], q.shape[1]), float("nan"), device="cuda")
    if bifocal:
        api.bifocal_prefill(qd, kd, vd, w_pretrained=w, w_local=w0, rope_theta=theta, out=out,
                            lse=lse)
    else:
        api.rope_attention(qd, kd, vd, rope_theta=theta, out=out, lse=lse)
    torch.cuda.synchronize()
    return (out, lse) if want_lse else out


def test_tiny_workload_full_tensor():
    w = synth.WORKLOADS["tiny_prefill"]
    q, k, v = synth.make_inputs(w)
    say("tiny bifocal prefill", q.shape, "G=%d" % api.group_size(w.L, w.w_pretrained))
    out, lse = _run(True, q, k, v, w.w_pretrained, w.w_local, want_lse=True)
    want, want_lse = O.prefill(q, k, v, theta=w.theta, w_pretrained=w.w_pretrained,
                               w_local=w.w_local)
    assert_close(to_f64(out), want, what="tiny bifocal")
    # LSE error budget: fp32 scores from bf16 operands, ~1e-2 in the logit at |s| ~ 10
    assert_close(lse.cpu().numpy(), want_lse, max_abs=5e-2, mean_abs=5e-3, what="tiny lse")


def test_tiny_workload_vanilla_full_tensor():
    w = synth.WORKLOADS["tiny_prefill"]
    q, k, v = synth.make_inputs(w)
    say("tiny vanilla prefill", q.shape)
    out = _run(False, q, k, v, 0, 0)
    want, _ = O.prefill(q, k, v, theta=w.theta, bifocal=False)
    assert_close(to_f64(out), want, what="tiny vanilla")


@pytest.mark.parametrize("L,g,w_pre,w0", [
    (1, 1, 1, 0), (2, 2, 1, 0), (63, 4, 16, 5), (65, 2, 20, 0), (127, 8, 40, 1),
    (129, 1, 32, 64), (300, 2, 64, 63), (300, 4, 70, 100), (517, 2, 100, 128), (640, 8, 128, 65),
    (200, 2, 300, 10),  # G == 1: must equal vanilla
])
def test_ragged_shapes_full_tensor(L, g, w_pre, w0):
    B, Hkv = 2, 2
    q, k, v = synth.prefill_inputs(B, g * Hkv, Hkv, L, 128, seed=L + g, outlier_channels=8)
    say("ragged prefill L=%d g=%d w_pre=%d w0=%d" % (L, g, w_pre, w0))
    out, lse = _run(True, q, k, v, w_pre, w0, want_lse=True)
    want, want_lse = O.prefill(q, k, v, theta=1e6, w_pretrained=w_pre, w_local=w0)
    assert_close(to_f64(out), want, what="ragged L=%d g=%d" % (L, g))
    assert_close(lse.cpu().numpy(), want_lse, max_abs=5e-2, mean_abs=5e-3, what="lse")
    if api.group_size(L, w_pre) == 1:
        van = _run(False, q, k, v, 0, 0)
        assert torch.equal(out.view(torch.int16), van.view(torch.int16))


@pytest.mark.parametrize("B,Hkv,g,L", [(2, 3, 2, 300), (4, 6, 1, 200), (1, 5, 8, 129)])
def test_kv_group_counts_and_block_orders(B, Hkv, g, L):
    """B * Hkv kv groups of 6, 24 and 5: the workgroup order differs when the
    count divides by 8 (each XCD takes whole groups) and when it does not."""
    w_pre, w0 = 64, 30
    q, k, v = synth.prefill_inputs(B, g * Hkv, Hkv, L, 128, seed=B * 100 + Hkv, outlier_channels=8)
    say("prefill B=%d Hkv=%d g=%d L=%d" % (B, Hkv, g, L))
    for bif in (True, False):
        out = _run(bif, q, k, v, w_pre, w0)
        want, _ = (O.prefill(q, k, v, theta=1e6, w_pretrained=w_pre, w_local=w0) if bif
                   else O.prefill(q, k, v, theta=1e6, bifocal=False))
        assert_close(to_f64(out), want, what="B=%d Hkv=%d bifocal=%s" % (B, Hkv, bif))


@pytest.mark.parametrize("bifocal", [True, False])
@pytest.mark.parametrize("L,g,w_pre,w0", [(300, 4, 70, 20), (517, 2, 100, 128), (64, 1, 16, 5)])
def test_rescale_path_on_every_tile(bifocal, L, g, w_pre, w0):
    """With the rescale bound lowered to 2^3 the kernel moves a row's softmax
    reference and rescales its running output on almost every tile of
    ordinary data; the result must still match the oracle.  (A jump large
    enough to cross the default 2^64 bound only occurs with scores of tens of
    nats, where bf16 rounding of the operands alone already changes the
    softmax weights, so the path is checked this way.)"""
    B, Hkv = 1, 2
    q, k, v = synth.prefill_inputs(B, g * Hkv, Hkv, L, 128, seed=L + 3 * g, outlier_channels=8)
    old = api.debug_prefill_rescale_log2(3.0)
    try:
        say("rescale-every-tile prefill L=%d g=%d bifocal=%d" % (L, g, bifocal))
        out, lse = _run(bifocal, q, k, v, w_pre, w0, want_lse=True)
    finally:
        api.debug_prefill_rescale_log2(old)
    want, want_lse = O.prefill(q, k, v, theta=1e6, w_pretrained=w_pre, w_local=w0,
                               bifocal=bifocal)
    assert_close(to_f64(out), want, what="rescale path")
    assert_close(lse.cpu().numpy(), want_lse, max_abs=5e-2, mean_abs=5e-3, what="rescale lse")


@pytest.mark.parametrize("g,Hkv", [(64, 2), (128, 2), (256, 1)])
def test_rescale_rerun_list_holds_every_block(g, Hkv):
    """Wide GQA groups give query blocks of a few positions (one at g = 256),
    so a 300-token call has up to 300 blocks per kv head.  With the bound
    lowered to 2^3 nearly every block trips the check and is run again by its
    own workgroup with the checked pass; the result must still match the
    oracle."""
    B, L, w_pre, w0 = 1, 300, 70, 20
    q, k, v = synth.prefill_inputs(B, g * Hkv, Hkv, L, 128, seed=g, outlier_channels=8)
    old = api.debug_prefill_rescale_log2(3.0)
    try:
        say("rescale rerun list, wide group g=%d L=%d" % (g, L))
        out, lse = _run(True, q, k, v, w_pre, w0, want_lse=True)
    finally:
        api.debug_prefill_rescale_log2(old)
    want, want_lse = O.prefill(q, k, v, theta=1e6, w_pretrained=w_pre, w_local=w0)
    assert_close(to_f64(out), want, what="wide group g=%d" % g)
    assert_close(lse.cpu().numpy(), want_lse, max_abs=5e-2, mean_abs=5e-3, what="wide lse")


def test_all_scores_far_below_zero():
    """Every score of a row is about -300 nats: exp2 against the initial
    reference underflows, so the reference must move down to the row maximum
    before anything is accumulated."""
    B, Hq, Hkv, L, w_pre, w0 = 1, 2, 1, 300, 100, 20
    q, k, v = (synth.bf16_to_f32(x) for x in synth.prefill_inputs(B, Hq, Hkv, L, 128, seed=9))
    q, k = q.copy(), k.copy()
    # the lowest RoPE frequency pair (dims 63, 127) barely rotates over 300
    # positions, so a shared component there makes every q.k strongly negative
    q[..., 63] = -60.0
    k[..., 63] = 60.0
    qb, kb, vb = synth.bf16_bits(q), synth.bf16_bits(k), synth.bf16_bits(v)
    say("far-negative scores prefill")
    out = _run(True, qb, kb, vb, w_pre, w0)
    want, _ = O.prefill(qb, kb, vb, theta=1e6, w_pretrained=w_pre, w_local=w0)
    assert_close(to_f64(out), want, what="negative scores")


def test_deterministic_and_theta_variants():
    q, k, v = synth.prefill_inputs(1, 4, 2, 333, 128, seed=41)
    for theta in (1e4, 5e5):
        say("prefill theta=%g" % theta)
        a = _run(True, q, k, v, 100, 17, theta=theta)
        b = _run(True, q, k, v, 100, 17, theta=theta)
        assert torch.equal(a.view(torch.int16), b.view(torch.int16))
        want, _ = O.prefill(q, k, v, theta=theta, w_pretrained=100, w_local=17)
        assert_close(to_f64(a), want, what="theta=%g" % theta)


def _sampled_parity(name, n_random):
    w = synth.WORKLOADS[name]
    say("generating", name)
    q, k, v = synth.make_inputs(w)
    G = api.group_size(w.L, w.w_pretrained)
    say("%s bifocal prefill B=%d Hq=%d Hkv=%d L=%d G=%d" % (name, w.B, w.Hq, w.Hkv, w.L, G))
    out = _run(True, q, k, v, w.w_pretrained, w.w_local)
    block_q = prefill_block_q(w.Hq, w.Hkv)
    pos = sample_positions(w.L, w.w_local, w.w_pretrained, G, block_q, n_random)
    rows = rows_for(w.B, w.Hq, pos)
    say("oracle rows", len(rows))
    want, nthreads = O.prefill_rows(q, k, v, rows, theta=w.theta, w_pretrained=w.w_pretrained,
                                    w_local=w.w_local)
    o = out.float().cpu().numpy()
    got = o[rows[:, 0], rows[:, 2], rows[:, 1]].astype(np.float64)
    assert_close(got, want, what=name)
    assert np.isfinite(o).all()
    return q, k, v, out


def test_within_window_equals_vanilla_and_oracle():
    q, k, v, out = _sampled_parity("qwen3_1p7b_within_32k", 32)
    w = synth.WORKLOADS["qwen3_1p7b_within_32k"]
    say("within-window vanilla prefill")
    van = _run(False, q, k, v, 0, 0)
    assert torch.equal(out.view(torch.int16), van.view(torch.int16))


def test_long_1p7b_128k_sampled_rows():
    _sampled_parity("qwen3_1p7b_prefill_128k", 24)


def test_long_8b_128k_sampled_rows():
    _sampled_parity("qwen3_8b_prefill_128k", 16)


def test_long_8b_64k_sampled_rows():
    _sampled_parity("qwen3_8b_prefill_64k", 16)


@pytest.mark.parametrize("w0", [299, 1 << 30, 2 ** 31 - 1])
def test_band_covering_every_key_is_vanilla(w0):
    """w_local >= L - 1 leaves no remote pair (Eq. (1)), so the bifocal call
    is the base model whatever G is (here G = 5): the fused kernel then visits
    the vanilla kernel's tiles in its order with its masks, bit for bit."""
    B, Hkv, g, L, w_pre = 2, 2, 4, 300, 64
    assert api.group_size(L, w_pre) == 5
    q, k, v = synth.prefill_inputs(B, g * Hkv, Hkv, L, 128, seed=w0 % 1000, outlier_channels=8)
    say("prefill band over every key, w0=%d" % w0)
    out = _run(True, q, k, v, w_pre, w0)
    van = _run(False, q, k, v, 0, 0)
    assert torch.equal(out.view(torch.int16), van.view(torch.int16))
    want, _ = O.prefill(q, k, v, theta=1e6, w_pretrained=w_pre, w_local=w0)
    assert_close(to_f64(out), want, what="band over every key")
