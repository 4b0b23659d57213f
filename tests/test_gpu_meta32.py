"""Decode with fp32 metadata on the matrix-core kernel: a page's sums are formed exactly (high limbs on
one grid a head and value group), so the output agrees with the double-precision oracle to fp32 rounding."""
import numpy as np
import pytest

from paper_2605_19660_amd import synth
from test_gpu_parity import _ob, make_pair, to_dev, assert_cache_equal

pytestmark = pytest.mark.gpu

# What fp32 arithmetic costs against the oracle's doubles, whichever kernel runs: a logit is a sum
# of 128 products times the token norm, good to about 2^-22 of its magnitude (|logit| < 128 here),
# and moves its probability by that much: 2^-22 * 128 * ln 2 = 2.1e-5 for one token, less for the
# norm over all outputs.
REL = 2.2e-5


def _run(w, splits, lens=None, zp=0, scale_pages=None, cap=8):
    ob = _ob()
    import torch
    k, v = synth.make_kv_batch(w)
    if scale_pages is not None:
        for i, f in enumerate(scale_pages):
            v[:, 128 * i:128 * (i + 1)] *= np.float32(f)
    q = synth.make_q(w)
    g, o = make_pair(w, cap, zp_mode=zp)
    nl = None if lens is None else np.asarray(lens, np.int32)
    ob.quantize_append(g, to_dev(k, w.io_dtype), to_dev(v, w.io_dtype), eager=True, max_seq_len_hint=0,
                       new_lens=None if nl is None else torch.from_numpy(nl).cuda())
    o.append(k, v, eager=True, new_lens=nl)
    assert_cache_equal(g, o, w)
    out = ob.decode_attn(g, to_dev(q, w.io_dtype), max_seq_len_hint=w.context, num_splits=splits)
    out = out.cpu().numpy().astype(np.float64)
    want = o.decode_attn(q).astype(np.float64)
    assert np.isfinite(out).all()
    return out, want


def _close(out, want):
    rel = np.linalg.norm(out - want) / np.linalg.norm(want)
    assert rel <= REL, rel


@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("gq", [4, 7])
@pytest.mark.parametrize("bits", [2, 4])
@pytest.mark.parametrize("kg,vg", [(128, 32), (128, 64), (128, 128), (64, 32), (64, 64), (64, 128),
                                   (32, 32), (32, 64), (32, 128)])
def test_every_variant(kg, vg, bits, gq, zp):
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=2 * gq, n_kv_heads=2, context=128 * 5 + 70,
                                  io_dtype="f32", meta_dtype="f32", bits=bits, k_group=kg, v_group=vg)
    _close(*_run(w, 2, zp=zp))


@pytest.mark.parametrize("io", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("splits", [1, 3])
def test_lengths_at_the_page_edges(io, splits):
    w = synth.LLAMA8B_32K.replace(batch=6, n_q_heads=8, n_kv_heads=2, context=128 * 6 - 1,
                                  io_dtype=io, meta_dtype="f32")
    out, want = _run(w, splits, lens=[0, 1, 127, 128, 129, 128 * 6 - 1])
    assert (out[0] == 0).all()
    _close(out, want)


@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("scale_pages", [
    (2.0 ** -100,) * 6,                    # step sizes far below anything fp16 holds
    (2.0 ** 90,) * 6,
    (2.0 ** 60, 1.0, 2.0 ** -60, 1.0, 2.0 ** 60, 2.0 ** -60),   # neighbours 2^120 apart
])
def test_value_magnitudes_over_the_fp32_range(scale_pages, zp):
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=8, n_kv_heads=2, context=128 * 5 + 40,
                                  io_dtype="f32", meta_dtype="f32")
    _close(*_run(w, 1, zp=zp, scale_pages=scale_pages))


# ---- values of mixed magnitude inside one page -----------------------------------------------------
# Each kv head's first page holds the tokens below; the error is taken per value group, so that a small
# group is not hidden by a large one.  The bound is REL for each: what moves an output is the probabilities'
# error, which all channels share, and a group's own rounding is a few 2^-24 of its largest p * Delta.

def _per_group(vg, gq, bits, kg, zp, edit, splits=1):
    ob = _ob()
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=2 * gq, n_kv_heads=2, context=128 * 3 + 40,
                                  io_dtype="f32", meta_dtype="f32", bits=bits, k_group=kg, v_group=vg)
    k, v = (np.array(x) for x in synth.make_kv_batch(w))
    q = synth.make_q(w)
    edit(k, v, q.reshape(w.batch, 2, gq, 128).sum(2))
    g, o = make_pair(w, 4, zp_mode=zp)
    ob.quantize_append(g, to_dev(k, "f32"), to_dev(v, "f32"), eager=True, max_seq_len_hint=0)
    o.append(k, v, eager=True)
    out = ob.decode_attn(g, to_dev(q, "f32"), max_seq_len_hint=w.context, num_splits=splits)
    out = out.cpu().numpy().astype(np.float64)
    want = o.decode_attn(q).astype(np.float64)
    shape = (w.batch, 2 * gq, 128 // vg, vg)
    err = np.linalg.norm((out - want).reshape(shape), axis=-1)
    ref = np.linalg.norm(want.reshape(shape), axis=-1)
    assert (err <= REL * ref).all(), (err / ref).max()


# (query heads per kv head, bits, key group): one and two head slots, both code widths
FORMS = [(4, 2, 128), (7, 4, 32), (4, 4, 64)]


@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("gq,bits,kg", FORMS)
@pytest.mark.parametrize("spread", [1e-2, 1e-3, 1e-6])
@pytest.mark.parametrize("peaked", [False, True])
def test_a_nearly_constant_group_beside_ordinary_ones(gq, bits, kg, zp, spread, peaked):
    """Values 1 +- spread: a zero-point of 1 / step, times p * Delta of far fewer bits than the product needs."""
    def edit(k, v, qsum):
        r = np.random.default_rng(1)
        v[..., 96:] = 1 + spread * r.standard_normal(v[..., 96:].shape)
        if peaked:
            k[:, 40] = 1.5 * qsum
    _per_group(32, gq, bits, kg, zp, edit)


@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("gq,bits,kg", FORMS)
@pytest.mark.parametrize("e", [8, 12, 30])
def test_a_few_tokens_far_above_the_others(gq, bits, kg, zp, e):
    """Tokens that hold 2^e times the values and next to none of the softmax."""
    def edit(k, v, qsum):
        for t in (5, 77, 200):
            k[:, t] = -3.0 * qsum
            v[:, t] *= np.float32(2.0 ** e)
    _per_group(64, gq, bits, kg, zp, edit, splits=2)


@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("gq,bits,kg", FORMS)
@pytest.mark.parametrize("e", [8, 12, 30])
def test_the_softmax_peak_far_below_the_others(gq, bits, kg, zp, e):
    def edit(k, v, qsum):
        k[:, 40] = 1.5 * qsum
        v[:, 40] *= np.float32(2.0 ** -e)
    _per_group(128, gq, bits, kg, zp, edit)


@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("gq,bits,kg", FORMS)
@pytest.mark.parametrize("e", [8, 12, 30])
def test_a_value_group_far_above_the_others(gq, bits, kg, zp, e):
    def edit(k, v, qsum):
        v[..., :32] *= np.float32(2.0 ** e)
    _per_group(32, gq, bits, kg, zp, edit)


@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("gq", [4, 7])
def test_an_infinite_value_stays_in_its_group(gq, zp):
    """One infinite channel of one token: its step size is infinite and its group has no number; the
    other groups of the page are what they are without it."""
    import torch
    ob = _ob()
    outs = []
    for x in (1.0, float("inf")):
        w = synth.LLAMA8B_32K.replace(batch=1, n_q_heads=gq, n_kv_heads=1, context=256, io_dtype="f32",
                                      meta_dtype="f32")
        k, v = (np.array(t) for t in synth.make_kv_batch(w))
        v[0, 9, 0, 3] = x
        g, _ = make_pair(w, 2, zp_mode=zp)
        ob.quantize_append(g, to_dev(k, "f32"), to_dev(v, "f32"), eager=True, max_seq_len_hint=0)
        outs.append(ob.decode_attn(g, to_dev(synth.make_q(w), "f32"), max_seq_len_hint=256, num_splits=1))
    assert not torch.isfinite(outs[1][..., :32]).any()
    assert torch.equal(outs[0][..., 32:], outs[1][..., 32:])
