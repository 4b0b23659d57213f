"""Decode with fp32 metadata on the matrix-core kernel: the page sums are formed exactly
(high limbs on one grid), so the output agrees with the double-precision oracle to fp32 rounding."""
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
