"""The matrix-core decode kernel's two forms, eight waves a workgroup for launches of at most one
workgroup a compute unit and four for larger ones: the same streams through both against the oracle, at
page counts around one and two rounds of the waves and at the edges of the window's passes, and the
decode step's bits in the four-wave form (the small shapes of the other tests run in the eight-wave one)."""
import numpy as np
import pytest

from paper_2605_19660_amd import synth
from test_gpu_parity import DT, _ob, make_pair, to_dev, assert_decode_close
from test_gpu_step_forms import _run

pytestmark = pytest.mark.gpu

# pages x 128 + window: below, at and past 8 and 16 pages (one and two rounds of a split's eight waves);
# windows that end in every wave's share of a pass of 32 tokens
LENS = [0, 1, 31, 128 + 32, 128 * 3 + 33, 128 * 7 + 64, 128 * 8, 128 * 8 + 127, 128 * 9 + 5, 128 * 16 + 96,
        128 * 17 + 2]


@pytest.mark.parametrize("splits", [1, 2, 3])
@pytest.mark.parametrize("io,meta,bits,kg,vg,gq,zp", [
    ("bf16", "f16", 2, 128, 32, 4, 0), ("f16", "f16", 4, 128, 64, 3, 1), ("bf16", "f16", 2, 32, 32, 7, 1),
    ("f32", "f32", 2, 128, 32, 4, 0), ("f32", "f32", 2, 64, 64, 8, 1), ("bf16", "f16", 4, 32, 32, 2, 0),
])
def test_both_forms_against_the_oracle(io, meta, bits, kg, vg, gq, zp, splits):
    import torch
    ob = _ob()
    w = synth.LLAMA8B_32K.replace(batch=len(LENS), n_q_heads=2 * gq, n_kv_heads=2, context=max(LENS), io_dtype=io,
                                  meta_dtype=meta, bits=bits, k_group=kg, v_group=vg)
    k, v = synth.make_kv_batch(w)
    q = synth.make_q(w)
    g, o = make_pair(w, 18, zp_mode=zp)
    lens = np.asarray(LENS, np.int32)
    ob.quantize_append(g, to_dev(k, io), to_dev(v, io), eager=True, max_seq_len_hint=0,
                       new_lens=torch.from_numpy(lens).cuda())
    o.append(k, v, eager=True, new_lens=lens)
    few = ob.decode_attn(g, to_dev(q, io), max_seq_len_hint=w.context, num_splits=splits)
    want = o.decode_attn(q)
    assert_decode_close(few.cpu().numpy(), want)
    # the same cache several times over, until the launch has more workgroups than the chip has units
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    times = cus // (splits * w.n_kv_heads * w.batch) + 1
    cfg = ob.Config(w.n_q_heads, w.n_kv_heads, bits=bits, k_group=kg, v_group=vg, io_dtype=DT[io],
                    meta_dtype=DT[meta], zp_mode=zp)
    many = ob.Cache(cfg, w.batch * times, 18)
    for name in ("seq_lens", "res_lens", "res_k", "res_v", "res_norm", "k_codes", "k_meta", "k_norms", "v_codes",
                 "v_meta"):
        src = getattr(g, name)
        dst = getattr(many, name)
        assert dst.numel() == src.numel() * times, name
        dst.view(-1).copy_(src.view(-1).repeat(times))
    out = ob.decode_attn(many, to_dev(np.tile(q, (times, 1, 1)), io), max_seq_len_hint=w.context, num_splits=splits)
    out = out.view(times, w.batch, w.n_q_heads, 128)
    assert_decode_close(out[0].cpu().numpy(), want)
    for i in range(1, times):
        assert torch.equal(out[i], out[0]), i


@pytest.mark.parametrize("splits", [1, 2])
@pytest.mark.parametrize("io,bits,kg,vg,gq", [("bf16", 2, 128, 32, 4), ("f16", 4, 64, 32, 3), ("bf16", 2, 64, 64, 7),
                                              ("f32", 2, 128, 32, 4), ("f32", 4, 64, 64, 2), ("f32", 2, 64, 32, 7)])
def test_bits_of_the_two_calls_in_the_four_wave_form(io, bits, kg, vg, gq, splits):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    starts = ([0, 1, 126, 127, 128, 255, 256, 300] * (cus // 8 + 1))[:cus + 1]
    w = synth.LLAMA8B_32K.replace(batch=len(starts), n_q_heads=gq, n_kv_heads=1, context=300 + 4, io_dtype=io,
                                  bits=bits, k_group=kg, v_group=vg)
    _run(w, starts, 3, splits, 4)


@pytest.mark.parametrize("bits,hkv,splits", [(4, 2, 2), (4, 1, 5), (2, 4, 0)])   # 0: past the unit count by itself
def test_bits_of_a_sequence_where_its_batch_does_not_choose_the_form(bits, hkv, splits):
    import torch
    ob = _ob()
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    splits = splits or cus // hkv + 1
    w = synth.LLAMA8B_32K.replace(batch=1, n_q_heads=4 * hkv, n_kv_heads=hkv, context=128 * 9 + 50, bits=bits)
    k, v = synth.make_kv_batch(w)
    kd, vd, q = to_dev(k, w.io_dtype), to_dev(v, w.io_dtype), to_dev(synth.make_q(w), w.io_dtype)
    outs = []
    for batch in (1, cus // (hkv * min(splits, cus)) + 2):
        c = ob.Cache(ob.Config(w.n_q_heads, hkv, bits=bits), batch, 10)
        ob.quantize_append(c, kd.repeat(batch, 1, 1, 1), vd.repeat(batch, 1, 1, 1), eager=True, max_seq_len_hint=0)
        outs.append(ob.decode_attn(c, q.repeat(batch, 1, 1), max_seq_len_hint=w.context, num_splits=splits))
    assert torch.equal(outs[0].expand_as(outs[1]), outs[1])
