"""Multi-token appends in the 512-thread forms (small launches; the smallest have two workgroups a block,
one for the keys and one for the values) and the 256-thread form of the encoder: block edges, tails, and blocks that mix the residual window with new tokens, bit for bit
against the oracle, at launch sizes on both sides of the choice."""
import numpy as np
import pytest
import torch

from paper_2605_19660_amd import synth
from test_gpu_parity import _ob, make_pair, to_dev, assert_cache_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm_all", [False, True])
@pytest.mark.parametrize("zp", [0, 1])
@pytest.mark.parametrize("io,meta,bits,kg,vg", [
    ("bf16", "f16", 2, 128, 32), ("f16", "f16", 4, 32, 64), ("f32", "f32", 2, 64, 128),
    ("f32", "f16", 4, 128, 32), ("bf16", "f32", 2, 32, 128), ("f16", "f32", 4, 64, 32),
])
def test_pieces_at_block_edges(io, meta, bits, kg, vg, zp, norm_all):
    pieces = [2, 31, 33, 62, 127, 128, 129, 1, 160, 255, 257, 500, 3]
    total = sum(pieces)
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=4, n_kv_heads=2, context=total, io_dtype=io,
                                  meta_dtype=meta, bits=bits, k_group=kg, v_group=vg)
    k, v = synth.make_kv_batch(w)
    g, o = make_pair(w, total // 128 + 2, zp_mode=zp, norm_scope=1 if norm_all else 0)
    ob = _ob()
    at = 0
    for n in pieces:
        kp, vp = np.ascontiguousarray(k[:, at:at + n]), np.ascontiguousarray(v[:, at:at + n])
        ob.quantize_append(g, to_dev(kp, io), to_dev(vp, io), eager=True, max_seq_len_hint=at)
        o.append(kp, vp, eager=True)
        assert_cache_equal(g, o, w)
        at += n
    assert int(g.dev_status.item()) == 0


@pytest.mark.parametrize("context", [128 * 3 + 70, 128 * 4])   # 32 x 4 and 32 x 5 x batch 4: 512, 640 workgroups
def test_the_two_forms_meet_at_the_launch_size(context):
    import torch
    w = synth.LLAMA8B_32K.replace(batch=4, n_q_heads=32, n_kv_heads=32, context=context)
    k, v = synth.make_kv_batch(w)
    g, o = make_pair(w, 6)
    lens = np.array([context, 127, 128, 300], np.int32)
    ob = _ob()
    ob.quantize_append(g, to_dev(k, w.io_dtype), to_dev(v, w.io_dtype), eager=True, max_seq_len_hint=0,
                       new_lens=torch.from_numpy(lens).cuda())
    o.append(k, v, eager=True, new_lens=lens)
    assert_cache_equal(g, o, w)


@pytest.mark.parametrize("eager", [True, False])
@pytest.mark.parametrize("norm_all", [False, True])
@pytest.mark.parametrize("io,bits,kg", [("bf16", 2, 128), ("f32", 4, 32)])
def test_pieces_at_the_choice_of_the_form_by_length(io, bits, kg, norm_all, eager):
    """16 tokens and fewer take the 256-thread form, 17 and more the 512-thread one, into the same window."""
    pieces = [16, 17, 15, 64, 17, 16, 2, 16, 110, 18, 16, 17]
    total = sum(pieces)
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=4, n_kv_heads=2, context=total, io_dtype=io, bits=bits, k_group=kg)
    k, v = synth.make_kv_batch(w)
    g, o = make_pair(w, total // 128 + 2, norm_scope=1 if norm_all else 0)
    ob = _ob()
    at = 0
    for n in pieces:
        kp, vp = np.ascontiguousarray(k[:, at:at + n]), np.ascontiguousarray(v[:, at:at + n])
        ob.quantize_append(g, to_dev(kp, io), to_dev(vp, io), eager=eager, max_seq_len_hint=at)
        o.append(kp, vp, eager=eager)
        assert_cache_equal(g, o, w)
        at += n


@pytest.mark.parametrize("norm_all", [False, True])
@pytest.mark.parametrize("io,meta,bits,kg", [("bf16", "f16", 2, 128), ("f32", "f32", 4, 32)])
@pytest.mark.parametrize("blocks,past", [(3, 0), (3, 1), (2, 0), (2, 1)])   # of the longest piece; past half a workgroup a unit
def test_pieces_where_a_block_becomes_one_workgroup(blocks, past, io, meta, bits, kg, norm_all):
    hkv = torch.cuda.get_device_properties(0).multi_processor_count // 2 // blocks + past   # 42, 43, 64, 65 of 256
    pieces = [150, 300, 17, 131, 256]
    total = sum(pieces)
    w = synth.LLAMA8B_32K.replace(batch=1, n_q_heads=hkv, n_kv_heads=hkv, context=total, io_dtype=io, meta_dtype=meta,
                                  bits=bits, k_group=kg)
    k, v = synth.make_kv_batch(w)
    g, o = make_pair(w, total // 128 + 2, norm_scope=1 if norm_all else 0)
    ob = _ob()
    at = 0
    for n in pieces:
        kp, vp = np.ascontiguousarray(k[:, at:at + n]), np.ascontiguousarray(v[:, at:at + n])
        ob.quantize_append(g, to_dev(kp, io), to_dev(vp, io), eager=True, max_seq_len_hint=at)
        o.append(kp, vp, eager=True)
        at += n
        if n in (150, 300, 256):
            assert_cache_equal(g, o, w)
    assert int(g.tickets.item()) == 0


@pytest.mark.parametrize("eager", [True, False])
@pytest.mark.parametrize("batch,hkv", [(1, 3), (3, 40), (9, 30)])   # 256 threads for all pieces past 16 in the last
@pytest.mark.parametrize("io,meta,bits,kg", [("bf16", "f16", 2, 128), ("f32", "f32", 4, 32)])
def test_window_places_taken_while_their_old_norms_are_needed(io, meta, bits, kg, batch, hkv, eager):
    """One norm over all heads: a new tail takes the places of old tokens that move into a page in the same
    call.  Old and new windows of all relations: shorter, longer, equal, full, empty."""
    pieces = [100, 40, 128, 88, 128, 200, 1, 127, 16, 130, 254]
    total = sum(pieces)
    w = synth.LLAMA8B_32K.replace(batch=batch, n_q_heads=hkv, n_kv_heads=hkv, context=total, io_dtype=io,
                                  meta_dtype=meta, bits=bits, k_group=kg)
    k, v = synth.make_kv_batch(w)
    g, o = make_pair(w, total // 128 + 2, norm_scope=1)
    ob = _ob()
    at = 0
    for i, n in enumerate(pieces):
        kp, vp = np.ascontiguousarray(k[:, at:at + n]), np.ascontiguousarray(v[:, at:at + n])
        lens = None
        if batch > 1 and i == 5:   # one sequence gets nothing, one a token
            lens = np.full(batch, n, np.int32)
            lens[0], lens[1] = 0, 1
        ob.quantize_append(g, to_dev(kp, io), to_dev(vp, io), None if lens is None else torch.from_numpy(lens).cuda(), eager=eager,
                           max_seq_len_hint=at)
        o.append(kp, vp, **({} if lens is None else {"new_lens": lens}), eager=eager)
        at += n
        if batch == 1 or i in (3, 5, 10):
            assert_cache_equal(g, o, w)


@pytest.mark.parametrize("eager", [True, False])
@pytest.mark.parametrize("io,meta,bits,kg", [("bf16", "f16", 2, 128), ("f16", "f32", 4, 32), ("f32", "f16", 4, 64)])
def test_few_tokens_across_a_page_edge_with_one_norm_over_all_heads(io, meta, bits, kg, eager):
    """Appends of up to 16 tokens: the norms of those that move into a page come from the launch in front, the
    others' from the encoder.  The edge at every place of an append, sequences of a batch at different ones."""
    pieces = [120, 16, 111, 1, 1, 127, 16, 112, 15, 1, 114, 14, 128, 16, 16]
    total = sum(pieces)
    w = synth.LLAMA8B_32K.replace(batch=5, n_q_heads=6, n_kv_heads=3, context=total, io_dtype=io, meta_dtype=meta,
                                  bits=bits, k_group=kg)
    k, v = synth.make_kv_batch(w)
    g, o = make_pair(w, total // 128 + 2, norm_scope=1)
    ob = _ob()
    at = 0
    for i, n in enumerate(pieces):
        kp, vp = np.ascontiguousarray(k[:, at:at + n]), np.ascontiguousarray(v[:, at:at + n])
        lens = np.array([n, max(n - 1, 0), n, (n + 1) // 2, 0 if i % 3 == 1 else n], np.int32)
        ob.quantize_append(g, to_dev(kp, io), to_dev(vp, io), torch.from_numpy(lens).cuda(), eager=eager, max_seq_len_hint=at)
        o.append(kp, vp, new_lens=lens, eager=eager)
        assert_cache_equal(g, o, w)
        at += n
