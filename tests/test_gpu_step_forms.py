"""oscar_decode_step with the append inside the attention kernel: same cache bytes, lengths and output
bits as the two calls, step by step through window fills and flushes."""
import numpy as np
import pytest

from paper_2605_19660_amd import synth
from test_gpu_parity import DT, _ob, assert_decode_close, make_pair, to_dev

pytestmark = pytest.mark.gpu

STATE = ("seq_lens", "res_lens", "res_k", "res_v", "res_norm", "k_codes", "k_meta", "k_norms", "v_codes",
         "v_meta", "tickets", "dev_status")


def _run(w, starts, cap, splits, steps, zp=0, fused=True, perm=None, out_dt=None):
    import torch
    ob = _ob()
    cfg = ob.Config(w.n_q_heads, w.n_kv_heads, bits=w.bits, k_group=w.k_group, v_group=w.v_group,
                    io_dtype=DT[w.io_dtype], zp_mode=zp)
    k, v = synth.make_kv_batch(w)
    n0 = max(max(starts), 1)
    pair = []
    for _ in range(2):
        c = ob.Cache(cfg, w.batch, cap, page_perm=perm, fused=fused)
        ob.quantize_append(c, to_dev(np.ascontiguousarray(k[:, :n0]), w.io_dtype),
                           to_dev(np.ascontiguousarray(v[:, :n0]), w.io_dtype), eager=False, max_seq_len_hint=0,
                           new_lens=torch.from_numpy(np.asarray(starts, np.int32)).cuda())
        pair.append(c)
    a, b = pair
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[w.io_dtype]
    odt = torch.float32 if out_dt is None else dt
    outs = [torch.empty(w.batch, w.n_q_heads, 128, dtype=odt, device="cuda") for _ in range(2)]
    ws = [torch.empty(ob.decode_workspace_bytes(cfg, w.batch, splits), dtype=torch.uint8, device="cuda")
          for _ in range(2)]
    rng = np.random.default_rng(5)
    for t in range(steps):
        kt = to_dev(np.ascontiguousarray(k[:, n0 + t:n0 + t + 1]), w.io_dtype)
        vt = to_dev(np.ascontiguousarray(v[:, n0 + t:n0 + t + 1]), w.io_dtype)
        q = torch.from_numpy(rng.standard_normal((w.batch, w.n_q_heads, 128)).astype(np.float32)).cuda().to(dt)
        hint = min(n0 + t + 1, 128 * cap)      # (the host refuses a hint past the table by itself)
        ob.decode_step(a, kt, vt, q, outs[0], ws[0], splits, hint)
        ob.quantize_append(b, kt, vt, max_seq_len_hint=-1)
        ob.decode_attn(b, q, out=outs[1], max_seq_len_hint=hint, num_splits=splits, workspace=ws[1])
        for name in STATE:
            assert torch.equal(getattr(a, name), getattr(b, name)), (t, name)
        assert torch.equal(outs[0].view(torch.uint8), outs[1].view(torch.uint8)), t
    return a


@pytest.mark.parametrize("splits", [1, 2, 5, 20])
@pytest.mark.parametrize("io,bits,kg,vg,hq,hkv,zp", [
    ("bf16", 2, 128, 32, 8, 2, 0), ("f16", 4, 32, 64, 14, 2, 0), ("f32", 2, 64, 128, 4, 4, 0),
    ("bf16", 4, 128, 32, 8, 2, 1), ("f32", 4, 32, 32, 16, 2, 1), ("f16", 2, 32, 32, 7, 1, 0),
])
def test_bits_of_the_two_calls_through_fill_and_flush(io, bits, kg, vg, hq, hkv, zp, splits):
    starts = [0, 1, 15, 126, 127, 128, 129, 383, 384, 511]   # empty, window edges, full windows
    w = synth.LLAMA8B_32K.replace(batch=len(starts), n_q_heads=hq, n_kv_heads=hkv, context=511 + 20,
                                  io_dtype=io, bits=bits, k_group=kg, v_group=vg)
    perm = np.random.default_rng(1).permutation(len(starts) * 6)
    _run(w, starts, 6, splits, 20, zp=zp, perm=perm)


@pytest.mark.parametrize("splits", [1, 3])
def test_a_whole_window_of_steps(splits):
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=8, n_kv_heads=2, context=300)
    _run(w, [130, 7], 4, splits, 135, out_dt="io")


@pytest.mark.parametrize("splits", [1, 2])
def test_without_tickets(splits):
    w = synth.LLAMA8B_32K.replace(batch=3, n_q_heads=8, n_kv_heads=2, context=150)
    _run(w, [128, 127, 1], 3, splits, 4, fused=False)


@pytest.mark.parametrize("splits", [1, 2])
def test_a_sequence_whose_page_table_is_full_stays_as_it_is(splits):
    """One page per sequence, window full behind it: the flush has nowhere to go, the other sequence
    goes on, and both calls report it the same way."""
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=8, n_kv_heads=2, context=262)
    c = _run(w, [256, 20], 1, splits, 3)
    assert c.seq_lens.tolist() == [256, 23] and c.res_lens.tolist() == [128, 23]
    assert int(c.dev_status.item()) == _ob().ERR_CAPACITY


# ---- which calls take the fused form: the launches of one captured step ------------------------------
FUSED, TWO_CALLS = "fused", "two calls"


def _launches(fn):
    """Kernel launches of fn() (its graph's nodes, all of them kernels)."""
    import ctypes as C
    import torch
    ob = _ob()
    graph = torch.cuda.CUDAGraph(keep_graph=True)
    with torch.cuda.graph(graph):
        fn()
    count, kind = C.c_size_t(0), C.c_int(-1)
    raw = C.c_void_p(graph.raw_cuda_graph())
    assert ob.lib().hipGraphGetNodes(raw, None, C.byref(count)) == 0
    nodes = (C.c_void_p * count.value)()
    assert ob.lib().hipGraphGetNodes(raw, nodes, C.byref(count)) == 0
    for node in nodes:
        assert ob.lib().hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)) == 0 and kind.value == 0   # a kernel
    return count.value


def _route(splits, batch=2, gq=4, hkv=2, generic=False, tickets=True, **cfg):
    import torch
    ob = _ob()
    cfg = ob.Config(gq * hkv, hkv, **cfg)
    c = ob.Cache(cfg, batch, 3, fused=tickets)
    kv = torch.randn(batch, 1, hkv, 128, device="cuda").bfloat16()
    q = torch.randn(batch, gq * hkv, 128, device="cuda").bfloat16()
    out = torch.empty(batch, gq * hkv, 128, device="cuda")
    ws = torch.empty(ob.decode_workspace_bytes(cfg, batch, splits), dtype=torch.uint8, device="cuda")
    ob.debug_force_generic_decode(generic)
    step = lambda: ob.decode_step(c, kv, kv, q, out, ws, splits, 1)
    step()
    n = _launches(step)
    ob.debug_force_generic_decode(False)
    append = 1 if tickets else 2   # without tickets the length update is its own launch
    reduce = 1 if splits > 1 or generic else 0
    if n == 1 + reduce and not generic:
        return FUSED
    assert n == append + 1 + reduce, n
    return TWO_CALLS


@pytest.mark.parametrize("splits", [1, 2, 5, 20])
@pytest.mark.parametrize("bits,kg,vg,gq,zp", [(2, 128, 32, 4, 0), (4, 32, 32, 4, 1), (2, 64, 128, 1, 0),
                                              (4, 128, 32, 7, 0), (2, 32, 32, 7, 0), (4, 32, 64, 4, 0)])
def test_the_usual_step_is_fused(bits, kg, vg, gq, zp, splits):
    assert _route(splits, bits=bits, k_group=kg, v_group=vg, gq=gq, zp_mode=zp) == FUSED


def test_steps_outside_the_fused_form():
    ob = _ob()
    assert _route(2, meta_dtype=ob.F32) == TWO_CALLS
    assert _route(2, norm_scope=ob.NORM_ALL_KV_HEADS) == TWO_CALLS
    assert _route(2, rotation=ob.ROTATION_OFF) == TWO_CALLS
    assert _route(2, scale_mode=ob.SCALE_MAX) == TWO_CALLS
    assert _route(2, generic=True) == TWO_CALLS
    assert _route(1, tickets=False) == TWO_CALLS
    assert _route(2, tickets=False) == FUSED


@pytest.mark.parametrize("bits,kg,vg,gq", [(2, 32, 32, 7), (4, 32, 64, 4), (4, 32, 128, 4), (4, 128, 128, 7),
                                           (4, 64, 128, 7)])
def test_variants_without_registers_to_spare_are_fused_up_to_a_workgroup_a_cu(bits, kg, vg, gq):
    import torch
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    at = lambda splits, batch: _route(splits, batch=batch, hkv=1, bits=bits, k_group=kg, v_group=vg, gq=gq)
    assert at(1, cus) == FUSED and at(2, cus // 2) == FUSED
    assert at(1, cus + 1) == TWO_CALLS and at(2, cus // 2 + 1) == TWO_CALLS


@pytest.mark.parametrize("vg", [64, 128])
def test_the_variants_that_need_several_splits(vg):
    assert _route(1, bits=2, k_group=32, v_group=vg, gq=7) == TWO_CALLS
    assert _route(2, bits=2, k_group=32, v_group=vg, gq=7) == FUSED


@pytest.mark.parametrize("splits", [1, 6])
@pytest.mark.parametrize("bits,kg,vg,gq", [(4, 32, 64, 4), (4, 32, 128, 3), (4, 128, 128, 7), (4, 64, 128, 8),
                                           (2, 32, 128, 6)])
def test_bits_of_the_variants_without_registers_to_spare(bits, kg, vg, gq, splits):
    starts = [0, 126, 128, 384, 511]
    w = synth.LLAMA8B_32K.replace(batch=5, n_q_heads=gq, n_kv_heads=1, context=511 + 4, bits=bits, k_group=kg,
                                  v_group=vg)
    _run(w, starts, 6, splits, 4, zp=splits & 1)


@pytest.mark.parametrize("gq,kg,vg,bits", [(4, 128, 32, 2), (4, 128, 32, 4), (7, 64, 64, 2), (7, 32, 64, 2), (7, 32, 128, 2)])
def test_a_step_of_the_automatic_count_is_fused(gq, kg, vg, bits):
    """Between half and all of the compute units in (sequence, kv head) pairs, where the rule looks at the variant."""
    import torch
    ob = _ob()
    batch = torch.cuda.get_device_properties(0).multi_processor_count * 11 // 64
    splits = ob.decode_auto_splits(ob.Config(4 * gq, 4, bits=bits, k_group=kg, v_group=vg), batch, 4000)
    assert _route(splits, batch=batch, gq=gq, hkv=4, bits=bits, k_group=kg, v_group=vg) == FUSED


@pytest.mark.parametrize("gq,kg,scale", [(4, 128, "l2"), (7, 32, "l2"), (2, 128, "mean_abs")])
def test_calls_of_the_automatic_count_against_the_oracle(gq, kg, scale):
    """The count worked out by the calls themselves, workspace and all, in the same range of pairs."""
    import torch
    ob = _ob()
    batch = torch.cuda.get_device_properties(0).multi_processor_count * 11 // 64
    n = 2048 + 70   # (16 pages: two splits at most)
    w = synth.LLAMA8B_32K.replace(batch=batch, n_q_heads=4 * gq, n_kv_heads=4, context=n, k_group=kg, v_group=64)
    k, v = synth.make_kv_batch(w)
    q = synth.make_q(w)
    g, o = make_pair(w, 17, scale=scale)
    ob.quantize_append(g, to_dev(k, w.io_dtype), to_dev(v, w.io_dtype), eager=True, max_seq_len_hint=0)
    o.append(k, v, eager=True)
    qd = to_dev(q, w.io_dtype)
    assert_decode_close(ob.decode_attn(g, qd, max_seq_len_hint=n).cpu().numpy(), o.decode_attn(q))
    k1, v1 = np.ascontiguousarray(np.roll(k, 9, 1)[:, :1]), np.ascontiguousarray(np.roll(v, 9, 1)[:, :1])
    splits = ob.decode_auto_splits(g.cfg, batch, n + 1)
    work = torch.empty(ob.decode_workspace_bytes(g.cfg, batch, splits), dtype=torch.uint8, device="cuda")
    out = torch.empty(batch, w.n_q_heads, 128, device="cuda")
    ob.decode_step(g, to_dev(k1, w.io_dtype), to_dev(v1, w.io_dtype), qd, out, work, 0, max_seq_len_hint=n + 1)
    o.append(k1, v1, eager=False)
    assert_decode_close(out.cpu().numpy(), o.decode_attn(q))
