"""oscar_decode_step with the append inside the attention kernel: same cache bytes, lengths and output
bits as the two calls, step by step through window fills and flushes."""
import numpy as np
import pytest

from paper_2605_19660_amd import synth
from test_gpu_parity import DT, _ob, to_dev

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
