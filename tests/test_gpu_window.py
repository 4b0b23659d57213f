"""The residual window in the decode kernels, which read whole passes of it: what lies behind its last token, or
belongs to another split, must not reach a result.  Windows of all pass remainders, one and several splits, four and
eight waves, every value type, attention alone and step (whose new token takes a staged place), against the same cache
with infinities and NaN in the unused places, and against the oracle."""
import numpy as np
import pytest
import torch

from paper_2605_19660_amd import synth
from test_gpu_parity import _ob, make_pair, to_dev, assert_decode_close

pytestmark = pytest.mark.gpu


def _poison(g, w, seqs):
    hkv, es = w.n_kv_heads, 4 if w.io_dtype == "f32" else 2
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[w.io_dtype]
    k = g.res_k.view(torch.float16).view(w.batch, hkv, 128, 128)
    v = g.res_v[:w.batch * hkv * 128 * 128 * es].view(dt).view(w.batch, hkv, 128, 128)
    n = g.res_norm.view(torch.float32 if w.meta_dtype == "f32" else torch.float16).view(w.batch, hkv, 128)
    for b, r in enumerate(seqs):
        k[b, :, r:], v[b, :, r:], n[b, :, r:] = float("nan"), float("inf"), float("inf")


@pytest.mark.parametrize("io,meta,bits,gq", [("bf16", "f16", 2, 4), ("f16", "f16", 4, 7), ("f32", "f16", 2, 1),
                                             ("bf16", "f32", 4, 4), ("f32", "f32", 2, 7)])
@pytest.mark.parametrize("hkv", [2, 140])   # eight waves a workgroup; four, also with one split
def test_places_behind_the_window(io, meta, bits, gq, hkv):
    ob = _ob()
    for lens in ([0, 1], [3, 4], [5, 16], [17, 31], [32, 33], [63, 64], [65, 95], [100, 127], [128, 96]):
        n = [128 + r for r in lens]
        w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=gq * hkv, n_kv_heads=hkv, context=max(n), io_dtype=io,
                                      meta_dtype=meta, bits=bits)
        if hkv > 2 and lens[0] not in (0, 17, 100):
            continue
        k, v = synth.make_kv_batch(w)
        q = synth.make_q(w)
        k1, v1 = np.roll(k, 7, 1)[:, :1], np.roll(v, 7, 1)[:, :1]
        g, o = make_pair(w, 3)
        new = np.array(n, np.int32)
        # (128 tokens in the window stay there by the decode rule: the step's flush)
        ob.quantize_append(g, to_dev(k, io), to_dev(v, io), eager=False, max_seq_len_hint=0, new_lens=torch.from_numpy(new).cuda())
        o.append(k, v, eager=False, new_lens=new)
        seqs = g.res_lens.tolist()
        before = {name: getattr(g, name).clone() for name in vars(g) if isinstance(getattr(g, name), torch.Tensor)}
        outs, want = [], o.decode_attn(q)
        for splits in (1, 2, 8):
            work = torch.empty(ob.decode_workspace_bytes(g.cfg, 2, splits), dtype=torch.uint8, device="cuda")
            got = []
            for poison in (False, True):
                for name, t in before.items():
                    getattr(g, name).copy_(t)
                if poison:
                    _poison(g, w, seqs)
                attn = ob.decode_attn(g, to_dev(q, io), max_seq_len_hint=max(n), num_splits=splits).clone()
                out = torch.empty(2, gq * hkv, 128, device="cuda")
                ob.decode_step(g, to_dev(np.ascontiguousarray(k1), io), to_dev(np.ascontiguousarray(v1), io), to_dev(q, io),
                               out, work, splits, max_seq_len_hint=max(n) + 1)
                got.append((attn, out))
            assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1]), (lens, splits)
            outs.append([t.cpu().numpy() for t in got[0]])
        for attn, _ in outs:
            assert_decode_close(attn, want)
        o.append(np.ascontiguousarray(k1), np.ascontiguousarray(v1), eager=False)
        want = o.decode_attn(q)
        for _, out in outs:
            assert_decode_close(out, want)
