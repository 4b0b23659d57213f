"""Long walks of the matrix-core decode kernel: a wave keeps 64 block-table entries in a register, works 63
pages off them and reloads.  Page counts one below, at and past one and two such chunks for every wave, in
the eight-wave form (launches of at most one workgroup a compute unit) and the four-wave one, over tables that
name a few physical pages many times in random order; attention alone against the oracle, and the step's bits."""
import numpy as np
import pytest

import oracle as orc
from paper_2605_19660_amd import synth
from test_gpu_parity import DT, _ob, make_pair, to_dev, assert_decode_close

pytestmark = pytest.mark.gpu

PHYS = 23
CHUNK = 63
POOLS = ("k_codes", "k_meta", "k_norms", "v_codes", "v_meta")


def _check(waves, splits, io, meta, bits, kg, vg, gq, zp=0):
    import torch
    ob = _ob()
    walk = waves * splits          # pages a round of all waves of a sequence takes
    pages = [walk * CHUNK - 1, walk * CHUNK, walk * CHUNK + 1, walk * 2 * CHUNK, walk * 2 * CHUNK + 1,
             walk * 2 * CHUNK + walk + 3]
    cap = max(pages) + 1
    w = synth.LLAMA8B_32K.replace(batch=1, n_q_heads=gq, n_kv_heads=1, context=128 * PHYS, io_dtype=io,
                                  meta_dtype=meta, bits=bits, k_group=kg, v_group=vg)
    k, v = synth.make_kv_batch(w)
    src, o1 = make_pair(w, PHYS, zp_mode=zp)
    ob.quantize_append(src, to_dev(k, io), to_dev(v, io), eager=True, max_seq_len_hint=0)
    o1.append(k, v, eager=True)

    # sequence i of the launch has the length and the table row of i modulo the number of lengths
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    n = len(pages)
    batch = n if waves == 8 else (cus // (n * splits) + 1) * n
    assert (batch * splits <= cus) == (waves == 8)
    rng = np.random.default_rng(waves + splits)
    rows = rng.integers(0, PHYS, size=(n, cap))
    cfg = ob.Config(gq, 1, bits=bits, k_group=kg, v_group=vg, io_dtype=DT[io], meta_dtype=DT[meta], zp_mode=zp)
    table = np.tile(rows, (batch // n, 1))
    caches = []
    for _ in range(3):
        c = ob.Cache(cfg, batch, cap, num_pages=PHYS, page_perm=table.reshape(-1))
        for name in POOLS:
            getattr(c, name).copy_(getattr(src, name))
        c.seq_lens.copy_(torch.from_numpy(np.tile(np.asarray(pages, np.int32) * 128, batch // n)))
        caches.append(c)

    # the oracle's arrays of those sequences
    o = orc.OracleCache(o1.cfg, n, 1, cap * 128)
    for i, p in enumerate(pages):
        tok = (rows[i, :p, None] * 128 + np.arange(128)).reshape(-1)
        grp = (rows[i, :p, None] * (128 // kg) + np.arange(128 // kg)).reshape(-1)
        for name in ("k_codes", "k_norm", "v_codes", "v_delta", "v_zero"):
            getattr(o, name)[i, 0, :len(tok)] = getattr(o1, name)[0, 0, tok]
        for name in ("k_delta", "k_zero"):
            getattr(o, name)[i, 0, :len(grp)] = getattr(o1, name)[0, 0, grp]
        o.n_packed[i] = 128 * p
    q = np.tile(synth.make_q(w), (n, 1, 1)) * np.linspace(0.5, 1.5, n, dtype=np.float32)[:, None, None]
    q = to_dev(q, io)
    want = o.decode_attn(q.float().cpu().numpy(), nthreads=4)
    qd = q.repeat(batch // n, 1, 1)
    hint = 128 * cap
    out = ob.decode_attn(caches[0], qd, max_seq_len_hint=hint, num_splits=splits)
    assert_decode_close(out[:n].cpu().numpy(), want)
    assert torch.equal(out.view(batch // n, n, gq, 128), out[:n].expand(batch // n, n, gq, 128))

    # one step: the bits of the append and the attention by themselves
    new = synth.make_kv_batch(w.replace(context=1, batch=n))
    kn, vn = (to_dev(np.tile(x, (batch // n, 1, 1, 1)), io) for x in new)
    outs = [torch.empty(batch, gq, 128, device="cuda") for _ in range(2)]
    ws = torch.empty(ob.decode_workspace_bytes(cfg, batch, splits), dtype=torch.uint8, device="cuda")
    ob.decode_step(caches[1], kn, vn, qd, outs[0], ws, splits, hint)
    ob.quantize_append(caches[2], kn, vn, max_seq_len_hint=-1)
    ob.decode_attn(caches[2], qd, out=outs[1], max_seq_len_hint=hint, num_splits=splits, workspace=ws)
    assert torch.equal(outs[0], outs[1])
    assert torch.equal(caches[1].seq_lens, caches[2].seq_lens)


@pytest.mark.parametrize("io,meta,bits,kg,vg,gq,zp,splits", [
    ("bf16", "f16", 2, 128, 32, 4, 0, 1), ("bf16", "f16", 2, 32, 64, 7, 1, 2), ("f16", "f16", 4, 128, 64, 3, 0, 1),
    ("f32", "f32", 2, 128, 32, 4, 0, 1),
])
def test_eight_waves(io, meta, bits, kg, vg, gq, zp, splits):
    _check(8, splits, io, meta, bits, kg, vg, gq, zp)


@pytest.mark.parametrize("io,meta,bits,kg,vg,gq,zp,splits", [
    ("bf16", "f16", 2, 128, 32, 4, 0, 1), ("bf16", "f16", 2, 64, 32, 7, 1, 2), ("f16", "f16", 4, 32, 32, 3, 0, 2),
    ("f32", "f32", 4, 128, 32, 4, 0, 1),
])
def test_four_waves(io, meta, bits, kg, vg, gq, zp, splits):
    _check(4, splits, io, meta, bits, kg, vg, gq, zp)
