"""Small appends, where a block's keys and values are two workgroups and every load is a buffer load: windows and
tails of all relations, bit for bit against the oracle.  What a place must not take from beside it (old window, new
tokens, neighbouring heads) is non-zero everywhere."""
import numpy as np
import pytest

from paper_2605_19660_amd import synth
from test_gpu_parity import _ob, make_pair, to_dev, assert_cache_equal

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("norm_all", [False, True])
@pytest.mark.parametrize("io,meta,bits,kg,vg", [("bf16", "f16", 2, 128, 32), ("f32", "f32", 4, 32, 64), ("f16", "f32", 2, 64, 128)])
def test_windows_and_tails(io, meta, bits, kg, vg, norm_all):
    w = synth.LLAMA8B_32K.replace(batch=2, n_q_heads=3, n_kv_heads=3, context=128 + 257, io_dtype=io, meta_dtype=meta,
                                  bits=bits, k_group=kg, v_group=vg)
    k, v = synth.make_kv_batch(w)
    ob = _ob()
    for old in (0, 1, 16, 111, 127, 128):
        for new in (17, 32, 33, 112, 127, 128, 129, 256, 257):
            for eager in (True, False):
                g, o = make_pair(w, 4, norm_scope=1 if norm_all else 0)
                at = 0
                for n, rule in ((old, False), (new, eager)):
                    if n:
                        kp, vp = np.ascontiguousarray(k[:, at:at + n]), np.ascontiguousarray(v[:, at:at + n])
                        ob.quantize_append(g, to_dev(kp, io), to_dev(vp, io), eager=rule, max_seq_len_hint=at)
                        o.append(kp, vp, eager=rule)
                        at += n
                assert_cache_equal(g, o, w)
                assert int(g.tickets.item()) == 0 and int(g.dev_status.item()) == 0, (old, new, eager)
