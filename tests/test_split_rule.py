"""The automatic split count where two splits of four-wave workgroups would fill the chip: one of eight waves instead,
in the variants that have that form.  (Without a GPU the library counts 256 compute units.)"""
import pytest
import torch

from paper_2605_19660_amd import binding as ob


@pytest.mark.skipif(torch.cuda.is_available(), reason="the numbers are those of 256 compute units")
def test_two_splits_become_one():
    rule = ob.decode_auto_splits
    for bits in (2, 4):
        cfg = ob.Config(32, 8, bits=bits)
        assert [rule(cfg, b, 8192) for b in (16, 17, 21, 22, 32, 33)] == [4, 3, 3, 1, 1, 1]
    assert rule(ob.Config(28, 4), 44, 8192) == 1                              # seven query heads a kv head
    assert rule(ob.Config(32, 8, meta_dtype=ob.F32), 24, 8192) == 2           # fp32 metadata: as before
    assert rule(ob.Config(32, 8, bits=4, k_group=32, v_group=64), 24, 8192) == 2   # no eight-wave form
    assert rule(ob.Config(32, 8), 1, 2048 + 128) == 2                         # two by the pages, not by the chip


def _units():
    return torch.cuda.get_device_properties(0).multi_processor_count if torch.cuda.is_available() else 256


@pytest.mark.parametrize("share", [0.55, 0.7, 1.0])   # of the compute units, as (sequence, kv head) pairs
def test_where_one_split_does_not_stand_for_two(share):
    rule, batch = ob.decode_auto_splits, int(share * _units()) // 4
    for tokens in (2060, 2900):   # (16 .. 23 pages: two splits at most)
        at = lambda gq=4, **kw: rule(ob.Config(4 * gq, 4, **kw), batch, tokens)
        assert at() == 1 and at(gq=7) == 1 and at(bits=4) == 1 and at(k_group=32, v_group=64) == 1
        # a step with one split is two calls there, with two it is not
        assert at(gq=7, k_group=32, v_group=64) == 2 and at(gq=7, k_group=32, v_group=128) == 2


@pytest.mark.parametrize("n_q_heads,n_kv_heads", [(32, 8), (28, 4), (8, 8)])
def test_the_comparator_keeps_the_count_of_four_waves(n_q_heads, n_kv_heads, monkeypatch):
    """Without a count bf16_decode_attn sizes its workspace for its own one: two splits, not one of eight waves."""
    batch = int(0.7 * _units()) // n_kv_heads
    assert ob.decode_auto_splits(ob.Config(n_q_heads, n_kv_heads), batch, 4000) == 1

    class Seen(Exception):
        pass

    def sized(cfg, b, num_splits):
        raise Seen(num_splits)

    class Rows:   # what the wrapper asks of a tensor before it needs the device
        def __init__(self, *shape):
            self.shape, self.is_cuda, self.device = shape, True, "cpu"

        def is_contiguous(self):
            return True

    monkeypatch.setattr(ob, "decode_workspace_bytes", sized)
    kv = Rows(batch, 4000, n_kv_heads, 128)
    with pytest.raises(Seen) as seen:
        ob.bf16_decode_attn(Rows(batch, n_q_heads, 128), kv, kv, None, out=kv)
    assert seen.value.args == (2,)
