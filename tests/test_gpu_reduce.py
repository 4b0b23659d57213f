"""The reduce pass at split counts on both sides of its three forms (1 .. 16, 17 .. 64, more), with
splits that hold no token, against the definition in doubles."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("splits", [1, 2, 16, 17, 18, 33, 63, 64, 65, 130, 512])
@pytest.mark.parametrize("out_dt,offset", [("f32", 0), ("bf16", 0), ("f32", 1)])
def test_split_counts(splits, out_dt, offset):
    import torch
    from paper_2605_19660_amd import binding as ob
    dt = {"f32": torch.float32, "bf16": torch.bfloat16}[out_dt]
    B, H = 3, 4
    cfg = ob.Config(H, 2)
    cache = ob.Cache(cfg, B, 1)
    rng = np.random.default_rng(splits)
    rec = rng.standard_normal((B, H, splits, 130)).astype(np.float32)
    rec[..., 128] *= 8
    rec[..., 129] = np.abs(rec[..., 129]) + 0.1
    empty = rng.random((B, H, splits)) < 0.3
    empty[0, 0] = True                         # a sequence that holds nothing
    empty[1, 1, :-1], empty[1, 1, -1] = True, False
    rec[empty, 128] = -np.inf
    rec[empty, :128] = 0
    rec[empty, 129] = 0
    ws = torch.zeros(rec.size + offset, dtype=torch.float32, device="cuda")[offset:]   # (offset 1: 4-byte aligned)
    ws.copy_(torch.from_numpy(rec.reshape(-1)))
    out = torch.empty(B, H, 128, dtype=dt, device="cuda")
    ob.decode_attn_reduce(cache, out, ws.view(torch.uint8), splits)
    got = out.float().cpu().numpy()
    r = rec.astype(np.float64)
    with np.errstate(invalid="ignore"):
        m = r[..., 128].max(-1, keepdims=True)
        wgt = np.where(empty, 0.0, np.exp2(r[..., 128] - m))
    den = (wgt * r[..., 129]).sum(-1)
    want = (wgt[..., None] * r[..., :128]).sum(2) / np.where(den > 0, den, 1.0)[..., None]
    # each weight is good to 2 ulp, the sums add one rounding a term; bf16 output: half a step more
    scale = (wgt[..., None] * np.abs(r[..., :128])).sum(2) / np.where(den > 0, den, 1.0)[..., None]
    bound = scale * (splits + 8) * 2.0 ** -24 + (np.abs(want) * 2.0 ** -8 if out_dt == "bf16" else 0)
    assert (np.abs(got - want) <= bound + 1e-30).all()
    assert (got[0, 0] == 0).all()


@pytest.mark.parametrize("splits", [1, 2, 15, 16, 17, 18, 33, 63, 64, 65, 130])
@pytest.mark.parametrize("at", ["first", "last"])
def test_an_infinite_partial_gives_an_infinite_output(splits, at):
    """A split that holds an infinite value (16-bit window) has an infinite partial in that channel: the
    weighted sum is infinite there whatever the form does with the places past the last split."""
    import torch
    from paper_2605_19660_amd import binding as ob
    cache = ob.Cache(ob.Config(2, 1), 1, 1)
    rng = np.random.default_rng(splits)
    rec = rng.standard_normal((1, 2, splits, 130)).astype(np.float32)
    rec[..., 129] = np.abs(rec[..., 129]) + 0.1
    rec[0, 1, 0 if at == "first" else splits - 1, [5, 6]] = [np.inf, -np.inf]
    ws = torch.from_numpy(rec.reshape(-1)).cuda()
    out = torch.empty(1, 2, 128, device="cuda")
    ob.decode_attn_reduce(cache, out, ws.view(torch.uint8), splits)
    got = out.cpu().numpy()
    assert got[0, 1, 5] == np.inf and got[0, 1, 6] == -np.inf
    got[0, 1, [5, 6]] = 0
    assert np.isfinite(got).all()
