"""oscar_rotate_columns at widths and alignments on both sides of its two kernels: bit-exact
against the butterfly in its prescribed order."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _reference(w):
    """H / sqrt(128) along the rows of every 128-row block, fp32, stages 1 .. 64 in order."""
    x = w.astype(np.float32).reshape(-1, 128, w.shape[1]).copy()
    h = 1
    while h < 128:
        y = x.reshape(x.shape[0], 128 // (2 * h), 2, h, x.shape[2])
        a, b = y[:, :, 0].copy(), y[:, :, 1].copy()
        y[:, :, 0], y[:, :, 1] = a + b, a - b
        h *= 2
    return (x * np.float32(0.08838834764831845)).reshape(w.shape)


@pytest.mark.parametrize("io", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("cols,offset", [(4, 0), (60, 0), (64, 0), (68, 0), (132, 0), (1000, 0), (2880, 0),
                                         (1, 0), (63, 0), (1002, 0), (64, 1), (64, 2)])
def test_widths_and_alignments(cols, offset, io):
    import torch
    from paper_2605_19660_amd import binding as ob
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[io]
    rows = 256
    rng = np.random.default_rng(cols + offset)
    store = torch.from_numpy(rng.standard_normal(rows * cols + offset).astype(np.float32)).to(dt)
    dev = store.cuda()[offset:].view(rows, cols)
    got = ob.rotate_columns(dev).cpu().numpy()
    want = _reference(store[offset:].view(rows, cols).float().numpy())
    assert np.array_equal(got, want)


@pytest.mark.parametrize("io", ["bf16", "f16", "f32"])
@pytest.mark.parametrize("blocks,cols", [(32, 500), (32, 516), (33, 500), (32, 512), (4, 4100), (3, 4100)])
def test_both_sides_of_a_wave_a_cu(blocks, cols, io):
    """Widths that are not whole cache lines change kernels where the grid passes a wave a CU (256)."""
    import torch
    from paper_2605_19660_amd import binding as ob
    dt = {"bf16": torch.bfloat16, "f16": torch.float16, "f32": torch.float32}[io]
    host = torch.from_numpy(np.random.default_rng(cols).standard_normal((128 * blocks, cols)).astype(np.float32)).to(dt)
    got = ob.rotate_columns(host.cuda()).cpu().numpy()
    assert np.array_equal(got, _reference(host.float().numpy()))
