"""Network kernels at the edges of their tiles (2 x 8 x 32 voxels): single
voxels, exactly one tile, one voxel more or less on an axis, more tiles than
workgroups' first round, and crops whose neighbours in memory belong to
another crop.  Inputs are bfloat16-representable; the reference is the FP64
CPU network, and FP32 accumulation of K products stays within K 2^-24 of the
sum of magnitudes: bound 1e-5 of the largest result, as the sums here hold
at most a few thousand products of like size.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 1, 1, 1), (3, 1, 1, 2), (1, 2, 8, 32), (2, 3, 9, 33), (3, 1, 7, 31), (1, 5, 17, 64),
          (2, 2, 16, 65), (70, 2, 8, 17)]


def _bits(a):
    from oracle import cnn
    r = cnn.bf16_round(a)
    b = (np.asarray(r, dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
    return torch.from_numpy(b.view(np.int16).copy()).cuda(), r


@pytest.mark.parametrize("shape", SHAPES)
def test_weight_gradient_at_tile_edges(shape):
    from oracle import cnn
    from paper_1701_06254_amd import r2p
    rng = np.random.default_rng(sum(shape))
    g_t, g = _bits(rng.normal(size=shape + (32,)))
    x_t, x = _bits(rng.normal(size=shape + (32,)))
    dw = torch.full((27 * 32 * 32,), float("nan"), dtype=torch.float32, device="cuda")
    db = torch.full((32,), float("nan"), dtype=torch.float32, device="cuda")
    r2p.cnn_conv_dw(g_t, x_t, shape, dw, db)
    rdw, rdb = cnn.conv_grad_weight(g, x)
    got = dw.cpu().numpy().astype(np.float64)
    assert np.max(np.abs(got - rdw.reshape(-1))) <= 1e-5 * np.max(np.abs(rdw))
    # the bias sums cancel: bound by the sum of magnitudes
    mag = np.abs(g).reshape(-1, 32).sum(0)
    assert np.all(np.abs(db.cpu().numpy() - rdb) <= 1e-6 * mag + 1e-12)
