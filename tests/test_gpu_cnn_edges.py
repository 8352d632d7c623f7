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


# k_conv walks columns of 16 x 16 voxels through ranges of planes
CONV_SHAPES = SHAPES + [(1, 3, 16, 16), (2, 4, 17, 15), (1, 2, 1, 33), (300, 1, 3, 2), (1, 64, 2, 2)]


@pytest.mark.parametrize("flip", [False, True])
@pytest.mark.parametrize("shape", CONV_SHAPES)
def test_layer_at_column_edges(shape, flip):
    from oracle import cnn
    from paper_1701_06254_amd import r2p
    rng = np.random.default_rng(sum(shape) + 1)
    x_t, x = _bits(rng.normal(size=shape + (32,)))
    W = cnn.bf16_round(rng.normal(0, 0.05, size=(27, 32, 32)))
    w_t, _ = _bits(np.ascontiguousarray(W.transpose(0, 2, 1)) if flip else W)
    a_t, a = _bits(rng.normal(size=shape + (32,)))
    m_t, m = _bits(rng.normal(size=shape + (32,)))
    b = rng.normal(size=32).astype(np.float32)
    V = int(np.prod(shape))
    outf = torch.full((V * 32,), float("nan"), dtype=torch.float32, device="cuda")
    r2p.cnn_conv(x_t, shape, w_t, bias=torch.from_numpy(b).cuda(), addend=a_t, mask=m_t, flip=flip,
                 outf=outf)
    ref = cnn.conv_grad_input(x, W) if flip else cnn.conv(x, W, np.zeros(32))
    ref = (ref + b + a) * (m > 0)
    got = outf.cpu().numpy().astype(np.float64).reshape(ref.shape)
    assert np.max(np.abs(got - ref)) <= 1e-5 * np.max(np.abs(ref))


@pytest.mark.parametrize("shape", [(1, 1, 1, 1), (2, 3, 17, 33)])
def test_features_at_any_alignment(shape):
    """The feature tensor may start at any 2-byte address: same results as
    from an aligned one."""
    from oracle import cnn
    from paper_1701_06254_amd import r2p
    rng = np.random.default_rng(5)
    net = r2p.Cnn(blocks=1)
    net.set_params(cnn.init_params(rng, 32, 1).astype(np.float32))
    V = int(np.prod(shape))
    f = np.zeros((V, 32))
    f[:, :6] = rng.normal(size=(V, 6))
    f_t, _ = _bits(f)
    ref = net.forward(f_t, shape).clone()
    shifted = torch.zeros(V * 32 + 1, dtype=torch.int16, device="cuda")
    shifted[1:] = f_t.reshape(-1)
    assert torch.equal(net.forward(shifted[1:], shape), ref)


@pytest.mark.parametrize("shape", [(600, 1, 3, 2), (300, 3, 1, 2), (1, 50, 48, 97)])
def test_weight_gradient_over_several_tiles(shape):
    """More than twice as many tiles of 2 x 8 x 32 voxels as the device has
    CUs: a workgroup requests its next tile while it works on one and carries
    its sums across them, the last round uneven.  A sum is built in at most
    this many FP32 additions one after another, each off by 2^-24 of the sum of
    magnitudes: 32 products and one addition per row of a tile, the tiles of a
    workgroup, then the workgroups in eighths."""
    from oracle import cnn
    from paper_1701_06254_amd import r2p
    nb, nz, ny, nx = shape
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tiles = nb * -(-nz // 2) * -(-ny // 8) * -(-nx // 32)
    assert tiles > 2 * cus and tiles % cus
    rng = np.random.default_rng(sum(shape))
    g_t, g = _bits(rng.normal(size=shape + (32,)))
    x_t, x = _bits(rng.normal(size=shape + (32,)))
    dw = torch.full((27 * 32 * 32,), float("nan"), dtype=torch.float32, device="cuda")
    db = torch.full((32,), float("nan"), dtype=torch.float32, device="cuda")
    r2p.cnn_conv_dw(g_t, x_t, shape, dw, db)
    chain = -(-tiles // cus) * 16 * 33 + cus // 8 + 8
    for got, ref, mag in zip((dw, db), cnn.conv_grad_weight(g, x),
                             cnn.conv_grad_weight(np.abs(g), np.abs(x))):
        err = np.abs(got.cpu().numpy().astype(np.float64) - ref.reshape(-1))
        assert np.all(err <= chain * 2.0 ** -24 * mag.reshape(-1))


# columns of 4, 8 and 16 rows by the grid's extent in y, and cross-sections
# (ny = 1), which run as one plane of nz rows with two axes of taps exchanged
THIN = [(2, 5, 1, 40), (1, 17, 1, 16), (3, 9, 1, 7), (1, 4, 1, 15), (1, 33, 1, 33), (1, 2, 1, 1),
        (2, 3, 2, 17), (1, 3, 4, 20), (1, 5, 5, 17), (2, 2, 8, 16), (1, 3, 9, 18)]


@pytest.mark.parametrize("flip", [False, True])
@pytest.mark.parametrize("shape", THIN)
def test_layer_on_thin_grids(shape, flip):
    test_layer_at_column_edges(shape, flip)


@pytest.mark.parametrize("shape", [(2, 12, 1, 21), (1, 6, 4, 9), (1, 1, 8, 30)])
def test_cross_section_network_matches_its_transpose(shape):
    """A grid with the y and z axes exchanged and the weights' taps with them
    is the same problem: the forward pass agrees to FP32 rounding of each
    layer's sums (BF16 activations may then round the other way: 2^-8 of the
    largest output a layer, five layers here)."""
    from oracle import cnn
    from paper_1701_06254_amd import r2p
    nb, nz, ny, nx = shape
    K = 1
    theta = cnn.bf16_round(cnn.init_params(np.random.default_rng(3), 32, K, out_scale=1.0)).astype(np.float32)
    f = np.zeros(shape + (32,))
    f[..., :6] = np.random.default_rng(4).normal(size=shape + (6,))
    swapped, o = theta.copy(), 0
    for l in range(2 * K + 2):
        cin, cout = 6 if l == 0 else 32, 2 if l == 2 * K + 1 else 32
        m = 27 * cin * cout
        W = theta[o:o + m].reshape(3, 3, 3, cout, cin)
        swapped[o:o + m] = np.ascontiguousarray(W.transpose(1, 0, 2, 3, 4)).reshape(-1)
        o += m + cout
    assert o == theta.size
    out = []
    for th, a, sh in ((theta, f, shape), (swapped, f.transpose(0, 2, 1, 3, 4), (nb, ny, nz, nx))):
        net = r2p.Cnn(blocks=K)
        net.set_params(th)
        out.append(net.forward(_bits(np.ascontiguousarray(a))[0], sh).cpu().numpy().reshape(sh + (2,)))
    ref = out[1].transpose(0, 2, 1, 3, 4)
    assert np.max(np.abs(out[0] - ref)) <= 5 * 2.0 ** -8 * np.max(np.abs(ref))
