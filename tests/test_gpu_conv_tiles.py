"""Convolution kernels at the edges of their tiles, against the FP64 reference
(oracle.conv) on BF16-representable operands.

Outputs are rounded to BF16 once (half a unit in the last place: 2^-9 of the
value) after FP32 accumulation of at most 27 * 136 products (relative error
below 2^-12 of the largest output for these operands), so the largest
difference stays within 2^-8 of the largest reference value.  FP32 weight and
bias gradients: sums of at most 2^12 products, 2^12 * 2^-24 of the largest
sum of magnitudes, bounded by 1e-5 of the largest reference value as the
other weight-gradient checks are."""
import numpy as np
import pytest

from oracle import conv

pytestmark = pytest.mark.gpu

TOL = 2.0 ** -8


def _operands(c, seed):
    rng = np.random.default_rng(seed)
    xs = (c["n"], c["d"], c["h"], c["w"], c["ci"])
    s = c.get("s", 1)
    ys = (c["n"],) + tuple(-(-v // s) for v in xs[1:4]) + (c["co"],)
    x = conv.bf16_round(rng.standard_normal(xs))
    w = conv.bf16_round(rng.standard_normal((c["co"], c.get("k", 3) ** 3, c["ci"])) * 0.1)
    b = rng.standard_normal(c["co"]).astype(np.float32)
    dy = conv.bf16_round(rng.standard_normal(ys))
    return x, w, b, dy


def _sliced(S, a, off, extra):
    """The array as a channel slice (from `off`) of a buffer `extra` channels wider, filled with NaN elsewhere."""
    n, d, h, w, c = a.shape
    wide = np.full((n, d, h, w, c + extra), np.nan)
    wide[..., off:off + c] = a
    return S.from_numpy(wide).slice(off, c)


def _check(c, seed):
    from paper_1007_1388_amd import surrogate as S
    k, s = c.get("k", 3), c.get("s", 1)
    x, w, b, dy = _operands(c, seed)
    layer = S.Conv(c["ci"], c["co"], k=k, stride=s, relu=True)
    layer.set_weights(w, b)
    X, DY = _sliced(S, x, 8, 16), _sliced(S, dy, 16, 24)
    # forward into a slice; its neighbours stay untouched
    Y = _sliced(S, np.zeros(dy.shape), 8, 16)
    layer.forward(X, Y)
    ref = conv.conv3d(x, w, b.astype(np.float64), k, s, True)
    assert np.abs(Y.to_numpy() - ref).max() <= TOL * np.abs(ref).max()
    assert np.isnan(S.Act(c["n"], *dy.shape[1:4], c["co"] + 16, buf=Y.buf, ldc=Y.ldc).to_numpy()[..., :8]).all()
    # input gradient added to a previous one and masked by ReLU'(x)
    prev = conv.bf16_round(np.random.default_rng(seed + 1).standard_normal(x.shape))
    DX = _sliced(S, prev, 8, 8)
    st = S.lib().lbm_conv3d_bwd_data(DY.ref, layer.wt.data_ptr(), DX.ref, X.ref, k, s, 1, None)
    assert st == 0
    ref = prev + conv.conv3d_bwd_data(dy, w, x.shape, k, s) * (x > 0)
    assert np.abs(DX.to_numpy() - ref).max() <= TOL * np.abs(ref).max()


# stride 1: one voxel short of, on and past the 16-column tiles and the 8- and
# 16-row tiles; one plane; channels below, on and off the 32-channel chunks and
# column tiles; enough tiles for the larger kind
ROWS = [
    dict(n=1, d=1, h=1, w=1, ci=8, co=8),
    dict(n=2, d=2, h=7, w=15, ci=24, co=40),
    dict(n=1, d=3, h=8, w=16, ci=32, co=32),
    dict(n=1, d=2, h=9, w=17, ci=40, co=72),
    dict(n=1, d=2, h=16, w=33, ci=136, co=24),
    dict(n=4, d=17, h=17, w=31, ci=8, co=64),
    dict(n=3, d=22, h=16, w=32, ci=40, co=40),
]


# the 8-channel forward: partial tiles along every axis (four planes per tile)
ROWS += [dict(n=2, d=5, h=17, w=17, ci=8, co=40), dict(n=1, d=9, h=15, w=16, ci=8, co=32)]


@pytest.mark.parametrize("case", range(len(ROWS)))
def test_stride1_row_tiles(case):
    _check(ROWS[case], 100 + case)


# stride 1, 64, 128 and 256 channels off rows of whole 32s or onto more than 64
# channels: the plane tiles of one and two planes, 4 and 8 rows, 32 and 64
# columns (with partial ones), odd depths (a tile's second plane past the
# volume), and enough tiles for the largest kind
PLANES = [
    dict(n=1, d=1, h=1, w=1, ci=64, co=8),
    dict(n=2, d=3, h=5, w=7, ci=256, co=40),
    dict(n=1, d=5, h=9, w=17, ci=128, co=72),
    dict(n=2, d=2, h=8, w=32, ci=64, co=96),
    dict(n=4, d=33, h=16, w=18, ci=64, co=64),
]


@pytest.mark.parametrize("case", range(len(PLANES)))
def test_stride1_plane_tiles(case):
    _check(PLANES[case], 200 + case)


def test_forward_does_not_depend_on_the_tile_sizes():
    """The same sample alone and as part of a batch large enough for other tile sizes: bit for bit."""
    from paper_1007_1388_amd import surrogate as S
    for ci, co, d, h, w in ((64, 32, 6, 18, 40), (32, 32, 9, 17, 33), (128, 96, 4, 16, 16)):
        rng = np.random.default_rng(ci + w)
        x = conv.bf16_round(rng.standard_normal((24, d, h, w, ci)))
        layer = S.Conv(ci, co, relu=True, seed=5)
        X, Y = S.from_numpy(x), S.Act(24, d, h, w, co)
        layer.forward(X, Y)
        X1, Y1 = S.from_numpy(x[3:4]), S.Act(1, d, h, w, co)
        layer.forward(X1, Y1)
        assert np.array_equal(Y.to_numpy()[3:4], Y1.to_numpy())


# weight gradients: rows of 32, 16 and 8 voxels (one, two and four planes, a
# partial last group of planes), partial rows and row blocks, channel tiles of
# 32 and 64 (partial ones), channels off 32, both strides, one voxel, and a
# volume that is split over several workgroups
WGRADS = [
    dict(n=1, d=1, h=1, w=1, ci=16, co=8),
    dict(n=2, d=3, h=5, w=31, ci=24, co=40),
    dict(n=1, d=5, h=9, w=16, ci=40, co=64),
    dict(n=1, d=7, h=3, w=7, ci=32, co=72),
    dict(n=2, d=4, h=17, w=33, ci=32, co=32),
    dict(n=1, d=5, h=7, w=9, ci=40, co=24, s=2),
    dict(n=3, d=13, h=21, w=43, ci=40, co=24, s=2),
    dict(n=1, d=9, h=6, w=33, ci=32, co=72, s=2),
    dict(n=1, d=3, h=9, w=65, ci=16, co=64, s=2),
    dict(n=2, d=16, h=32, w=32, ci=32, co=32),
]


# the 8-channel layer's weight gradient alike, and pointwise layers: voxel counts
# off the 64- and 256-voxel pieces, channels on and off 32
WGRADS += [
    dict(n=1, d=2, h=9, w=33, ci=8, co=40),
    dict(n=2, d=3, h=4, w=17, ci=8, co=8),
    dict(n=1, d=7, h=19, w=5, ci=8, co=32),
    dict(n=1, d=1, h=1, w=1, ci=8, co=8, k=1),
    dict(n=2, d=5, h=9, w=13, ci=40, co=72, k=1),
    dict(n=1, d=16, h=32, w=33, ci=32, co=8, k=1),
]


@pytest.mark.parametrize("case", range(len(WGRADS)))
def test_weight_gradient_row_steps(case):
    from paper_1007_1388_amd import surrogate as S
    c = WGRADS[case]
    k, s = c.get("k", 3), c.get("s", 1)
    x, w, b, dy = _operands(c, 300 + case)
    layer = S.Conv(c["ci"], c["co"], k=k, stride=s)
    layer.zero_grad()
    layer.backward(_sliced(S, x, 8, 16), _sliced(S, dy, 16, 24), None)
    dw, db = conv.conv3d_bwd_weight(x, dy, k, s)
    gw, K = layer.gw.cpu().numpy(), k ** 3 * c["ci"]
    assert np.abs(gw[:, :K].reshape(dw.shape) - dw).max() <= 1e-5 * np.abs(dw).max()
    assert np.all(gw[:, K:] == 0)
    assert np.abs(layer.gb.cpu().numpy() - db).max() <= 1e-5 * np.abs(db).max()


POINTS = [dict(n=1, d=1, h=1, w=1, ci=8, co=8, k=1), dict(n=2, d=5, h=9, w=13, ci=40, co=72, k=1),
          dict(n=1, d=4, h=8, w=8, ci=64, co=24, k=1), dict(n=1, d=7, h=5, w=11, ci=8, co=32, k=1)]


@pytest.mark.parametrize("case", range(len(POINTS)))
def test_pointwise(case):
    _check(POINTS[case], 400 + case)


# stride-2 input gradients of 32 and 64 channels: odd and even extents (the last
# odd voxel missing), partial tiles of 16 columns and 8 rows, partial columns;
# the last two stay with the tap-major kernel (tiles badly filled, 128 channels)
UPS = [
    dict(n=1, d=1, h=9, w=17, ci=8, co=32, s=2),
    dict(n=2, d=4, h=32, w=34, ci=40, co=32, s=2),
    dict(n=1, d=5, h=15, w=64, ci=24, co=64, s=2),
    dict(n=3, d=3, h=25, w=31, ci=72, co=64, s=2),
    dict(n=1, d=6, h=18, w=7, ci=32, co=64, s=2),
    dict(n=1, d=3, h=16, w=32, ci=72, co=128, s=2),
]


@pytest.mark.parametrize("case", range(len(UPS)))
def test_stride2_input_gradient(case):
    _check(UPS[case], 500 + case)
