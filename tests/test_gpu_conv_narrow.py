"""Convolutions of volumes narrower than the kernels' tiles, about the lines where
the choice by shape changes, against the FP64 reference (bounds as in the other
convolution tests: 2^-8 of the largest BF16 output, 1e-5 of the largest FP32
weight gradient, here of at most 2^12 products)."""
import numpy as np
import pytest

from oracle import conv
from tests.test_gpu_conv_tiles import TOL, _sliced

pytestmark = pytest.mark.gpu


def _untouched(S, act, off, c):
    """The NaN channels on both sides of a slice are still NaN."""
    wide = S.Act(act.n, act.d, act.h, act.w, act.ldc, buf=act.buf, ldc=act.ldc).to_numpy()
    return np.isnan(wide[..., :off]).all() and np.isnan(wide[..., off + c:]).all()


def _operands(n, d, h, w, ci, co, k, s, seed):
    rng = np.random.default_rng(seed)
    x = conv.bf16_round(rng.standard_normal((n, d, h, w, ci)))
    wt = conv.bf16_round(rng.standard_normal((co, k ** 3, ci)) * 0.1)
    dy = conv.bf16_round(rng.standard_normal((n, -(-d // s), -(-h // s), -(-w // s), co)))
    return x, wt, rng.standard_normal(co).astype(np.float32), dy


def _forward(S, layer, x):
    y = _sliced(S, np.zeros((x.shape[0],) + tuple(-(-v // layer.stride) for v in x.shape[1:4]) + (layer.cout,)), 8, 16)
    X = _sliced(S, x, 8, 16)
    layer.forward(X, y)
    assert _untouched(S, y, 8, layer.cout)
    return y.to_numpy(), S.kernel_of("forward", X, y, layer.k, layer.stride)


def _gradient(S, layer, dy, x, prev):
    """dx added to prev and masked by ReLU'(x)."""
    X, DY, DX = _sliced(S, x, 8, 8), _sliced(S, dy, 16, 24), _sliced(S, prev, 8, 16)
    assert S.lib().lbm_conv3d_bwd_data(DY.ref, layer.wt.data_ptr(), DX.ref, X.ref, layer.k, layer.stride, 1, None) == 0
    assert _untouched(S, DX, 8, x.shape[-1])
    return DX.to_numpy(), S.kernel_of("input gradient", DX, DY, layer.k, layer.stride)


# volumes narrower than the tiles, about the lines where the kernels change
@pytest.mark.parametrize("dims,ci,co,forward,weight", [
    ((300, 1, 1), 24, 32, "general", "wgrad general"), ((300, 1, 1), 8, 32, "general", "wgrad general"),
    ((130, 2, 2), 40, 64, "general", "wgrad rows64"), ((130, 2, 2), 24, 32, "general", "wgrad rows32"),
    ((40, 4, 4), 24, 40, "general", "wgrad rows64"), ((37, 9, 3), 32, 32, "tap", "wgrad rows32"),
    ((40, 4, 7), 8, 40, "general", "wgrad c8"), ((40, 5, 9), 8, 40, "c8", "wgrad c8"),
    ((40, 4, 9), 40, 24, "rows2", "wgrad rows32"), ((300, 1, 1), 32, 64, "tap", "wgrad rows64"),
    ((65, 17, 1), 24, 32, "general", "wgrad rows32"),
])
def test_narrow_volumes(dims, ci, co, forward, weight):
    from paper_1007_1388_amd import surrogate as S
    x, w, b, dy = _operands(2, *dims, ci, co, 3, 1, 1000 + ci + co)
    layer = S.Conv(ci, co, relu=True)
    layer.set_weights(w, b)
    got, kernel = _forward(S, layer, x)
    assert kernel == forward
    ref = conv.conv3d(x, w, b.astype(np.float64), 3, 1, True)
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
    prev = conv.bf16_round(np.random.default_rng(9).standard_normal(x.shape))
    got, _ = _gradient(S, layer, dy, x, prev)
    ref = prev + conv.conv3d_bwd_data(dy, w, x.shape, 3, 1) * (x > 0)
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
    X, DY = _sliced(S, x, 8, 16), _sliced(S, dy, 16, 24)
    assert S.kernel_of("weight gradient", X, DY) == weight
    layer.zero_grad()
    layer.backward(X, DY, None)
    dw, db = conv.conv3d_bwd_weight(x, dy, 3, 1)
    gw = layer.gw.cpu().numpy()[:, :27 * ci].reshape(dw.shape)
    assert np.abs(gw - dw).max() <= 1e-5 * np.abs(dw).max()
    assert np.abs(layer.gb.cpu().numpy() - db).max() <= 1e-5 * np.abs(db).max()


# rows of one, two and four voxels of the stride-2 weight gradient, both channel tiles
@pytest.mark.parametrize("dims,ci,co", [((70, 9, 1), 32, 64), ((70, 16, 1), 64, 32), ((35, 11, 3), 32, 64),
                                        ((35, 11, 4), 32, 24), ((21, 13, 7), 32, 64), ((21, 13, 8), 64, 32)])
def test_narrow_stride2_weight_gradient(dims, ci, co):
    from paper_1007_1388_amd import surrogate as S
    x, w, b, dy = _operands(3, *dims, ci, co, 3, 2, 1100 + ci + co)
    layer = S.Conv(ci, co, stride=2)
    X, DY = _sliced(S, x, 8, 16), _sliced(S, dy, 16, 24)
    assert S.kernel_of("weight gradient", X, DY, 3, 2) == ("wgrad rows64" if co == 64 else "wgrad rows32")
    layer.backward(X, DY, None)
    dw, db = conv.conv3d_bwd_weight(x, dy, 3, 2)
    gw = layer.gw.cpu().numpy()[:, :27 * ci].reshape(dw.shape)
    assert np.abs(gw - dw).max() <= 1e-5 * np.abs(dw).max()
    assert np.abs(layer.gb.cpu().numpy() - db).max() <= 1e-5 * np.abs(db).max()


@pytest.mark.parametrize("c", [24, 32, 40, 56, 64])
def test_pointwise_in_place(c):
    from paper_1007_1388_amd import surrogate as S
    x, w, b, _ = _operands(2, 9, 31, 33, c, c, 1, 1, 1200 + c)
    layer = S.Conv(c, c, k=1)
    layer.set_weights(w, b)
    X, Y, DX = S.from_numpy(x), S.Act(2, 9, 31, 33, c), S.Act(2, 9, 31, 33, c)
    layer.forward(X, Y)
    assert S.lib().lbm_conv3d_bwd_data(X.ref, layer.wt.data_ptr(), DX.ref, None, 1, 1, 0, None) == 0
    for run, out in ((lambda a: layer.forward(a, a), Y), (lambda a: S.lib().lbm_conv3d_bwd_data(
            a.ref, layer.wt.data_ptr(), a.ref, None, 1, 1, 0, None), DX)):
        a = S.from_numpy(x)
        run(a)
        assert np.array_equal(a.to_numpy(), out.to_numpy())
