"""Every convolution kernel that the choice by shape can reach, with the choice
asserted: against the FP64 reference, and against the other kernels that take
the same products, bit for bit where they are said to agree.

Outputs are BF16, rounded once (2^-9 of the value), of FP32 sums of at most
27 * 256 products of random signs (off by about sqrt(27 * 256 / 2) * 2^-24, under
2^-18 of their size): within 2^-8 of the largest reference value."""
import numpy as np
import pytest

from oracle import conv
from tests.test_gpu_conv_narrow import _forward, _gradient, _operands
from tests.test_gpu_conv_tiles import TOL

pytestmark = pytest.mark.gpu


# gathered and output channels, sample size, batch, the kernel of the batch and
# of one sample: the three plane tiles of 64, 128 and 256 channels with partial
# rows, columns, planes and column tiles, the tap-major kernel on the same
# products, the row tiles of 8 and 16 rows with channels in 32s (one to three
# chunks) and in 8s
BATCHES = [
    (64, 72, (1, 9, 9), 96, "plane big", "plane small"),
    (64, 72, (1, 7, 9), 160, "plane mid", "plane small"),
    (64, 72, (3, 9, 7), 96, "tap", "plane small"),
    (128, 72, (1, 9, 9), 48, "plane big", "plane small"),
    (128, 72, (1, 7, 18), 48, "plane mid", "plane small"),
    (128, 72, (3, 9, 9), 48, "tap", "plane small"),
    (256, 72, (1, 9, 9), 24, "plane big", "plane small"),
    (256, 72, (1, 7, 9), 24, "plane mid", "plane small"),
    (256, 72, (1, 9, 7), 160, "tap", "plane small"),
    (32, 40, (3, 15, 33), 16, "rows4", "rows2"),
    (96, 72, (1, 31, 33), 16, "rows4", "rows2"),
    (64, 32, (1, 31, 32), 64, "rows4", "rows2"),
    (40, 72, (3, 15, 31), 16, "rows4", "rows2"),
]


@pytest.mark.parametrize("case", range(len(BATCHES)))
def test_forward_of_a_batch_and_of_one_sample(case):
    from paper_1007_1388_amd import surrogate as S
    c, o, dims, n, many, one = BATCHES[case]
    x, w, b, _ = _operands(n, *dims, c, o, 3, 1, 600 + case)
    layer = S.Conv(c, o, relu=True)
    layer.set_weights(w, b)
    got, kernel = _forward(S, layer, x)
    assert kernel == many
    for k in sorted({0, n // 2, n - 1}):
        ref = conv.conv3d(x[k:k + 1], w, b.astype(np.float64), 3, 1, True)
        assert np.abs(got[k:k + 1] - ref).max() <= TOL * np.abs(ref).max()
        alone, kernel = _forward(S, layer, x[k:k + 1])
        assert kernel == one and np.array_equal(got[k:k + 1], alone)


@pytest.mark.parametrize("case", range(len(BATCHES)))
def test_input_gradient_of_a_batch_and_of_one_sample(case):
    from paper_1007_1388_amd import surrogate as S
    c, o, dims, n, many, one = BATCHES[case]
    x, w, b, dy = _operands(n, *dims, o, c, 3, 1, 700 + case)
    prev = conv.bf16_round(np.random.default_rng(800 + case).standard_normal(x.shape))
    layer = S.Conv(o, c)
    layer.set_weights(w, b)
    got, kernel = _gradient(S, layer, dy, x, prev)
    assert kernel == many
    for k in sorted({0, n // 2, n - 1}):
        s = slice(k, k + 1)
        ref = prev[s] + conv.conv3d_bwd_data(dy[s], w, x[s].shape, 3, 1) * (x[s] > 0)
        assert np.abs(got[s] - ref).max() <= TOL * np.abs(ref).max()
        alone, kernel = _gradient(S, layer, dy[s], x[s], prev[s])
        assert kernel == one and np.array_equal(got[s], alone)


@pytest.mark.parametrize("dims,ci,co", [((3, 15, 31), 32, 32), ((5, 16, 33), 40, 32), ((1, 31, 64), 8, 32),
                                        ((3, 15, 31), 72, 64), ((2, 32, 63), 32, 64)])
def test_stride2_input_gradient_on_both_kernels(dims, ci, co):
    """All parities in one workgroup, and one parity at a time: the same layer with 96 output channels, those past co
    zero, whose products add zeros.  Odd extents: the last odd voxel is missing."""
    from paper_1007_1388_amd import surrogate as S
    x, w, b, dy = _operands(2, *dims, ci, co, 3, 2, 900 + ci + co)
    prev = conv.bf16_round(np.random.default_rng(9).standard_normal(x.shape))
    layer, wide = S.Conv(ci, co, stride=2), S.Conv(ci, 96, stride=2)
    layer.set_weights(w, b)
    wide.set_weights(np.concatenate([w, np.zeros((96 - co,) + w.shape[1:])]), np.zeros(96))
    got, kernel = _gradient(S, layer, dy, x, prev)
    assert kernel == "up"
    ref = prev + conv.conv3d_bwd_data(dy, w, x.shape, 3, 2) * (x > 0)
    assert np.abs(got - ref).max() <= TOL * np.abs(ref).max()
    other, kernel = _gradient(S, wide, np.concatenate([dy, np.zeros(dy.shape[:4] + (96 - co,))], -1), x, prev)
    assert kernel == "tap" and np.array_equal(got, other)
