"""Training repeats: the gradients' sums have a fixed order, so the same steps
from the same weights give the same bits."""
import numpy as np
import pytest

from oracle import conv

pytestmark = pytest.mark.gpu


def _train(steps, shape, seed):
    """Weights, biases and the gradient at the first layer after `steps` training steps on fixed random data."""
    import torch
    from paper_1007_1388_amd import surrogate as S
    n, d, h, w = shape
    net = S.UNet(n, d, h, w, seed=seed)
    g = torch.Generator(device="cuda").manual_seed(seed)
    net.x.buf.copy_(torch.randn(net.x.buf.shape, generator=g, device="cuda").bfloat16().view(torch.int16))
    target = torch.randn((n * d * h * w, 4), generator=g, device="cuda")
    dpred, loss = S.Act(n, d, h, w, 8), torch.zeros(1, device="cuda")
    for _ in range(steps):
        pred = net.forward()
        assert S.lib().lbm_mse_loss(pred.ref, target.data_ptr(), None, 4, 1.0 / target.numel(), dpred.ref,
                                    loss.data_ptr(), None) == 0
        net.zero_grad()
        net.backward(dpred)
        net.adam(1e-4)
    torch.cuda.synchronize()
    return [t.clone() for l in net.layers for t in (l.w, l.b, l.gw, l.gb)] + [net.g["a0"].buf.clone()]


@pytest.mark.parametrize("shape", [(2, 64, 32, 32), (1, 24, 40, 56)])
def test_training_steps_repeat_bit_for_bit(shape):
    import torch
    a, b = _train(3, shape, 3), _train(3, shape, 3)
    assert all(torch.equal(u, v) for u, v in zip(a, b))


# one layer of every weight-gradient kernel, each split over many workgroups:
# row steps of both strides and channel tiles, the 8-channel layer, pointwise,
# and the general kernel (1x1x1 onto many tiles; stride 2 on channels off 32s)
LAYERS = [dict(n=2, d=24, h=20, w=33, ci=32, co=64), dict(n=1, d=30, h=24, w=24, ci=40, co=32),
          dict(n=2, d=25, h=31, w=30, ci=32, co=64, s=2), dict(n=2, d=25, h=31, w=30, ci=32, co=32, s=2),
          dict(n=2, d=16, h=24, w=40, ci=8, co=40), dict(n=1, d=30, h=33, w=31, ci=32, co=40, k=1),
          dict(n=2, d=60, h=80, w=80, ci=40, co=40, k=1), dict(n=1, d=21, h=29, w=29, ci=24, co=32, s=2)]


@pytest.mark.parametrize("case", range(len(LAYERS)))
def test_weight_gradients_repeat_and_agree_with_the_atomics(case):
    """Fixed-order sums: equal bits over five calls, and the atomics' sums to FP32 rounding (each side off by at most
    sqrt(n / 2) 2^-24 of a sum of n products of its own size: 1e-5 of the largest covers 2^17 products ten times over).
    A gradient is added to what dw holds, and the K padding of dw stays."""
    import torch
    from paper_1007_1388_amd import surrogate as S
    c = LAYERS[case]
    k, s = c.get("k", 3), c.get("s", 1)
    rng = np.random.default_rng(40 + case)
    x = S.from_numpy(rng.standard_normal((c["n"], c["d"], c["h"], c["w"], c["ci"])))
    dy = S.from_numpy(rng.standard_normal((c["n"],) + tuple(-(-c[a] // s) for a in "dhw") + (c["co"],)))
    L, got = S.lib(), []
    need = L.lbm_conv3d_bwd_weight_scratch(x.ref, dy.ref, k, s)
    assert need > 0
    for _ in range(5):
        layer = S.Conv(c["ci"], c["co"], k=k, stride=s)
        layer.scratch._bufs[(torch.cuda.current_device(), 0)] = torch.full((need,), 0xFF, dtype=torch.uint8, device="cuda")
        layer.gw.fill_(1.0)
        layer.backward(x, dy, None)
        got.append((layer.gw, layer.gb))
    for gw, gb in got[1:]:
        assert torch.equal(gw, got[0][0]) and torch.equal(gb, got[0][1])
    K = k ** 3 * c["ci"]
    gw, gb = torch.zeros_like(layer.gw), torch.zeros_like(layer.gb)
    assert L.lbm_conv3d_bwd_weight(x.ref, dy.ref, gw.data_ptr(), gb.data_ptr(), k, s, None) == 0
    assert torch.all(got[0][0][:, K:] == 1.0)
    # (adding to 1 rounds to 2^-24 of the result)
    tol = 1e-5 * gw.abs().max() + 2.0 ** -23
    assert (got[0][0][:, :K] - 1.0 - gw[:, :K]).abs().max() <= tol
    assert (got[0][1] - gb).abs().max() <= 1e-5 * gb.abs().max()


def test_scratch_is_checked_and_a_capture_allocates_nothing():
    import torch
    from paper_1007_1388_amd import lbm, surrogate as S
    rng = np.random.default_rng(5)
    x = S.from_numpy(rng.standard_normal((1, 12, 16, 32, 32)))
    dy = S.from_numpy(rng.standard_normal((1, 12, 16, 32, 32)))
    layer, L = S.Conv(32, 32), S.lib()
    need = L.lbm_conv3d_bwd_weight_scratch(x.ref, dy.ref, 3, 1)
    buf = torch.empty(need + 16, dtype=torch.uint8, device="cuda")
    args = (x.ref, dy.ref, layer.gw.data_ptr(), layer.gb.data_ptr(), 3, 1)
    for ptr, size in ((None, need), (buf.data_ptr(), need - 4), (buf.data_ptr() + 4, need)):
        assert L.lbm_conv3d_bwd_weight_ordered(*args, ptr, size, None) == lbm.LBM_EINVAL
    assert L.lbm_conv3d_bwd_weight_scratch(x.ref, dy.ref, 3, 2) == -1
    dw, db = conv.conv3d_bwd_weight(x.to_numpy(), dy.to_numpy(), 3, 1)
    for warm in (False, True):   # a graph holds no scratch memory, be it at hand or not
        layer = S.Conv(32, 32)
        stream = torch.cuda.Stream()
        if warm:
            layer.backward(x, dy, None, stream=stream.cuda_stream)
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            layer.backward(x, dy, None, stream=stream.cuda_stream)
        bufs = list(layer.scratch._bufs.values())
        assert len(bufs) == warm
        for buf in bufs:
            buf.fill_(0x55)
        for _ in range(3):
            layer.zero_grad()
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert np.abs(layer.gw.cpu().numpy()[:, :864].reshape(dw.shape) - dw).max() <= 1e-5 * np.abs(dw).max()
            assert np.abs(layer.gb.cpu().numpy() - db).max() <= 1e-5 * np.abs(db).max()
        assert all(bool((buf == 0x55).all()) for buf in bufs)


def test_scratch_of_streams_and_copies():
    """One buffer per stream, at most four kept, none in a copy; gradients on several streams agree bit for bit."""
    import copy
    import torch
    from paper_1007_1388_amd import surrogate as S
    rng = np.random.default_rng(6)
    x = S.from_numpy(rng.standard_normal((1, 12, 16, 32, 32)))
    dy = S.from_numpy(rng.standard_normal((1, 12, 16, 32, 32)))
    layer = S.Conv(32, 32)
    layer.backward(x, dy, None)
    torch.cuda.synchronize()
    want = layer.gw.clone()
    streams = [torch.cuda.Stream() for _ in range(6)]
    for st in streams:
        layer.zero_grad()
        torch.cuda.synchronize()
        layer.backward(x, dy, None, stream=st.cuda_stream)
        st.synchronize()
        assert torch.equal(layer.gw, want)
    assert len(layer.scratch._bufs) == S.Scratch.STREAMS
    assert len({b.data_ptr() for b in layer.scratch._bufs.values()}) == S.Scratch.STREAMS
    assert not copy.deepcopy(layer.scratch)._bufs
