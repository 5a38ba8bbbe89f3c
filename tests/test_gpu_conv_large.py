"""Convolutions on channel slices of buffers just under 2 GiB, where byte offsets
come within 2 KiB of the bit that marks a load as out of range, against the same
layer on the last planes alone: outputs and input gradients bit for bit (a
kernel's sums do not depend on the volume), weight gradients of the same
products grouped otherwise to 1e-5 of the largest, as in the other tests."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

D, H, W, LDC = 2048, 16, 32, 1024   # 2^20 voxels of 2 KiB; the slice ends the buffer
CUT = 8                             # planes of the small volume


def _wide(S, planes, c, rows):
    """Zeros but for the last `planes` planes of the last c channels; and those planes alone."""
    import torch
    buf = torch.zeros((1, D, H, W, LDC), dtype=torch.int16, device="cuda")
    buf[0, D - planes:, :, :, LDC - c:] = rows[0, -planes:]
    return S.Act(1, D, H, W, c, buf=buf, off=LDC - c, ldc=LDC)


def _rows(c, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randn((1, CUT, H, W, c), generator=g, device="cuda").bfloat16().view(torch.int16)


def _alone(S, rows):
    a = S.Act(1, CUT, H, W, rows.shape[-1])
    a.buf.copy_(rows)
    return a


@pytest.mark.parametrize("ci,co,k,s,kernel", [(32, 32, 3, 1, "rows4"), (24, 32, 3, 1, "rows4"), (64, 72, 3, 1, "plane"),
                                              (8, 32, 3, 1, "c8"), (40, 24, 1, 1, "point"), (32, 40, 3, 2, "tap")])
def test_forward(ci, co, k, s, kernel):
    import torch
    from paper_1007_1388_amd import surrogate as S
    rows = _rows(ci, 1)
    x, small = _wide(S, CUT, ci, rows), _alone(S, rows)
    layer = S.Conv(ci, co, k=k, stride=s, seed=2)
    out = lambda d: S.Act(1, -(-d // s), -(-H // s), -(-W // s), co)
    y, part = out(D), out(CUT)
    assert S.kernel_of("forward", x, y, k, s).startswith(kernel)
    layer.forward(x, y)
    layer.forward(small, part)
    assert torch.equal(y.buf[:, -CUT // s + 1:], part.buf[:, 1:]) and part.buf.any()


@pytest.mark.parametrize("c,ci,k,s,kernel", [(32, 32, 3, 1, "rows4"), (40, 32, 3, 1, "rows4"), (64, 72, 3, 1, "plane"),
                                             (32, 24, 1, 1, "point"), (32, 8, 3, 2, "up"), (64, 16, 3, 2, "up"),
                                             (96, 8, 3, 2, "tap")])
def test_input_gradient(c, ci, k, s, kernel):
    import torch
    from paper_1007_1388_amd import surrogate as S
    rows = _rows(c, 3)
    dy, small = _wide(S, CUT, c, rows), _alone(S, rows)
    layer = S.Conv(ci, c, k=k, stride=s, seed=4)
    dx, part = (S.Act(1, d * s, H * s, W * s, ci) for d in (D, CUT))
    assert S.kernel_of("input gradient", dx, dy, k, s).startswith(kernel)
    for g, d in ((dy, dx), (small, part)):
        assert S.lib().lbm_conv3d_bwd_data(g.ref, layer.wt.data_ptr(), d.ref, None, k, s, 0, None) == 0
    assert torch.equal(dx.buf[:, -(CUT - 1) * s:], part.buf[:, s:]) and part.buf.any()


@pytest.mark.parametrize("ci,co,k,kernel", [(32, 64, 3, "wgrad rows64"), (40, 32, 3, "wgrad rows32"),
                                            (8, 32, 3, "wgrad c8"), (32, 8, 1, "wgrad point")])
def test_weight_gradient(ci, co, k, kernel):
    """Once with x, once with dy the large one; only the last planes of dy are not zero."""
    import torch
    from paper_1007_1388_amd import surrogate as S
    xr, dr = _rows(ci, 5), _rows(co, 6)
    dr[:, 0] = 0    # (the plane before the small volume adds nothing)
    ref = S.Conv(ci, co, k=k)
    ref.backward(_alone(S, xr), _alone(S, dr), None)
    big = lambda c, r: _wide(S, CUT, c, r)

    def narrow(c, r):
        a = S.Act(1, D, H, W, c)
        a.buf[:, -CUT:] = r
        return a
    for x, dy in ((big(ci, xr), narrow(co, dr)), (narrow(ci, xr), big(co, dr))):
        assert S.kernel_of("weight gradient", x, dy, k, 1) == kernel
        layer = S.Conv(ci, co, k=k)
        layer.backward(x, dy, None)
        assert (layer.gw - ref.gw).abs().max() <= 1e-5 * ref.gw.abs().max() and ref.gw.any()
        assert (layer.gb - ref.gb).abs().max() <= 1e-5 * ref.gb.abs().max()


def test_views_of_two_gib_take_the_general_kernels():
    from paper_1007_1388_amd import surrogate as S
    x = S.lbm_tensor5(256, 1, D, H, W, 32, LDC)
    full = S.lbm_tensor5(256, 1, D, H, W, LDC, LDC)
    y = S.lbm_tensor5(256, 1, D, H, W, 32, 32)
    assert S.kernel_of("forward", x, y) == "rows4"       # (the last voxel's channels end short of 2 GiB)
    assert S.kernel_of("forward", full, y) == "general"
    assert S.kernel_of("input gradient", y, full) == "general"
    assert S.kernel_of("weight gradient", full, y) == "wgrad general"
