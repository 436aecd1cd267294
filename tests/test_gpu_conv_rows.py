"""The row-staged convolution (any filter size, channel count and alignment): every instance, bit-exact on integers."""
import numpy as np
import pytest

from oracle import ops
from paper_2502_11407_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


def _rows_instances(gs, p):
    out = []
    for idx in range(gs.num_instances()):
        s = gs.instance_schedule(idx, p)
        if s is not None and s.direct_lds and s.vec_bytes != 16:
            out.append(s)
    return out


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("geom", [
    # n, c, h, w, k, r, s, stride, pad
    (3, 3, 33, 31, 70, 7, 7, 2, 3),       # image layer, ragged filters, odd rows, tiles over several images
    (1, 1, 9, 300, 5, 5, 5, 1, 2),        # one channel, rows longer than a tile
    (2, 7, 13, 12, 33, 3, 3, 1, 1),       # odd channel count: the last chunk of a stage is the zero one
    (2, 5, 11, 17, 32, 1, 1, 3, 1),       # one tap per channel
    (1, 4, 20, 21, 16, 2, 9, 1, 4),       # a filter row of two chunks (three for fp32)
    (1, 2, 40, 40, 8, 17, 17, 2, 0),      # three (five) chunks, a filter almost as large as the image
    (4, 40, 6, 6, 64, 5, 5, 1, 2),        # several channel stages, the last one partial; tiny images
    (1, 3, 8, 8, 130, 3, 3, 1, 5),        # padding wider than the filter needs
])
def test_every_row_staged_instance_bit_exact(gs, dtype, geom):
    import torch
    n, c, h, w, k, r, s, stride, pad = geom
    I = inputs.small_ints(71, (n, c, h, w), dtype, -2, 2)
    W = inputs.small_ints(72, (k, c, r, s), dtype, -2, 2)
    want = ops.conv2d(I, W, dtype, stride=stride, pad=pad)
    assert np.abs(want).max() < 2 ** 22
    p = gs.conv_problem(dtype, n, c, h, w, k, r, s, stride, pad)
    scheds = _rows_instances(gs, p)
    assert scheds
    dI, dW = gs.to_device(I, dtype), gs.to_device(W, dtype)
    oI, oW = (torch.empty(t.numel() + 3, dtype=t.dtype, device="cuda").fill_(float("inf")) for t in (dI, dW))
    oI[1:1 + dI.numel()] = dI.view(-1)     # the same operands one element off, infinities around them
    oW[1:1 + dW.numel()] = dW.view(-1)
    for sch in scheds:
        print("row-staged instance", sch.kernel_id, geom, dtype, flush=True)
        for a, b in ((dI, dW), (oI[1:], oW[1:])):
            O = gs.empty_device(want.shape).fill_(float("nan"))
            gs.conv2d(p, a, b, O, sch)
            torch.cuda.synchronize()
            assert np.array_equal(gs.to_host_f64(O), want), sch.kernel_id
    O = gs.empty_device(want.shape).fill_(float("nan"))
    gs.conv2d(p, dI, dW, O, None, gs.conv_workspace(p))
    assert np.array_equal(gs.to_host_f64(O), want)


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("r,s,pad", [(7, 7, 3), (5, 3, 1), (1, 5, 2)])
def test_infinities_reach_only_the_windows_that_hold_them(gs, dtype, r, s, pad):
    """The chunk a filter row is padded to reads input next to the window; a filter row's neighbour is another filter."""
    import torch
    n, c, h, w, k = 2, 3, 14, 19, 24
    I = inputs.small_ints(73, (n, c, h, w), dtype, 1, 3)
    W = inputs.small_ints(74, (k, c, r, s), dtype, 1, 2)
    I[0, 1, 6, 9] = I[1, 0, 0, w - 1] = np.inf
    p = gs.conv_problem(dtype, n, c, h, w, k, r, s, 1, pad)
    want = ops.conv2d(I, W, dtype, stride=1, pad=pad)
    for sch in _rows_instances(gs, p):
        O = gs.empty_device(want.shape).fill_(float("nan"))
        gs.conv2d(p, gs.to_device(I, dtype), gs.to_device(W, dtype), O, sch)
        assert np.array_equal(gs.to_host_f64(O), want), sch.kernel_id


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_16_bit_output_is_the_rounded_fp32_output(gs, dtype):
    p32 = gs.conv_problem(dtype, 2, 3, 30, 29, 40, 5, 5, 1, 2)
    p16 = gs.conv_problem(dtype, 2, 3, 30, 29, 40, 5, 5, 1, 2, dtype)
    dI, dW = gs.to_device(inputs.normal(75, (2, 3, 30, 29), dtype), dtype), gs.to_device(inputs.normal(76, (40, 3, 5, 5), dtype), dtype)
    for a, b in zip(_rows_instances(gs, p32), _rows_instances(gs, p16)):
        O32, O16 = gs.empty_device((2, 40, 30, 29)), gs.empty_device((2, 40, 30, 29), dtype)
        gs.conv2d(p32, dI, dW, O32, a)
        gs.conv2d(p16, dI, dW, O16, b)
        assert (a.tile[0][0], a.tile[1][0]) == (b.tile[0][0], b.tile[1][0])
        assert (O32.to(O16.dtype) == O16).all().item()
