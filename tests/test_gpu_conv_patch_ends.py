"""Patch-staged convolutions of odd rows, whose last vectors would run past the end of the input: every instance that takes the layer,
bit-exact on integers, with infinities right behind the input; down to inputs of a single vector."""
import numpy as np
import pytest

from oracle import ops
from paper_2502_11407_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


@pytest.mark.parametrize("dtype,out", [("f16", "f32"), ("bf16", "f32"), ("f16", "f16"), ("f32", "f32")])
@pytest.mark.parametrize("n,c,h,w,k,stride", [
    (1, 8, 1, 1, 8, 1),          # one vector of 16-bit elements: every channel's runs past the end
    (1, 8, 2, 3, 33, 1),         # rows shorter than a vector
    (2, 16, 5, 7, 64, 1),
    (3, 24, 9, 13, 40, 2),       # a partial channel stage behind it
    (1, 72, 15, 53, 65, 1),      # more channels than one stage of any depth
    (5, 40, 17, 31, 130, 2),
    (2, 136, 6, 9, 32, 1),
])
def test_inputs_end_inside_a_vector(gs, dtype, out, n, c, h, w, k, stride):
    import torch
    I = inputs.small_ints(31, (n, c, h, w), dtype, -1, 1)
    W = inputs.small_ints(32, (k, c, 3, 3), dtype, -1, 1)
    want = ops.conv2d(I, W, dtype, stride=stride, pad=1)
    p = gs.conv_problem(dtype, n, c, h, w, k, 3, 3, stride, 1, out)
    dI, dW = gs.to_device(I, dtype), gs.to_device(W, dtype)
    buf = torch.empty(dI.numel() + 64, dtype=dI.dtype, device="cuda").fill_(float("inf"))
    buf[:dI.numel()] = dI.view(-1)
    O = gs.empty_device(want.shape, out)
    expect = torch.from_numpy(np.asarray(want, dtype=np.float32)).cuda().to(O.dtype)
    ran = 0
    for idx in range(gs.num_instances()):
        s = gs.instance_schedule(idx, p)
        if s is None or not s.direct_lds or s.vec_bytes != 16:
            continue
        print("patch instance", idx, (n, c, h, w, k), "stride", stride, dtype, out, flush=True)
        O.fill_(float("nan"))
        gs.conv2d(p, buf, dW, O, s)
        torch.cuda.synchronize()
        assert torch.equal(O, expect), idx
        ran += 1
    assert ran
