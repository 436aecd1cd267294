"""AvgPooling on both sides of the sizes from which inputs are read, and up to which fp32 outputs are stored, past the caches, beside the same planes
pooled a few at a time."""
import pytest

pytestmark = pytest.mark.gpu


# planes on both sides of the size, the last of them ending inside a 16-byte vector, a workgroup's share not dividing them
@pytest.mark.parametrize("dtype,out,planes,h,w,f,stride", [
    ("f16", "f32", 19501, 83, 83, 2, 2), ("f16", "f32", 19481, 83, 83, 2, 2), ("bf16", "bf16", 149331, 29, 31, 3, 2), ("f32", "f32", 152203, 21, 21, 3, 1),
    ("f16", "f16", 12001, 106, 107, 2, 2),
    # outputs of 1 KiB a plane: 32 MiB (16-bit input) and 16 MiB (fp32), and a plane more
    ("f16", "f32", 32768, 33, 33, 2, 2), ("bf16", "f32", 32769, 33, 33, 2, 2), ("f32", "f32", 16384, 33, 33, 2, 2), ("f32", "f32", 16385, 33, 33, 2, 2)])
def test_large_pools_equal_pools_of_their_planes(dtype, out, planes, h, w, f, stride):
    import torch
    from paper_2502_11407_amd import binding as gs
    TYPES = dict(f32=torch.float32, f16=torch.float16, bf16=torch.bfloat16)
    g = torch.Generator(device="cuda")
    g.manual_seed(planes)
    x = torch.randint(-8, 9, (1, planes, h, w), generator=g, device="cuda").to(TYPES[dtype])
    P, Q = (h - f) // stride + 1, (w - f) // stride + 1
    O = torch.full((1, planes, P, Q), float("nan"), dtype=TYPES[out], device="cuda")
    print("pool", dtype, out, planes, h, w, f, stride, x.numel() * x.element_size(), flush=True)
    gs.avgpool2d(dtype, x, O, f, stride, out)
    for a in (0, planes // 2 & ~7, (planes & ~7) - 64):
        n = min(200, planes - a)
        part = torch.empty((1, n, P, Q), dtype=O.dtype, device="cuda")
        gs.avgpool2d(dtype, x[:, a:a + n].contiguous(), part, f, stride, out)
        assert torch.equal(O[:, a:a + n], part)
    # small whole numbers: their sums are exact, and the quotient is rounded once to fp32 and once to the output.  (torch divides fp32 by a
    # number as a product with its reciprocal, up to 1.5 units in the last place away; from 64 bits, where no quotient of whole numbers
    # below 2^8 lies within 2^-29 of the middle between two fp32 numbers, the rounding to fp32 is the same as that of the quotient)
    total = sum(x[:, :, i:i + stride * (P - 1) + 1:stride, j:j + stride * (Q - 1) + 1:stride].float() for i in range(f) for j in range(f))
    assert torch.equal(O, (total.double() / (f * f)).float().to(O.dtype))
