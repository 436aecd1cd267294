"""16-bit outputs are stored as dwords of two columns where the launch allows it (even N and ldc, C on a dword), element by
element otherwise.  Every 16-bit-output instance over tiles with ragged last rows and columns, at leading dimensions and
addresses on both sides of that rule: small integers, so that every result is exact, and nothing outside C is written."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

TORCH = {"f16": "float16", "bf16": "bfloat16"}


def _instances(gs, dtype, tb):
    p = gs.gemm_problem(dtype, 64, 64, 128, 0, tb, 1, dtype)
    found = [(i, gs.instance_schedule(i, p)) for i in range(gs.num_instances())]
    return [(i, s) for i, s in found if s is not None]


@pytest.mark.parametrize("N,pad,offset", [(264, 0, 0), (264, 2, 1), (258, 0, 0), (258, 2, 2), (258, 1, 0), (258, 2, 1), (257, 1, 0), (34, 0, 0), (2, 0, 0), (1, 1, 0)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_every_16_bit_output_instance(dtype, N, pad, offset):
    from paper_2502_11407_amd import binding as gs
    td = getattr(torch, TORCH[dtype])
    M, K, ldc, seen = 261, 128, N + pad, 0
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    A = torch.randint(-1, 2, (M, K), device="cuda", generator=g).to(td)
    B = torch.randint(-1, 2, (N, K), device="cuda", generator=g).to(td)
    want = (A.double() @ B.double().t().contiguous()).to(td)             # at most 128 in magnitude: exact in both types
    for tb in ((0, 1) if N % 8 == 0 else (1,)):
        p = gs.gemm_problem(dtype, M, N, K, 0, tb, 1, dtype)
        for idx, s in _instances(gs, dtype, tb):
            buf = torch.full((M * ldc + 16,), 3.0, device="cuda").to(td)
            C = buf[offset:offset + M * ldc].view(M, ldc)
            gs.gemm(p, A, B if tb else B.t().contiguous(), C, schedule=s, ldc=ldc)
            assert torch.equal(C[:, :N], want), (idx, dtype, N, pad, offset)
            rest = buf.clone()
            rest[offset:offset + M * ldc].view(M, ldc)[:, :N] = 3.0
            assert bool((rest == 3.0).all()), (idx, "wrote outside C")
            seen += 1
    assert seen >= 4


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_rounding_is_to_nearest_even(dtype):
    """The paired conversion rounds like the element one: the same product stored by both (C off a dword boundary or not)."""
    from paper_2502_11407_amd import binding as gs
    td = getattr(torch, TORCH[dtype])
    M, N, K = 256, 256, 192
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    A = torch.randn((M, K), device="cuda", generator=g).to(td)
    B = torch.randn((N, K), device="cuda", generator=g).to(td)
    p = gs.gemm_problem(dtype, M, N, K, 0, 1, 1, dtype)
    for idx, s in _instances(gs, dtype, 1):
        even = torch.empty((M, N), device="cuda", dtype=td)
        odd = torch.empty((M * N + 1,), device="cuda", dtype=td)[1:].view(M, N)
        gs.gemm(p, A, B, even, schedule=s)
        gs.gemm(p, A, B, odd, schedule=s)
        assert torch.equal(even, odd), idx
        assert torch.equal(even, (A.double() @ B.double().t().contiguous()).float().to(td)) or \
            ((even.double() - A.double() @ B.double().t().contiguous()).norm() / even.double().norm()).item() < 2.0 ** -8, idx
