"""Operands that start anywhere on an element boundary, with odd leading dimensions and extents: every GEMM instance
that does not ask for aligned vectors, bit-exact on integers, with infinities stored in every element around the
operands (an element from beyond K must not reach a product: infinity times zero is not zero)."""
import numpy as np
import pytest

from oracle import ops
from paper_2502_11407_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


def _embed(gs, x, dtype, offset, pad, tail):
    """x as a strided view inside a buffer of infinities: `offset` elements before it, rows `pad` elements longer than
    they need to be, `tail` elements after its last one (0: the buffer ends with it)."""
    import torch
    r, c = x.shape
    ld = c + pad
    buf = gs.empty_device((offset + (r - 1) * ld + c + tail,), dtype).fill_(float("inf"))
    view = torch.as_strided(buf, (r, c), (ld, 1), offset)
    view.copy_(gs.to_device(x, dtype))
    return view


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("k_of", [lambda bk: 1, lambda bk: 3, lambda bk: bk - 1, lambda bk: bk, lambda bk: bk + 2, lambda bk: 2 * bk + 1,
                                  lambda bk: 3 * bk - 6], ids=["1", "3", "bk-1", "bk", "bk+2", "2bk+1", "3bk-6"])
def test_gemm_at_any_alignment_bit_exact(gs, dtype, ta, tb, k_of):
    import torch
    ran = 0
    for out in ([dtype, "f32"] if dtype != "f32" else ["f32"]):
        for idx in range(gs.num_instances()):
            s = gs.instance_schedule(idx, gs.gemm_problem(dtype, 64, 64, 64, ta, tb, 1, out))
            if s is None or s.vec_bytes == 16:
                continue
            bm, bn, bk = s.tile[0][0], s.tile[1][0], s.tile[2][0]
            M, N, K = bm + 1, bn + 3, k_of(bk)
            print("instance", idx, dtype, out, (M, N, K), "transA", ta, "transB", tb, flush=True)
            A = inputs.small_ints(10 + idx, (K, M) if ta else (M, K), dtype, -1, 1)
            B = inputs.small_ints(20 + idx, (N, K) if tb else (K, N), dtype, -1, 1)
            want = ops.gemm(A, B, dtype, transA=ta, transB=tb)
            for offset, pad, tail in ((0, 0, 0), (3, 1, 0), (1, 0, 5), (2, 4, 1)):
                dA, dB = _embed(gs, A, dtype, offset, pad, tail), _embed(gs, B, dtype, offset + 1, pad, tail)
                C = gs.empty_device((M, N), out).fill_(float("nan"))
                gs.gemm(gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out), dA, dB, C, schedule=s, lda=A.shape[1] + pad, ldb=B.shape[1] + pad)
                torch.cuda.synchronize()
                assert np.array_equal(gs.to_host_f64(C), want), (idx, offset, pad, tail)
            ran += 1
    assert ran >= 2


@pytest.mark.parametrize("dtype", ["f16", "f32"])
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (2, 3, 1), (1, 5, 9), (3, 1, 70), (5, 2, 2)])
def test_tiny_operands_bit_exact(gs, dtype, M, N, K):
    """Whole operands smaller than one vector."""
    for tb in (0, 1):
        A, B = inputs.small_ints(1, (M, K), dtype, -3, 3), inputs.small_ints(2, (N, K) if tb else (K, N), dtype, -3, 3)
        C = gs.empty_device((M, N)).fill_(float("nan"))
        gs.gemm(gs.gemm_problem(dtype, M, N, K, 0, tb), gs.to_device(A, dtype), gs.to_device(B, dtype), C)
        assert np.array_equal(gs.to_host_f64(C), ops.gemm(A, B, dtype, transB=tb))


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("M", [1, 2, 3, 9])
@pytest.mark.parametrize("vectors,extra", [(0, 1), (1, 0), (63, 3), (255, 1), (256, 0), (257, 1), (1024, 1), (1300, 3)])
def test_gemv_at_any_alignment_bit_exact(gs, dtype, M, vectors, extra):
    """Rows around the length from which four waves share them, at odd offsets and leading dimensions, with infinities
    around the matrix and the vector."""
    import torch
    N = vectors * (4 if dtype == "f32" else 8) + extra
    A, x = inputs.small_ints(81, (M, N), dtype, -2, 2), inputs.small_ints(82, (1, N), dtype, -2, 2)
    want = ops.gemv(A, x[0], dtype)
    for offset, pad in ((0, 0), (1, 0), (3, 5)):
        dA, dx = _embed(gs, A, dtype, offset, pad, 2), _embed(gs, x, dtype, 2 * offset + 1, 0, 1)[0]
        y = torch.full((M,), float("nan"), dtype=torch.float32, device="cuda")
        gs.gemv(dtype, dA, dx, y, lda=N + pad)
        assert np.array_equal(gs.to_host_f64(y), want), (offset, pad)
        y0 = inputs.small_ints(83, (M,), "f32", -4, 4)
        y = gs.to_device(y0, "f32")
        gs.gemv(dtype, dA, dx, y, 2.0, -1.0, lda=N + pad)
        assert np.array_equal(gs.to_host_f64(y), 2.0 * want - y0)


def test_gemv_with_more_rows_than_a_launch_holds_at_two_a_workgroup(gs):
    """2^25 rows of 256 vectors, 128 GiB."""
    import torch
    M, N = 2 ** 25, 2048
    if torch.cuda.mem_get_info()[0] < 150 * 10 ** 9:
        pytest.skip("needs 150 GB of device memory")
    A = gs.empty_device((M, N), "f16").fill_(1.0)
    A[M // 2], A[M - 1] = 3.0, 2.0
    y = gs.empty_device((M,)).fill_(float("nan"))
    gs.gemv("f16", A, torch.ones(N, dtype=torch.float16, device="cuda"), y)
    del A
    torch.cuda.empty_cache()
    assert y[M // 2].item() == 3 * N and y[M - 1].item() == 2 * N
    y[M // 2] = y[M - 1] = N
    assert (y == N).all().item()


@pytest.mark.parametrize("beta", [0.0, -1.0])
def test_large_output_with_rows_off_the_lines_bit_exact(gs, beta):
    """More than 32 MiB of 16-bit output whose rows do not start on 128-byte lines: stored write-back."""
    M, N, K = 4099, 4104, 16
    A, B = inputs.small_ints(91, (M, K), "f16", -3, 3), inputs.small_ints(92, (N, K), "f16", -3, 3)
    C0 = inputs.small_ints(93, (M, N), "f16", -4, 4)
    C = gs.to_device(C0, "f16")
    gs.gemm(gs.gemm_problem("f16", M, N, K, 0, 1, 1, "f16"), gs.to_device(A, "f16"), gs.to_device(B, "f16"), C, 1.0, beta)
    want = ops.gemm(A, B, "f16", transB=1, alpha=1.0, beta=beta, C0=C0.astype(np.float32))
    assert np.array_equal(gs.to_host_f64(C), want)


@pytest.mark.parametrize("dtype,out,M,N,K,ta,tb,lda,ldb", [
    ("f16", "f32", 201, 300, 1003, 1, 1, 20000001, None),
    ("bf16", "bf16", 70, 301, 203, 0, 0, None, 20000001),
    ("f32", "f32", 40, 131, 99, 0, 0, None, 20000001),
    ("f16", "f32", 130, 5000001, 71, 0, 0, None, None),            # output rows of 20 MB
    ("f16", "f32", 48, 304, 64, 0, 1, 20000000, None),             # aligned operands
    ("bf16", "bf16", 72, 304, 40, 0, 0, None, 20000000),
    ("f16", "f32", 304, 72, 40, 1, 1, 20000000, None),
    ("f32", "f32", 130, 600, 96, 0, 1, 12000000, None),
])
def test_leading_dimensions_beyond_the_larger_tiles(gs, dtype, out, M, N, K, ta, tb, lda, ldb):
    """Rows so far apart that the 32-bit offsets inside a large tile do not reach: a smaller tile takes them (operands on and off the
    vector boundaries)."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(101)

    def ints(rows, cols, ld):
        buf = gs.empty_device(((rows - 1) * (ld or cols) + cols,), dtype)
        view = torch.as_strided(buf, (rows, cols), (ld or cols, 1))
        return view.copy_(torch.randint(-1, 2, (rows, cols), generator=gen, device="cuda", dtype=torch.int8))

    A, B = ints(*((K, M) if ta else (M, K)), lda), ints(*((N, K) if tb else (K, N)), ldb)
    C = gs.empty_device((M, N), out)
    p = gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out)
    fa, b = (A.T if ta else A).float(), B.T if tb else B
    for s in (None, gs.construct(p)):
        C.fill_(float("nan"))
        gs.gemm(p, A, B, C, 1.0, 0.0, s, workspace=gs.gemm_workspace(p, s) if s is not None else None)
        for n in range(0, N, 1000000):       # sums of at most 203 ones: exact in fp32, and rounded to bf16
            assert (C[:, n:n + 1000000].float() == fa @ b[:, n:n + 1000000].float()).all().item(), n


@pytest.mark.parametrize("beta", [0.0, -1.0])
@pytest.mark.parametrize("N", [4096, 4100], ids=["rows on the lines", "rows off the lines"])
def test_large_fp32_output_bit_exact(gs, N, beta):
    """64 MiB of fp32 output and more: write-through with and without beta, write-back where rows start off the 128-byte lines."""
    M, K = 4101, 192
    A, B = inputs.small_ints(94, (M, K), "f16", -3, 3), inputs.small_ints(95, (N, K), "f16", -3, 3)
    C0 = inputs.small_ints(96, (M, N), "f32", -4, 4)
    C = gs.to_device(C0, "f32")
    gs.gemm(gs.gemm_problem("f16", M, N, K, 0, 1), gs.to_device(A, "f16"), gs.to_device(B, "f16"), C, 1.0, beta)
    assert np.array_equal(C.cpu().numpy(), A.astype(np.float32) @ B.astype(np.float32).T + beta * C0)      # integers: exact in fp32
