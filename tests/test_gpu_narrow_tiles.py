"""The instances whose wave groups alternate, where a launch cuts C into tiles of 192 columns: at the depths where prologue, steady
state and drain of their slots differ, with ragged last rows, columns and k tiles, operands inside infinities, one column of
tiles and several, a launch on either side of the rule's line, alpha and beta, and a batch.  Small integers: every result is exact."""
import pytest

from test_gpu_alternating_groups import _in_infinities

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


def _alternating(gs, p):
    s = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
         if s is not None and s.direct_lds and s.stages == 2 and s.tile[2][1] == 32 and (s.tile[0][0], s.tile[1][0]) == (256, 256)]
    assert len(s) == 1
    return s[0]


def _ints(g, *shape):
    import torch
    return torch.randint(-1, 2, shape, generator=g, device="cuda", dtype=torch.int8).float()


# (M, N): fewer columns than a tile and one short of it; two and three ragged column tiles, rows of tiles that are not full; an even
# N whose 16-bit stores are paired and an odd one (column-major B only), whose are not; more tiles than one round of 256 holds
@pytest.mark.parametrize("ta,tb", [(0, 1), (0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("dtype,out", [("f16", "f32"), ("bf16", "f32"), ("f16", "f16"), ("bf16", "bf16")])
def test_every_element(gs, dtype, out, ta, tb):
    import torch
    if ta and out != "f32":
        pytest.skip("not compiled")
    g = torch.Generator(device="cuda").manual_seed(15)
    shapes = [(264, 8, 64), (264, 184, 72), (520, 200, 128), (248, 384, 136), (264, 568, 192), (512, 440, 264), (264, 192, 320), (264, 576, 456), (256 * 32, 192 * 9, 64)]
    if tb and not ta:
        shapes += [(259, 191, 200), (259, 385, 256)]
    for M, N, K in shapes:
        p = gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out)
        s = _alternating(gs, p)
        A, B = _ints(g, *((K, M) if ta else (M, K))), _ints(g, *((N, K) if tb else (K, N)))
        want = ((A.T.contiguous() if ta else A) @ (B.T.contiguous() if tb else B)).to(getattr(torch, {"f32": "float32", "f16": "float16", "bf16": "bfloat16"}[out]))
        C = gs.empty_device((M + 1, N), out).fill_(float("nan"))
        print("instance", s.kernel_id, dtype, out, (M, N, K), "transA", ta, "transB", tb, flush=True)
        gs.gemm(p, _in_infinities(gs, A, dtype), _in_infinities(gs, B, dtype), C[:M], 1.0, 0.0, s)
        assert torch.equal(C[:M], want) and bool(torch.isnan(C[M]).all()), (s.kernel_id, M, N, K)


def test_products_on_either_side_of_the_rule(gs):
    """16 x 16 wide tiles are one round and 16 x 22 narrow ones two; 16 x 12 and 16 x 16 are one each.  (Which width a launch takes is
    checked in test_host_dispatch.py, on the host code.)"""
    import torch
    g = torch.Generator(device="cuda").manual_seed(16)
    for N in (4096, 3072):
        M, K = 4096, 136
        p = gs.gemm_problem("f16", M, N, K, 0, 1)
        A, B = _ints(g, M, K), _ints(g, N, K)
        C = gs.empty_device((M, N))
        print("columns", N, flush=True)
        gs.gemm(p, A.half(), B.half(), C, 1.0, 0.0, _alternating(gs, p))
        assert torch.equal(C, A @ B.T.contiguous()), N


@pytest.mark.parametrize("out", ["f32", "f16"])
def test_alpha_beta_and_batches(gs, out):
    import torch
    g = torch.Generator(device="cuda").manual_seed(17)
    batch, M, N, K = 3, 300, 376, 152
    A, B = _ints(g, batch, M, K).half(), _ints(g, batch, K, N).half()
    p = gs.gemm_problem("f16", M, N, K, 0, 0, batch, out)
    C0 = _ints(g, batch, M, N).to(torch.float32 if out == "f32" else torch.float16)
    for alpha, beta in ((0.5, 2.0), (2.0, 0.0)):
        C = C0.clone()
        gs.bmm(p, A, B, C, alpha, beta, _alternating(gs, p))
        for b in range(batch):
            want = alpha * (A[b].float() @ B[b].float().contiguous()) + beta * C0[b].float()
            assert torch.equal(C[b].float(), want), (alpha, beta, b)
