"""The 256x256 tiles whose two wave groups alternate (16x16 blocks, staged directly): every operand layout and output type at the
depths where prologue, steady state and drain of their slots differ, whole and split along k, at any K (the last k tile may be
partial), with ragged last rows and columns and infinities around the operands.  Small integers: every result is exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


def _in_infinities(gs, x, dtype):
    """x inside a buffer of infinities, 16 bytes before it and behind every row, rows still whole vectors."""
    import torch
    r, c = x.shape
    ld = (c + 7) // 8 * 8 + 8
    buf = gs.empty_device((8 + r * ld,), dtype).fill_(float("inf"))
    return torch.as_strided(buf, (r, c), (ld, 1), 8).copy_(x)


@pytest.mark.parametrize("ta,tb", [(0, 1), (0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("dtype,out", [("f16", "f32"), ("bf16", "f32"), ("f16", "f16"), ("bf16", "bf16")])
def test_k_depths_tails_and_splits(gs, dtype, out, ta, tb):
    import torch
    if ta and out != "f32":
        pytest.skip("not compiled")
    M, N = (264 if ta else 259), (520 if not tb else 517)
    g = torch.Generator(device="cuda").manual_seed(5)
    ran = 0
    for K, splits in ((8, (1,)), (56, (1,)), (64, (1,)), (72, (1, 2)), (128, (1, 2)), (136, (1, 3)), (192, (1,)), (200, (2, 4)), (256, (1,)),
                      (264, (1, 2)), (320, (1, 5)), (456, (1, 3))):
        p = gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out)
        scheds = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
                  if s is not None and s.direct_lds and s.stages == 2 and s.tile[2][1] == 32 and (s.tile[0][0], s.tile[1][0]) == (256, 256)]
        assert len(scheds) == 1
        A, B = (torch.randint(-1, 2, shape, generator=g, device="cuda", dtype=torch.int8).float()
                for shape in ((K, M) if ta else (M, K), (N, K) if tb else (K, N)))
        want = ((A.T.contiguous() if ta else A) @ (B.T.contiguous() if tb else B)).to(getattr(torch, {"f32": "float32", "f16": "float16", "bf16": "bfloat16"}[out]))
        for split in splits:
            s = gs.Schedule.from_buffer_copy(scheds[0])
            s.split_k = split
            C = gs.empty_device((M, N), out).fill_(float("nan"))
            ws = gs.gemm_workspace(p, s)
            if ws is not None:
                ws.fill_(0xAB)
            print("instance", s.kernel_id, dtype, out, (M, N, K), "transA", ta, "transB", tb, "split", split, flush=True)
            gs.gemm(p, _in_infinities(gs, A, dtype), _in_infinities(gs, B, dtype), C, 1.0, 0.0, s, workspace=ws)
            assert torch.equal(C, want), (s.kernel_id, K, split)
            ran += 1
    assert ran == 19


def test_alpha_beta_and_batches(gs):
    import torch
    g = torch.Generator(device="cuda").manual_seed(6)
    batch, M, N, K = 3, 300, 264, 152
    A = torch.randint(-2, 3, (batch, M, K), generator=g, device="cuda", dtype=torch.int8).half()
    B = torch.randint(-2, 3, (batch, K, N), generator=g, device="cuda", dtype=torch.int8).half()
    p = gs.gemm_problem("f16", M, N, K, 0, 0, batch)
    s = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
         if s is not None and s.direct_lds and s.stages == 2 and s.tile[2][1] == 32 and (s.tile[0][0], s.tile[1][0]) == (256, 256)][0]
    C0 = torch.randint(-4, 5, (batch, M, N), generator=g, device="cuda", dtype=torch.int8).float()
    C = C0.clone()
    gs.bmm(p, A, B, C, 0.5, 2.0, s)
    for b in range(batch):
        assert torch.equal(C[b], 0.5 * (A[b].float() @ B[b].float()) + 2.0 * C0[b]), b


@pytest.mark.parametrize("operand", ["A", "B", "C"])
def test_rows_too_long_for_256_row_tiles(gs, operand):
    """Leading dimensions that the offsets of a 256-row tile do not reach and those of a 128-row one do, in the schedule of an
    instance of 256 rows and with none named: a tile that reaches takes the call."""
    import torch
    g = torch.Generator(device="cuda").manual_seed(7)
    M, N, K, far = 300, 280, 72, {"A": 6000000, "B": 6000000, "C": 3000000}[operand]

    def rows(r, c, ld, dtype):
        return torch.as_strided(gs.empty_device(((r - 1) * ld + c,), dtype), (r, c), (ld, 1))

    ints = lambda r, c: torch.randint(-1, 2, (r, c), generator=g, device="cuda", dtype=torch.int8)
    A = rows(M, K, far if operand == "A" else K, "f16").copy_(ints(M, K))
    B = rows(N, K, far if operand == "B" else K, "f16").copy_(ints(N, K))
    C = rows(M, N + 8, far if operand == "C" else N + 8, "f32")
    p = gs.gemm_problem("f16", M, N, K, 0, 1)
    wide = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
            if s is not None and s.direct_lds and s.stages == 2 and s.tile[2][1] == 32 and (s.tile[0][0], s.tile[1][0]) == (256, 256)]
    assert len(wide) == 1
    for s in (wide[0], None):
        C.fill_(7.0)
        gs.gemm(p, A, B, C, 1.0, 0.0, s)
        assert torch.equal(C[:, :N], A.float() @ B.float().T.contiguous()) and bool((C[:, N:] == 7.0).all())
