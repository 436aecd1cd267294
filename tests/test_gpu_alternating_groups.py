"""The 256x256 tiles whose two wave groups alternate (16x16 blocks, staged directly): every operand layout and output type at the
depths where prologue, steady state and drain of their slots differ, whole and split along k, at any K (the last k tile may be
partial), with ragged last rows and columns and infinities around the operands.  A launch that splits nothing may cut C 192 columns
wide; here the compute units of the schedule's rounds are chosen so that both widths run, and the wide ones are not left to the
defaults.  Small integers: every result is exact."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


def widths(M, N, batch=1):
    """Rounds (Schedule.round_units) in which a launch cuts these extents 256 columns wide, and 192.  The library's rule: narrow if
    that takes no more rounds; of as many units as there are wide tiles, more narrow ones are a second round."""
    tiles = lambda w: -(-M // 256) * -(-N // w) * batch
    assert tiles(192) > tiles(256), "no round tells the widths apart"
    return (256, tiles(256)), (192, tiles(192))


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
    M, N = (264 if ta else 259), (712 if not tb else 709)              # 2 x 3 wide tiles, 2 x 4 narrow ones
    g = torch.Generator(device="cuda").manual_seed(5)
    ran = 0
    # whole: one to nine k tiles, with and without a partial last one; parts of one to five
    for K, splits in ((8, ()), (56, ()), (64, ()), (72, (2,)), (128, (2,)), (136, (3,)), (192, ()), (200, (2, 4)), (256, ()), (264, (2,)), (320, (5,)),
                      (328, ()), (384, ()), (392, (2,)), (456, (3,)), (512, ()), (520, (2,))):
        p = gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out)
        scheds = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
                  if s is not None and s.direct_lds and s.stages == 2 and s.tile[2][1] == 32 and (s.tile[0][0], s.tile[1][0]) == (256, 256)]
        assert len(scheds) == 1
        A, B = (torch.randint(-1, 2, shape, generator=g, device="cuda", dtype=torch.int8).float()
                for shape in ((K, M) if ta else (M, K), (N, K) if tb else (K, N)))
        want = ((A.T.contiguous() if ta else A) @ (B.T.contiguous() if tb else B)).to(getattr(torch, {"f32": "float32", "f16": "float16", "bf16": "bfloat16"}[out]))
        for split, (width, units) in [(1, w) for w in widths(M, N)] + [(split, (256, 0)) for split in splits]:
            s = gs.Schedule.from_buffer_copy(scheds[0])
            s.split_k, s.round_units = split, units
            C = gs.empty_device((M, N), out).fill_(float("nan"))
            ws = gs.gemm_workspace(p, s)
            if ws is not None:
                ws.fill_(0xAB)
            print("instance", s.kernel_id, dtype, out, (M, N, K), "transA", ta, "transB", tb, "split", split, "columns", width, flush=True)
            gs.gemm(p, _in_infinities(gs, A, dtype), _in_infinities(gs, B, dtype), C, 1.0, 0.0, s, workspace=ws)
            assert torch.equal(C, want), (s.kernel_id, K, split, width)
            ran += 1
    assert ran == 2 * 17 + 10


@pytest.mark.parametrize("ta,tb", [(0, 1), (0, 0), (1, 1), (1, 0)])
@pytest.mark.parametrize("dtype,out", [("f16", "f32"), ("bf16", "f32"), ("f16", "f16"), ("bf16", "bf16")])
def test_alpha_beta_and_batches(gs, dtype, out, ta, tb):
    import torch
    if ta and out != "f32":
        pytest.skip("not compiled")
    g = torch.Generator(device="cuda").manual_seed(6)
    batch, M, N, K = 3, 304, 712, 152
    td, to = (getattr(torch, {"f32": "float32", "f16": "float16", "bf16": "bfloat16"}[x]) for x in (dtype, out))
    ints = lambda *shape: torch.randint(-1, 2, shape, generator=g, device="cuda", dtype=torch.int8)
    A = ints(batch, *((K, M) if ta else (M, K))).to(td)
    B = ints(batch, *((N, K) if tb else (K, N))).to(td)
    p = gs.gemm_problem(dtype, M, N, K, ta, tb, batch, out)
    s = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
         if s is not None and s.direct_lds and s.stages == 2 and s.tile[2][1] == 32 and (s.tile[0][0], s.tile[1][0]) == (256, 256)][0]
    C0 = ints(batch, M, N).to(to)
    for alpha, beta in ((0.5, 2.0), (1.0, 0.0), (2.0, -1.0)):
        for width, units in widths(M, N, batch):
            s.round_units = units
            C = C0.clone()
            print("instance", s.kernel_id, dtype, out, "transA", ta, "transB", tb, "alpha", alpha, "beta", beta, "columns", width, flush=True)
            gs.bmm(p, A, B, C, alpha, beta, s)
            for b in range(batch):
                a, w = (A[b].T if ta else A[b]).float().contiguous(), (B[b].T if tb else B[b]).float().contiguous()
                # (multiples of 1/2 below 2^9: exact in fp32, and rounded once to 16 bits)
                assert torch.equal(C[b], (alpha * (a @ w) + beta * C0[b].float()).to(to)), (alpha, beta, b, width)


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
