"""Every GEMM loop that looks ahead (rings, two register sets, direct staging of either operand, read-ahead of the next batch) from one
k tile up, whole and split along k, bit-exact on integers: the depths at which prologue, steady state and tail differ."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


def _ints(gs, shape, dtype, seed, lo=-1, hi=1):
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    return gs.empty_device(shape, dtype).copy_(torch.randint(lo, hi + 1, shape, generator=gen, device="cuda", dtype=torch.int8))


def _embedded(gs, x, dtype, offset, pad):
    """x inside a buffer of infinities: `offset` elements before it, rows `pad` elements longer than they need to be."""
    import torch
    r, c = x.shape
    buf = gs.empty_device((offset + (r - 1) * (c + pad) + c + 1,), dtype).fill_(float("inf"))
    return torch.as_strided(buf, (r, c), (c + pad, 1), offset).copy_(x)


def _check(gs, p, s, A, B, ta, tb, out, split):
    """One call against fp32 sums of small integers (exact), rounded once to the output type."""
    import torch
    s = gs.Schedule.from_buffer_copy(s)
    s.split_k = split
    C = gs.empty_device((p.M, p.N), out).fill_(float("nan"))
    ws = gs.gemm_workspace(p, s)
    if ws is not None:
        ws.fill_(0xAB)
    gs.gemm(p, A, B, C, 1.0, 0.0, s, workspace=ws)
    a, b = (A.T if ta else A).float(), (B.T if tb else B).float()
    want = (a.contiguous() @ b.contiguous()).to(C.dtype)
    torch.cuda.synchronize()
    assert torch.equal(C, want), "instance %d %dx%dx%d split %d" % (s.kernel_id, p.M, p.N, p.K, split)


def _instances(gs, dtype, out, ta, tb, vec):
    p = gs.gemm_problem(dtype, 64, 64, 64, ta, tb, 1, out)
    found = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances())) if s is not None]
    return [s for s in found if (s.vec_bytes == 16) == vec]


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype,out", [("f16", "f32"), ("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16"), ("f32", "f32")])
def test_aligned_instances_across_k_depths_and_splits(gs, dtype, out, ta, tb):
    ring = split_ring = register = 0
    for s in _instances(gs, dtype, out, ta, tb, True):
        bm, bn, bk = s.tile[0][0], s.tile[1][0], s.tile[2][0]
        M, N = bm + 8, bn + 16
        print("instance", s.kernel_id, dtype, out, "transA", ta, "transB", tb, (bm, bn, bk), "stages", s.stages, "direct", s.direct_lds, flush=True)
        for tiles, tail, splits in ((1, 0, (1,)), (2, 0, (1, 2)), (3, 8, (1, 2, 3)), (4, 0, (1, 2)), (7, 0, (1, 2, 3)), (7, 8, (1, 3))):
            K = tiles * bk - tail
            if s.direct_lds and tail and not (s.stages == 2 and (bm, bn, bk, s.tile[2][1]) == (256, 256, 64, 32)):
                continue                               # direct staging takes whole k tiles only (but where the wave groups alternate)
            p = gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out)
            A = _ints(gs, (K, M) if ta else (M, K), dtype, 3 * K + 1)
            B = _ints(gs, (N, K) if tb else (K, N), dtype, 3 * K + 2)
            for split in splits:
                t = gs.Schedule.from_buffer_copy(s)
                t.split_k = split
                if split > 1 and gs.workspace_bytes(p, t) == 0:
                    continue                           # not compiled with split tiles
                _check(gs, p, s, A, B, ta, tb, out, split)
                ring += s.stages > 2
                split_ring += s.stages > 2 and split > 1
                register += not s.direct_lds and s.stages == 2
    assert register
    if dtype != "f32" and not (ta and out != "f32"):
        assert ring and split_ring


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_any_alignment_instances_split_along_k(gs, dtype, ta, tb):
    """Parts that begin and end inside the operands, and a last one with a k tail, with infinities around the operands."""
    ran = 0
    for s in _instances(gs, dtype, "f32", ta, tb, False):
        bm, bn, bk = s.tile[0][0], s.tile[1][0], s.tile[2][0]
        M, N = bm + 1, bn + 3
        for K, split in ((2 * bk - 1, 2), (3 * bk + 1, 2), (5 * bk - 3, 3), (4 * bk, 4), (9 * bk + 5, 3)):
            p = gs.gemm_problem(dtype, M, N, K, ta, tb)
            t = gs.Schedule.from_buffer_copy(s)
            t.split_k = split
            if gs.workspace_bytes(p, t) == 0:
                continue
            print("instance", s.kernel_id, dtype, (M, N, K), "transA", ta, "transB", tb, "split", split, flush=True)
            A, B = _ints(gs, (K, M) if ta else (M, K), dtype, K), _ints(gs, (N, K) if tb else (K, N), dtype, K + 1)
            for offset, pad in ((0, 0), (1, 2), (3, 1)):
                _check(gs, p, s, _embedded(gs, A, dtype, offset, pad), _embedded(gs, B, dtype, offset + 1, pad), ta, tb, "f32", split)
            ran += 1
    assert ran >= 5


@pytest.mark.parametrize("ta,tb,K,shared", [
    (0, 1, 64, ""), (0, 1, 128, "A"), (0, 1, 64, "B"), (0, 0, 64, ""), (0, 0, 128, "A"), (0, 0, 64, "B"), (1, 0, 64, ""), (1, 1, 128, ""),
])
def test_batches_that_read_the_next_one_ahead(gs, ta, tb, K, shared):
    """More than 256 MiB moved by batches of one or two k tiles on the tile compiled for it; operands of a batch its own or shared."""
    import torch
    batch, M, N = 72, 1000, 1016
    shapes = {"A": (K, M) if ta else (M, K), "B": (N, K) if tb else (K, N)}
    A, B = (_ints(gs, (1,) + shapes[x], "f16", K + 3).expand(batch, *shapes[x]) if x == shared else _ints(gs, (batch,) + shapes[x], "f16", K + i, -3, 3)
            for i, x in enumerate("AB"))
    p = gs.gemm_problem("f16", M, N, K, ta, tb, batch)
    scheds = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
              if s is not None and (s.tile[0][0], s.tile[1][0]) == (128, 128) and s.tile[0][1] * s.tile[1][1] == 64 * 32 and s.direct_lds]
    assert scheds
    C = gs.empty_device((batch, M, N))
    for s in scheds:
        print("read-ahead instance", s.kernel_id, ta, tb, K, shared, flush=True)
        C.fill_(float("nan"))
        gs.bmm(p, A, B, C, 1.0, 0.0, s)
        for b in range(batch):
            a, w = (A[b].T if ta else A[b]).float().contiguous(), (B[b].T if tb else B[b]).float().contiguous()
            assert torch.equal(C[b], a @ w), b


@pytest.mark.parametrize("beta", [0.0, 1.0])
@pytest.mark.parametrize("ta,tb,K", [(0, 1, 64), (0, 0, 64), (1, 0, 64), (1, 1, 128)])
def test_batches_that_read_the_next_one_ahead_and_store_whole_lines(gs, ta, tb, K, beta):
    """The same with rows of C that are whole lines, which are stored non-temporal, or beside C as they are without the read-ahead."""
    import torch
    batch, M, N = 72, 1000, 1024
    A, B = (_ints(gs, (batch,) + x, "f16", K + i, -3, 3) for i, x in enumerate(((K, M) if ta else (M, K), (N, K) if tb else (K, N))))
    p = gs.gemm_problem("f16", M, N, K, ta, tb, batch)
    scheds = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
              if s is not None and (s.tile[0][0], s.tile[1][0]) == (128, 128) and s.tile[0][1] * s.tile[1][1] == 64 * 32 and s.direct_lds and s.stages == 2]
    assert scheds
    before = _ints(gs, (batch, M, N), "f32", 9, -5, 5)
    C = gs.empty_device((batch, M, N))
    for s in scheds:
        print("read-ahead instance", s.kernel_id, ta, tb, K, beta, flush=True)
        C.copy_(before) if beta else C.fill_(float("nan"))
        gs.bmm(p, A, B, C, 1.0, beta, s)
        for b in range(batch):
            a, w = (A[b].T if ta else A[b]).float().contiguous(), (B[b].T if tb else B[b]).float().contiguous()
            assert torch.equal(C[b], a @ w + before[b] if beta else a @ w), b
