"""Rings of 16x16 blocks at a K that is no multiple of their k tile, from a part of one k tile to more tiles than stages, whole and
split along k: bit-exact on integers, with infinities behind every row and around the operands."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gs():
    from paper_2502_11407_amd import binding
    return binding


def _embedded(gs, rows, cols, dtype, seed):
    """Integers in rows 24 elements longer than they need to be, in a buffer of infinities."""
    import torch
    gen = torch.Generator(device="cuda").manual_seed(seed)
    buf = gs.empty_device((64 + rows * (cols + 24) + 64,), dtype).fill_(float("inf"))
    x = torch.as_strided(buf, (rows, cols), (cols + 24, 1), 64)
    return x.copy_(torch.randint(-2, 3, (rows, cols), generator=gen, device="cuda", dtype=torch.int8))


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype,out", [("f16", "f32"), ("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16")])
def test_rings_of_16x16_blocks_at_any_k(gs, dtype, out, ta, tb):
    import torch
    p = gs.gemm_problem(dtype, 64, 64, 64, ta, tb, 1, out)
    rings = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
             if s is not None and s.direct_lds and s.stages > 2 and s.tile[2][1] == 32]
    assert len(rings) == (0 if ta and out != "f32" else 2 if ta or not tb else 3)
    for s in rings:
        bm, bn, bk = s.tile[0][0], s.tile[1][0], s.tile[2][0]
        M, N = bm + 40, bn + 24
        for K, splits in ((8, (1,)), (56, (1,)), (72, (1, 2)), (120, (1, 2)), (184, (1, 3)), (200, (1, 2)), (328, (1, 3)), (456, (1, 4))):
            A, B = _embedded(gs, *((K, M) if ta else (M, K)), dtype, K), _embedded(gs, *((N, K) if tb else (K, N)), dtype, K + 1)
            want = (A.T if ta else A).float().contiguous() @ (B.T if tb else B).float().contiguous()
            q = gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out)
            for split in splits:
                t = gs.Schedule.from_buffer_copy(s)
                t.split_k = split
                print("instance", s.kernel_id, (bm, bn, bk), dtype, out, "transA", ta, "transB", tb, "K", K, "split", split, flush=True)
                C = gs.empty_device((M, N), out).fill_(float("nan"))
                ws = gs.gemm_workspace(q, t)
                assert (ws is not None) == (split > 1)
                gs.gemm(q, A, B, C, 1.0, 0.0, t, workspace=ws)
                torch.cuda.synchronize()
                assert torch.equal(C, want.to(C.dtype)), (s.kernel_id, K, split)
                # ... and beside beta, which takes the element stores
                gs.gemm(q, A, B, C, 2.0, 1.0, t, workspace=ws)
                torch.cuda.synchronize()
                assert torch.equal(C, (2.0 * want + want.to(C.dtype).float()).to(C.dtype)), (s.kernel_id, K, split)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_rings_of_16x16_blocks_at_odd_k(gs, dtype):
    """An m-contiguous A beside a row-major B leaves K free of the vector width: below, at and beyond one k tile, whole and in parts."""
    import torch
    p = gs.gemm_problem(dtype, 64, 64, 64, 1, 0)
    rings = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
             if s is not None and s.direct_lds and s.stages > 2 and s.tile[2][1] == 32]
    assert len(rings) == 2
    for s in rings:
        M, N = s.tile[0][0] + 40, s.tile[1][0] + 24
        for K, splits in ((1, (1,)), (7, (1,)), (33, (1,)), (63, (1,)), (65, (1, 2)), (127, (1, 2)), (193, (1, 2, 3)), (257, (1, 4)), (451, (1, 3)), (1601, (1, 2))):
            A, B = _embedded(gs, K, M, dtype, K), _embedded(gs, K, N, dtype, K + 1)
            want = A.T.float().contiguous() @ B.float().contiguous()
            q = gs.gemm_problem(dtype, M, N, K, 1, 0)
            for split in splits:
                t = gs.Schedule.from_buffer_copy(s)
                t.split_k = split
                print("instance", s.kernel_id, dtype, "K", K, "split", split, flush=True)
                C = gs.empty_device((M, N)).fill_(float("nan"))
                gs.gemm(q, A, B, C, 1.0, 0.0, t, workspace=gs.gemm_workspace(q, t))
                torch.cuda.synchronize()
                assert torch.equal(C, want), (s.kernel_id, K, split)
