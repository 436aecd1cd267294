"""Tiles that keep several sums per output (the kernels' CHAINS): which products share a sum, and the distance from 64 bits that this buys."""
import pytest
import torch

pytestmark = pytest.mark.gpu

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}


def _small_tiles(gs, p):
    """The 32x32 tiles of 256-byte k tiles: eight sums, told apart by the k step and the parity of the k tile."""
    deep = 64 if p.in_dtype == gs.DTYPE["f32"] else 128
    found = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
             if s is not None and (s.tile[0][0], s.tile[1][0], s.tile[2][0]) == (32, 32, deep) and s.tile[0][1] == 16]
    assert found
    return found


def _run(gs, p, s, A, B, M, N, split=1):
    C = torch.full((M, N), float("nan"), device="cuda")
    s.split_k = split
    gs.gemm(p, A, B, C, 1.0, 0.0, s, workspace=gs.gemm_workspace(p, s))
    torch.cuda.synchronize()
    return C


@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("tiles", [4, 6, 8, 10])
def test_last_tile_of_an_even_count_is_added_to_the_odd_tiles_sums(dtype, tiles, tb):
    """2^24 in the last even k tile, -2^24 in the first odd one and 1 in the last: with the odd tile's sum the 1 survives, with the even one's
    2^24 + 1 is rounded to 2^24."""
    from paper_2502_11407_amd import binding as gs
    M = N = 64
    K = 128 * tiles
    p = gs.gemm_problem(dtype, M, N, K, 0, tb)
    for step in range(4):
        A, B = torch.zeros(M, K), torch.zeros(K, N)
        for tile, a, b in ((tiles - 2, 4096.0, 4096.0), (1, 4096.0, -4096.0), (tiles - 1, 1.0, 1.0)):
            k = tile * 128 + step * 32 + 5
            A[:, k], B[k, :] = a, b
        a = A.to(TORCH[dtype]).cuda()
        b = (B.t().contiguous() if tb else B).to(TORCH[dtype]).cuda()
        for s in _small_tiles(gs, p):
            print(dtype, tiles, tb, step, "instance", s.kernel_id, flush=True)
            assert (_run(gs, p, s, a, b, M, N) == 1.0).all(), (s.kernel_id, step)


def _operands(dtype, M, N, K, ta, tb, terms):
    """A and B of which only the products a * b at the given k are not zero."""
    A, B = torch.zeros(M, K), torch.zeros(K, N)
    for k, a, b in terms:
        A[:, k], B[k, :] = a, b
    return tuple(x.to(TORCH[dtype]).cuda() for x in (A.t().contiguous() if ta else A, B.t().contiguous() if tb else B))


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_deep_rings_of_16x16_blocks_keep_several_sums(dtype, ta, tb):
    """2^24, then 1, then -2^24: the 1 survives where it is added to another sum.  Sums are told apart by the k step; in 128x128 tiles by the
    parity of the k tile, too."""
    from paper_2502_11407_amd import binding as gs
    p = gs.gemm_problem(dtype, 64, 64, 64, ta, tb)
    rings = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
             if s is not None and s.direct_lds and s.stages > 2 and s.tile[2][1] == 32]
    assert len(rings) == (2 if ta or not tb else 3)
    for s in rings:
        M, N = s.tile[0][0] + 8, s.tile[1][0] + 16
        for K, split in ((64 * 24, 1), (64 * 24 + 8, 1), (64 * 26 + 56, 1), (64 * 48, 2)):
            q = gs.gemm_problem(dtype, M, N, K, ta, tb)
            middles = [64 + 32 + 7] + ([64 + 7, 3 * 64 + 7] if s.stages == 4 else [])
            for k in middles:
                print(dtype, ta, tb, "instance", s.kernel_id, "K", K, "split", split, "k", k, flush=True)
                a, b = _operands(dtype, M, N, K, ta, tb, ((5, 4096.0, 4096.0), (k, 1.0, 1.0), (4 * 64 + 9, 4096.0, -4096.0)))
                assert (_run(gs, q, s, a, b, M, N, split) == 1.0).all(), (s.kernel_id, K, split, k)


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_deep_any_alignment_tiles_keep_four_sums(dtype, ta, tb):
    from paper_2502_11407_amd import binding as gs
    p = gs.gemm_problem(dtype, 63, 63, 63, ta, tb)
    tiles = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
             if s is not None and s.vec_bytes != 16 and (s.tile[0][0], s.tile[1][0], s.tile[2][0], s.tile[2][1]) == (64, 64, 64, 16)]
    assert tiles
    M, N = 67, 65
    for s in tiles:
        for K, split in ((64 * 15 + 1, 1), (64 * 16 + 63, 1), (64 * 13 + 5, 2), (64 * 14 + 1, 2)):
            q = gs.gemm_problem(dtype, M, N, K, ta, tb)
            for step in (1, 2, 3):
                print(dtype, ta, tb, "instance", s.kernel_id, "K", K, "split", split, "step", step, flush=True)
                a, b = _operands(dtype, M, N, K, ta, tb, ((5, 4096.0, 4096.0), (16 * step + 7, 1.0, 1.0), (4 * 64 + 9, 4096.0, -4096.0)))
                assert (_run(gs, q, s, a, b, M, N, split) == 1.0).all(), (s.kernel_id, K, split, step)


@pytest.mark.parametrize("ta,tb", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("dtype,bm,sums", [("f16", 128, 2), ("bf16", 128, 2), ("f32", 64, 8)])
def test_any_alignment_tiles_that_stood_for_parts_or_for_smaller_tiles_keep_several_sums(dtype, bm, sums, ta, tb):
    """128x64 tiles of 24 k tiles and more: two sums; fp32 64x64 tiles of a shallow k, one to two a compute unit: eight."""
    from paper_2502_11407_amd import binding as gs
    fp32 = dtype == "f32"
    step, bk = (8, 32) if fp32 else (16, 64)
    p = gs.gemm_problem(dtype, 63, 63, 63, ta, tb)
    tiles = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances()))
             if s is not None and s.vec_bytes != 16 and (s.tile[0][0], s.tile[1][0], s.tile[2][0], s.tile[2][1]) == (bm, 64, bk, step)]
    assert tiles
    M, N = (64 * 16 + 1, 64 * 16 - 1) if fp32 else (bm + 3, 67)
    for s in tiles:
        for K in (bk * 5 - 3, bk * 6) if fp32 else (bk * 23 + 1, bk * 25 - 1):
            q = gs.gemm_problem(dtype, M, N, K, ta, tb)
            for k in [step * i + 3 for i in range(1, sums // 2 if fp32 else sums)] + ([bk + 3, bk + 3 * step + 3] if fp32 else []):
                print(dtype, ta, tb, "instance", s.kernel_id, "K", K, "k", k, flush=True)
                a, b = _operands(dtype, M, N, K, ta, tb, ((1, 4096.0, 4096.0), (k, 1.0, 1.0), (2 * bk + 2, 4096.0, -4096.0)))
                assert (_run(gs, q, s, a, b, M, N) == 1.0).all(), (s.kernel_id, K, k)


def _distance(C, A, B):
    want = A.double() @ B.double()
    return ((C.double() - want).norm() / want.norm()).item()


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_several_sums_lose_less_than_one(dtype):
    """Distance from 64 bits at even and odd counts of k tiles, beside a 64x64 tile of a single sum on the same operands.  Rounding a running sum of n
    terms loses about sqrt(n / 2) roundings, so s sums that are then added up lose 1 / sqrt(s) of that, and the last rounding on top:
    bounds of 0.75 (eight sums, measured 0.37-0.68), 0.65 (four) and 0.8 (two: 0.67-0.73)."""
    from paper_2502_11407_amd import binding as gs
    M = N = 384
    fp32 = dtype == "f32"
    for K, tile, bound in ([(64 * n, (32, 32), 0.75) for n in (2, 3, 5, 8)] if fp32 else
                           [(128 * n, (32, 32), 0.75) for n in (2, 3, 4, 5, 8)] + [(64 * n, (128, 128), 0.65) for n in (24, 25, 40)] +
                           [(64 * n, (256, 128), 0.8) for n in (24, 25, 40)]):
        gen = torch.Generator(device="cuda").manual_seed(K)
        A, B = (torch.empty(s, device="cuda").uniform_(-1, 1, generator=gen).to(TORCH[dtype]) for s in ((M, K), (K, N)))
        b = B.t().contiguous()
        p = gs.gemm_problem(dtype, M, N, K, 0, 1)
        every = [s for s in (gs.instance_schedule(i, p) for i in range(gs.num_instances())) if s is not None and s.vec_bytes == 16]
        one = next(s for s in every if (s.tile[0][0], s.tile[1][0]) == (64, 64) and s.stages == 2)
        if tile == (32, 32):
            several = [s for s in every if (s.tile[0][0], s.tile[1][0]) == tile and s.tile[2][0] == (64 if fp32 else 128) and s.tile[0][1] == 16]
        else:
            several = [s for s in every if (s.tile[0][0], s.tile[1][0]) == tile and s.direct_lds and s.stages > 2 and s.tile[2][1] == 32]
        alone = _distance(_run(gs, p, one, A, b, M, N), A, B)
        assert several
        for s in several:
            d = _distance(_run(gs, p, s, A, b, M, N), A, B)
            print(dtype, K, "instance", s.kernel_id, "distance %.2e, one sum %.2e: %.2f" % (d, alone, d / alone), flush=True)
            assert d <= bound * alone, (s.kernel_id, K)
