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


def _run(gs, p, s, A, B, M, N):
    C = torch.full((M, N), float("nan"), device="cuda")
    s.split_k = 1
    gs.gemm(p, A, B, C, 1.0, 0.0, s)
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
