"""Workgroups are renumbered so that each of the 8 XCDs holds a contiguous range of tiles, whatever their number: every tile of a
launch is computed exactly once at counts around multiples of 8, whole and split along k.  Small integers, exact."""
import pytest

pytestmark = pytest.mark.gpu


def _ints(shape, seed):
    import torch
    g = torch.Generator(device="cuda").manual_seed(seed)
    return torch.randint(-2, 3, shape, generator=g, device="cuda", dtype=torch.int8).half()


@pytest.mark.parametrize("count", [1, 2, 7, 8, 9, 15, 17, 31, 63, 65, 259])
def test_batches_of_one_tile(count):
    import torch
    from paper_2502_11407_amd import binding as gs
    A, B = _ints((count, 64, 64), count), _ints((count, 64, 64), count + 1)
    p = gs.gemm_problem("f16", 64, 64, 64, 0, 0, 1)
    p.op, p.batch = gs.OP_BMM, count
    for idx in range(gs.num_instances()):
        s = gs.instance_schedule(idx, p)
        if s is None or (s.tile[0][0], s.tile[1][0]) != (64, 64):
            continue
        C = torch.full((count, 64, 64), float("nan"), device="cuda")
        gs.bmm(p, A, B, C, schedule=s)
        assert torch.equal(C, torch.stack([A[b].float() @ B[b].float() for b in range(count)])), (idx, count)


@pytest.mark.parametrize("tiles,parts", [(1, 2), (3, 3), (5, 2), (7, 7), (9, 5), (13, 16)])
def test_split_tiles(tiles, parts):
    import torch
    from paper_2502_11407_amd import binding as gs
    N, K = 64 * tiles, 64 * parts + 64
    A, B = _ints((64, K), tiles), _ints((K, N), parts)
    p = gs.gemm_problem("f16", 64, N, K, 0, 0)
    ran = 0
    for idx in range(gs.num_instances()):
        s = gs.instance_schedule(idx, p)
        if s is None or (s.tile[0][0], s.tile[1][0]) != (64, 64):
            continue
        s.split_k = parts
        ws = gs.gemm_workspace(p, s)
        if ws is None:
            continue
        ws.fill_(0xAB)
        C = torch.full((64, N), float("nan"), device="cuda")
        gs.gemm(p, A, B, C, schedule=s, workspace=ws)
        assert torch.equal(C, A.float() @ B.float()), (idx, tiles, parts)
        ran += 1
    assert ran
