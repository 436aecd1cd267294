"""What the entry points dispatch a call to, and what they refuse, on the library's host code alone (tests/stub_library.py)."""
import pytest

from stub_library import ACCEPTED, Stub


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    return Stub(tmp_path_factory.mktemp("stub"))


# (dtype, out, M, N, K, transA, transB, lda, ldb, ldc): rows too far apart for the 32-bit offsets of the 256-row tiles that are
# constructed for these shapes, and within those of 128 rows
LONG_ROWS = [
    ("f16", "f32", 3287, 2816, 704, 0, 1, 6000000, None, None),
    ("f16", "f32", 3287, 2816, 704, 0, 1, None, None, 3000000),
    ("f16", "f32", 3156, 3072, 768, 0, 1, None, 6000000, None),
    ("bf16", "bf16", 8192, 3072, 768, 0, 1, None, 6000000, None),
    ("bf16", "bf16", 8192, 3072, 768, 0, 0, None, None, 6000000),
    ("f16", "f32", 4096, 4096, 4096, 0, 0, 6000000, None, None),
    ("f16", "f32", 768, 3072, 8192, 1, 0, None, None, 3000000),
]


@pytest.mark.parametrize("case", LONG_ROWS)
def test_rows_too_long_for_the_constructed_tile_find_another(stub, case):
    dtype, out, M, N, K, ta, tb, lda, ldb, ldc = case
    p = stub.gs.gemm_problem(dtype, M, N, K, ta, tb, 1, out)
    s = stub.construct(p)
    es, os_ = 2, 4 if out == "f32" else 2
    need = stub.workspace_bytes(p, s)
    for schedule, room in ((s, need), (None, 0), (None, 1 << 30)):
        st, launch = stub.call(p, schedule, lda, ldb, ldc, room)
        assert st == ACCEPTED and launch, (case, schedule is not None, st)
        t = stub.gs.instance_schedule(launch["id"], p)
        assert t.vec_bytes == 16                                       # aligned operands keep aligned accesses
        bm, bn, bk = t.tile[0][0], t.tile[1][0], t.tile[2][0]
        a = (bk + 1) * (lda or M) + bm if ta else (bm + 1) * (lda or K)
        b = (bn + 1) * (ldb or K) if tb else (bk + 1) * (ldb or N) + bn
        assert max(a * es, b * es, (bm + 1) * (ldc or N) * os_) < 2 ** 31 - 1, (bm, bn, bk)


def test_one_construction_serves_all_rows_of_the_same_reach(stub):
    """Leading dimensions that differ from call to call: only the first pays for a construction (about 30 ms)."""
    import time
    p = stub.gs.gemm_problem("f16", 3287, 2816, 712, 0, 1)
    first = time.perf_counter()
    assert stub.call(p, None, lda=6000000)[0] == ACCEPTED
    second = time.perf_counter()
    for lda in range(6000008, 6000008 + 20 * 1000, 1000):
        assert stub.call(p, None, lda=lda)[0] == ACCEPTED
    assert time.perf_counter() - second < 0.5 * (second - first)


def test_rows_too_long_for_every_tile_stay_refused(stub):
    p = stub.gs.gemm_problem("f16", 3287, 2816, 704, 0, 1)
    for lda in (200000000, 2 ** 31, 2 ** 40):                          # (17 rows of 200 million 16-bit elements: beyond 2^31 bytes)
        for s in (stub.construct(p), None):
            st, launch = stub.call(p, s, lda=lda, room=1 << 30)
            assert st == 2 and launch is None, (lda, st)
    # a split schedule without its workspace is refused for that first, whatever the rows
    q = stub.gs.gemm_problem("f16", 512, 512, 32768, 0, 1)
    s = stub.construct(q)
    assert s.split_k > 1
    assert stub.call(q, s, lda=60000000)[0] == 4


# weight gradients (transA) whose constructed split fitted the static scratch while 256-row tiles were no choice, at least twice
# the bytes of it when they are
@pytest.mark.parametrize("M,N,K", [(768, 3072, 8192), (768, 3072, 5616), (3328, 832, 4568), (3840, 960, 3784), (3584, 896, 4504), (2520, 544, 10488)])
def test_constructed_splits_stay_within_the_static_scratch(stub, M, N, K):
    from paper_2502_11407_amd.binding import STATIC_SCRATCH_BYTES
    p = stub.gs.gemm_problem("f16", M, N, K, 1, 0)
    s = stub.construct(p)
    assert stub.workspace_bytes(p, s) <= STATIC_SCRATCH_BYTES and (s.split_k > 1 or M > 3500)      # (3840 and 3584 rows: unsplit is faster)
    assert stub.call(p, s, static=True)[0] == ACCEPTED
    assert stub.call(p, s, room=STATIC_SCRATCH_BYTES)[0] == ACCEPTED
    # and a call that names none runs the same in a workspace of that size
    st, launch = stub.call(p, None, room=STATIC_SCRATCH_BYTES)
    assert st == ACCEPTED and (launch["id"], launch["split"]) == (s.kernel_id, s.split_k)


def test_splits_beyond_the_static_scratch_where_no_other_fits_either(stub):
    """960 x 3840 x 7992 transA: every tile's best split needs more than the static scratch, so the alternating ones may, too."""
    from paper_2502_11407_amd.binding import STATIC_SCRATCH_BYTES
    p = stub.gs.gemm_problem("f16", 960, 3840, 7992, 1, 0)
    s = stub.construct(p)
    assert s.split_k > 1 and stub.workspace_bytes(p, s) > STATIC_SCRATCH_BYTES
    assert stub.call(p, s, static=True) == (4, None)


@pytest.mark.parametrize("M,N", [(960, 3840), (896, 3584), (4096, 768)])
@pytest.mark.parametrize("K", [6912, 6944, 6952, 6976, 6984, 7008, 7040])
def test_static_scratch_at_neighbouring_depths(stub, M, N, K):
    """Multiples of 64: what is constructed fits the static scratch.  Other depths: it may be the alternating tile that does not, which is then
    priced below what fits; a call that names no schedule runs within the scratch either way."""
    from paper_2502_11407_amd.binding import STATIC_SCRATCH_BYTES
    p = stub.gs.gemm_problem("f16", M, N, K, 1, 0)
    s = stub.construct(p)
    st, launch = stub.call(p, None, room=STATIC_SCRATCH_BYTES)
    t = stub.gs.instance_schedule(launch["id"], p)
    t.split_k = launch["split"]
    assert st == ACCEPTED and stub.workspace_bytes(p, t) <= STATIC_SCRATCH_BYTES
    if K % 64 == 0:
        assert (t.kernel_id, t.split_k) == (s.kernel_id, s.split_k)
    elif stub.workspace_bytes(p, s) > STATIC_SCRATCH_BYTES:
        assert s.kernel_id == _alternating(stub, p).kernel_id and s.predicted_us < stub.gs.predict_us(t, p)
    else:
        assert (t.kernel_id, t.split_k) == (s.kernel_id, s.split_k)


@pytest.mark.parametrize("dtype,M,N,K,ta,tb", [("f16", 768, 3072, 8192, 1, 0), ("bf16", 1024, 1024, 8192, 0, 1), ("f16", 512, 512, 32768, 0, 1),
                                               ("f16", 1096, 1568, 11552, 0, 0), ("f16", 2304, 576, 7944, 1, 0)])
def test_unnamed_schedules_split_as_far_as_the_workspace_goes(stub, dtype, M, N, K, ta, tb):
    """A workspace too small for the constructed split gets the cheapest one that fits it, not an unsplit schedule."""
    p = stub.gs.gemm_problem(dtype, M, N, K, ta, tb)
    s = stub.construct(p)
    full, seen = stub.workspace_bytes(p, s), []
    assert s.split_k > 1
    for room in (1 << 30, full, full - 1, full // 2, full // 4, full // 8, 1 << 19, 256, 0):
        st, launch = stub.call(p, None, room=room)
        assert st == ACCEPTED
        t = stub.gs.instance_schedule(launch["id"], p)
        t.split_k = launch["split"]
        assert stub.workspace_bytes(p, t) <= room
        if room >= full:
            assert (launch["id"], launch["split"]) == (s.kernel_id, s.split_k)
        seen.append((stub.gs.predict_us(t, p), launch["split"]))
    assert [us for us, _ in seen] == sorted(us for us, _ in seen)          # less room is never priced faster
    assert seen[-1][1] == 1 and any(split > 1 for _, split in seen[2:6])
    # the unsplit one is what a ranking without splits returns
    o = stub.gs.ConstructOpts(0, 0, 0, 0, 0, 0, 1, 0)
    assert seen[-1][0] == stub.gs.construct(p, opts=o).predicted_us


def _alternating(stub, p):
    s = [s for s in (stub.gs.instance_schedule(i, p) for i in range(stub.gs.num_instances()))
         if s is not None and s.direct_lds and s.stages == 2 and (s.tile[0][0], s.tile[1][0], s.tile[2][0], s.tile[2][1]) == (256, 256, 64, 32)]
    assert len(s) == 1
    return s[0]


# (M, N, batch, units of a round (0: the 256 of the chip), columns): both sides of the line, rounds wide / narrow counted by hand
@pytest.mark.parametrize("M,N,batch,units,columns", [
    (8192, 3072, 1, 0, 192),       # 32 x 12 = 384 / 32 x 16 = 512 tiles: 2 / 2
    (8192, 4096, 1, 0, 256),       # 512 / 704: 2 / 3
    (4096, 4096, 1, 0, 256),       # 256 / 352: 1 / 2
    (4096, 3072, 1, 0, 192),       # 192 / 256: 1 / 1, full
    (4097, 3072, 1, 0, 256),       # 204 / 272: 1 / 2
    (264, 8, 1, 0, 192), (264, 192, 1, 1, 192), (264, 192, 1, 2, 192),         # one column of either
    (256 * 128, 193, 1, 0, 192),   # 128 / 256: 1 / 1
    (256 * 128 + 1, 193, 1, 0, 256),
    (300, 712, 3, 18, 256),        # 18 / 24
    (300, 712, 3, 23, 256), (300, 712, 3, 24, 192), (300, 712, 3, 12, 192),        # 1 / 2, 1 / 1, 2 / 2
])
def test_width_of_alternating_tiles(stub, M, N, batch, units, columns):
    p = stub.gs.gemm_problem("f16", M, N, 136, 0, 1, batch)
    s = _alternating(stub, p)
    s.round_units = units
    st, launch = stub.call(p, s)
    rows, cols = -(-M // 256), -(-N // columns)
    assert st == ACCEPTED and launch["narrow"] == (columns == 192)
    assert (launch["tiles_m"], launch["tiles_n"], launch["whole"], launch["split"]) == (rows, cols, rows * cols * batch, 1)
    # parts of split tiles are always 256 columns wide
    s.split_k, s.round_units = 2, 4096
    need = stub.workspace_bytes(p, s)
    assert need == rows * -(-N // 256) * batch * 2 * 256 * 256 * 4
    st, launch = stub.call(p, s, room=need)
    assert st == ACCEPTED and launch["split_launch"] and not launch["narrow"] and launch["tiles_n"] == -(-N // 256)


@pytest.mark.parametrize("dtype,out,batch,M,N,K,stages", [
    ("f16", "f32", 96, 1000, 1000, 64, 2),         # the next batch is read ahead, rows of C are not whole lines
    ("bf16", "f32", 72, 1024, 1024, 64, 2),        # ... and where they are
    ("f16", "f32", 60, 1000, 1000, 64, 1),         # 240 MB, not read ahead
    ("f16", "f32", 1, 8192, 8200, 64, 2),          # 269 MB
    ("f16", "f32", 48, 1024, 1024, 64, 1), ("f16", "f32", 1, 8192, 8192, 64, 2),         # 201 MB, 268 MB written through
    ("bf16", "bf16", 200, 1000, 1000, 64, 1),      # 16-bit outputs are not read ahead for: 400 MB written back
    ("f16", "f16", 30, 1024, 1024, 64, 1), ("f16", "f16", 40, 1024, 1024, 64, 2),        # 63 MB, 84 MB written through
])
def test_stages_allocated_for_products_of_one_k_tile(stub, dtype, out, batch, M, N, K, stages):
    """Of the two stages of a directly staged tile a product of one k tile touches one; large outputs keep both allocated."""
    p = stub.gs.gemm_problem(dtype, M, N, K, 0, 1, batch, out)
    tile = [s for s in (stub.gs.instance_schedule(i, p) for i in range(stub.gs.num_instances())) if s is not None and s.direct_lds and s.stages == 2
            and (s.tile[0][0], s.tile[1][0], s.tile[2][0], s.tile[0][1], s.tile[1][1]) == (128, 128, 64, 64, 32)]
    st, launch = stub.call(p, tile[0])
    assert st == ACCEPTED and launch["lds_stages"] == stages
