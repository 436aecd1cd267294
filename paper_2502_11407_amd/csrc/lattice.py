"""The compiled part of the schedule lattice: which (tile, wave tile, MFMA block, virtual
thread, staging) points exist as kernel instances for each element type and operand source.
build.py turns this list into one translation unit per instance plus the registry table."""
from itertools import product

DT = {"f32": 0, "f16": 1, "bf16": 2}
BSRC = {"KC": 0, "NC": 1, "CONV": 2, "NCS2": 3}
ASRC = {"KC": 0, "MC": 1}
CT = {"f32": "f32_t", "f16": "f16_t", "bf16": "bf16_t"}


def full_v(dt, bk, bsrc, asrc="KC"):
    """Virtual threads at which the fragment reads of both operand tiles are free of bank conflicts: a
    k-contiguous tile needs as many phases as it has 16-byte chunks per row; an n-contiguous one has its
    4 (16-bit) or 2 (fp32) k rows that are read together spread by the row pad."""
    es = 4 if dt == "f32" else 2
    cpr = bk * es // 16
    strided = 2 if dt == "f32" else 4
    return (cpr if asrc == "KC" else strided), (cpr if bsrc == "KC" else strided)


def _inst(dt, out, bm, bn, bk, wm, wn, mb, vm=None, vn=None, bsrc="KC", vec=1, stages=2, direct=0, units=0, asrc="KC"):
    fm, fn = (1, 1) if units else full_v(dt, bk, bsrc, asrc)
    return dict(dt=dt, out=out, bm=bm, bn=bn, bk=bk, wm=wm, wn=wn, mb=mb, vm=vm or fm, vn=vn or fn,
                bsrc=bsrc, vec=vec, stages=stages, direct=direct, units=units, asrc=asrc)


def _convp(dt, out, bm, bn, bkc, wm, wn, units, stages=2):
    """Convolution with the input patch staged in LDS (direct = 1 on the CONV source); bk = channels per stage;
    stages = LDS buffers (1: more workgroups per CU hide the load latency, 2: the next stage is written while
    this one is multiplied)."""
    return _inst(dt, out, bm, bn, bkc, wm, wn, 32, 1, 1, "CONV", 1, stages, 1, units)


def conv_rows(d):
    """Convolution with the input rows staged in LDS as they lie, any alignment (direct = 1, vec = 0 on the CONV source)."""
    return d["bsrc"] == "CONV" and d["direct"] == 1 and d["vec"] == 0


def alternate(d):
    """Two groups of waves that take turns at reading and multiplying (the kernel's ALTERNATE)."""
    return d["direct"] == 1 and d["stages"] == 2 and d["mb"] == 16 and (d["bm"], d["bn"], d["bk"]) == (256, 256, 64)


def chains(d):
    """Sums that a lane keeps per output of a register-staged tile (the kernel's CHAINS or DEEP_CHAINS)."""
    es = 4 if d["dt"] == "f32" else 2
    loose = not d["vec"] and d["out"] == "f32" and d["bsrc"] in ("KC", "NC") and d["mb"] == 32 and d["bn"] == 64
    if loose and (d["bk"] == 64 and d["bm"] in (64, 128) if es == 2 else d["bk"] == 32 and d["bm"] == 64):
        return 8 if es == 4 else 4 if d["bm"] == 64 else 2
    one = d["direct"] or d["units"] or d["bsrc"] not in ("KC", "NC") or d["mb"] != 16 or d["bk"] * es != 256 or d["wm"] * d["wn"] > 2 * 256
    return 1 if one else 8


def _pad(v, row_bytes):
    if v == 1:
        return 0
    t = 64 if v >= 4 else 32
    return (3 * t - row_bytes % (2 * t)) % (2 * t)


def pad_n(d):
    """Row pad in bytes of a register-staged n-contiguous B tile (the kernel's PAD_N)."""
    return _pad(d["vn"], d["bn"] * (4 if d["dt"] == "f32" else 2))


def pad_m(d):
    """Row pad in bytes of an m-contiguous A tile (the kernel's PAD_M)."""
    return _pad(d["vm"], d["bm"] * (4 if d["dt"] == "f32" else 2))


def splittable(d):
    """Instances also compiled with split tiles (split-k): plainly fetched operands, two or more LDS stages; off the
    vector boundaries the fp32-output ones with a deep k tile."""
    if d["bsrc"] not in ("KC", "NC") or d["units"] or d["stages"] == 1:
        return False
    return d["vec"] == 1 or (d["out"] == "f32" and d["bk"] * (4 if d["dt"] == "f32" else 2) >= 128)


def lattice():
    out = []
    # 16-bit inputs, fp32 output: (BM, BN, BK, WM, WN, MB, VM, VN)
    tiles16 = [
        (256, 256, 64, 128, 128, 32, None, None),
        (256, 128, 64, 128, 64, 32, None, None),
        (128, 256, 64, 64, 128, 32, None, None),
        (128, 128, 64, 64, 64, 32, None, None),
        (128, 128, 64, 64, 64, 16, None, None),
        (128, 64, 64, 64, 32, 32, None, None),
        (64, 128, 64, 32, 64, 32, None, None),
        (64, 64, 64, 32, 32, 32, None, None),
        (64, 64, 64, 32, 32, 16, None, None),
        (32, 32, 64, 16, 16, 16, None, None),
        # eight waves per workgroup (two per SIMD)
        (256, 256, 64, 128, 64, 32, None, None),
        (256, 256, 64, 64, 128, 32, None, None),
        (256, 128, 64, 64, 64, 32, None, None),
        (128, 256, 64, 64, 64, 32, None, None),
        # other k depths
        (256, 256, 32, 128, 128, 32, None, None),
        (128, 128, 32, 64, 64, 32, None, None),
        (128, 128, 128, 64, 64, 32, None, None),
    ]
    for dt in ("f16", "bf16"):
        for bsrc in ("KC", "NC", "CONV"):
            for (bm, bn, bk, wm, wn, mb, vm, vn) in tiles16:
                out.append(_inst(dt, "f32", bm, bn, bk, wm, wn, mb, vm, vn, bsrc))
            # any alignment, any extents
            out.append(_inst(dt, "f32", 64, 64, 32, 32, 32, 16, None, None, bsrc, vec=0))
        # pointwise convolution with stride 2: the n-contiguous B operand sampled while it is fetched
        for (bm, bn, bk, wm, wn, mb, vm, vn) in tiles16:
            if bm * bn >= 64 * 64 and bk == 64 and mb == 32 and wm * wn < 128 * 128:
                out.append(_inst(dt, "f32", bm, bn, bk, wm, wn, mb, vm, vn, "NCS2"))
        # direct global->LDS staging for k-contiguous operands
        for (bm, bn, bk, wm, wn, mb, vm, vn) in tiles16:
            if bm * bn >= 128 * 128:
                out.append(_inst(dt, "f32", bm, bn, bk, wm, wn, mb, vm, vn, "KC", direct=1))
        # the same for an n-contiguous B (rows of at least 16 chunks: its swizzle needs them)
        for (bm, bn, bk, wm, wn, mb, vm, vn) in tiles16:
            if bm * bn >= 128 * 128 and bn >= 128:
                out.append(_inst(dt, "f32", bm, bn, bk, wm, wn, mb, vm, vn, "NC", direct=1))
        # a ring of three LDS stages (two k tiles in flight) for the mid-size eight-wave tiles; measured to pay
        # for k-contiguous operands only
        for (bm, bn) in ((128, 256), (256, 128)):
            out.append(_inst(dt, "f32", bm, bn, 64, 64, 64, 32, None, None, "KC", stages=3, direct=1))
        # one LDS stage: half the LDS, twice the resident workgroups, for contractions of a single k tile
        for bsrc in ("KC", "NC"):
            for (bm, bn, wm, wn) in ((128, 128, 64, 64), (128, 64, 64, 32)):
                out.append(_inst(dt, "f32", bm, bn, 64, wm, wn, 32, None, None, bsrc, stages=1))
        # 16-bit output variants
        out.append(_inst(dt, dt, 128, 128, 64, 64, 64, 32, None, None, "KC"))
        out.append(_inst(dt, dt, 128, 128, 64, 64, 64, 32, None, None, "NC"))
        out.append(_inst(dt, dt, 256, 256, 64, 128, 64, 32, None, None, "KC", direct=1))
        out.append(_inst(dt, dt, 128, 128, 64, 64, 64, 32, None, None, "KC", direct=1))
        out.append(_inst(dt, dt, 128, 256, 64, 64, 64, 32, None, None, "NC"))
        out.append(_inst(dt, dt, 256, 256, 64, 128, 64, 32, None, None, "NC"))
        out.append(_inst(dt, dt, 256, 256, 64, 128, 64, 32, None, None, "NCS2"))
        out.append(_inst(dt, dt, 64, 64, 32, 32, 32, 16, None, None, "KC", vec=0))
        out.append(_inst(dt, dt, 64, 64, 32, 32, 32, 16, None, None, "NC", vec=0))
        out.append(_inst(dt, dt, 128, 128, 64, 64, 64, 32, None, None, "CONV"))
        out.append(_inst(dt, dt, 64, 64, 32, 32, 32, 16, None, None, "CONV", vec=0))
        # patch-staged convolution: (BM filters, BN pixels, channels per stage, WM, WN, units)
        # two LDS stages (the 64x256 tile of 64x64 wave tiles compiles to one wave per SIMD with two stages
        # and is left out: its single-stage twin below is faster everywhere)
        for (bm, bn, bkc, wm, wn, units) in [(64, 128, 16, 32, 64, 1), (64, 64, 16, 32, 32, 1),
                                             (128, 128, 16, 64, 64, 1), (128, 256, 16, 64, 64, 1), (256, 128, 16, 64, 64, 1),
                                             (32, 256, 16, 32, 64, 1), (128, 128, 16, 64, 64, 2)]:
            out.append(_convp(dt, "f32", bm, bn, bkc, wm, wn, units))
        for (bm, bn, bkc, wm, wn, units) in [(64, 256, 16, 64, 64, 1), (64, 128, 16, 32, 64, 1), (64, 64, 16, 32, 32, 1),
                                             (32, 256, 16, 32, 64, 1), (32, 128, 16, 32, 32, 1), (64, 256, 16, 32, 64, 1),
                                             (64, 256, 16, 64, 64, 2), (128, 128, 16, 64, 64, 1), (128, 256, 16, 64, 64, 1),
                                             (128, 128, 16, 32, 64, 1)]:
            out.append(_convp(dt, "f32", bm, bn, bkc, wm, wn, units, stages=1))
        out.append(_convp(dt, dt, 64, 128, 16, 32, 64, 1))
        out.append(_convp(dt, dt, 64, 256, 16, 64, 64, 1, stages=1))
        out.append(_convp(dt, dt, 128, 256, 16, 64, 64, 1, stages=1))
    for (bm, bn, bkc, wm, wn, units) in [(64, 128, 8, 32, 64, 1), (64, 64, 8, 32, 32, 1), (128, 128, 8, 64, 64, 2)]:
        out.append(_convp("f32", "f32", bm, bn, bkc, wm, wn, units))
    tiles32 = [
        (128, 128, 32, 64, 64, 32, None, None),
        (64, 64, 32, 32, 32, 32, None, None),
        (64, 64, 32, 32, 32, 16, None, None),
        (32, 32, 32, 16, 16, 16, None, None),
        (64, 32, 32, 32, 16, 16, None, None),
    ]
    for (bm, bn, bk, wm, wn, mb, vm, vn) in tiles32[:3:2]:
        out.append(_inst("f32", "f32", bm, bn, bk, wm, wn, mb, vm, vn, "NCS2"))
    for bsrc in ("KC", "NC", "CONV"):
        for (bm, bn, bk, wm, wn, mb, vm, vn) in tiles32:
            out.append(_inst("f32", "f32", bm, bn, bk, wm, wn, mb, vm, vn, bsrc))
        out.append(_inst("f32", "f32", 64, 64, 16, 32, 32, 16, None, None, bsrc, vec=0))
    # 128x128 tiles of eight 64x32 waves (two workgroups, sixteen waves per CU), direct staging: the mid-size
    # shapes whose k loop waits on memory gain 3-6 % from the extra waves (appended last: ids above stay put)
    for dt in ("f16", "bf16"):
        for bsrc in ("KC", "NC"):
            out.append(_inst(dt, "f32", 128, 128, 64, 64, 32, 32, None, None, bsrc, direct=1))
    for dt in ("f16", "bf16"):
        for bsrc in ("KC", "NC"):
            out.append(_inst(dt, dt, 128, 128, 64, 64, 32, 32, None, None, bsrc, direct=1))
    # shallower virtual-thread interleaves of the tiles the benchmark shapes end in (fp16): what the walk can
    # reach when setVThread stops early, and all it can reach without setVThread (V = 1: the plain LDS layout)
    for bsrc in ("KC", "NC"):
        for (bm, bn, wm, wn) in ((256, 256, 128, 128), (256, 256, 128, 64), (128, 256, 64, 64), (256, 128, 64, 64),
                                 (128, 128, 64, 64), (128, 128, 64, 32)):
            for v in ((1, 2, 4) if (bm, bn, wm, wn) in ((256, 256, 128, 128), (128, 256, 64, 64), (128, 128, 64, 32)) else (1,)):
                out.append(_inst("f16", "f32", bm, bn, 64, wm, wn, 32, v, min(v, full_v("f16", 64, bsrc)[1]), bsrc, direct=1))
    for bsrc in ("KC", "NC"):
        out.append(_inst("f16", "f32", 128, 128, 64, 64, 64, 32, 1, 1, bsrc))
        out.append(_inst("f32", "f32", 64, 64, 32, 32, 32, 32, 1, 1, bsrc))
        out.append(_inst("f32", "f32", 32, 32, 32, 16, 16, 16, 1, 1, bsrc))
    out.append(_inst("f16", "f32", 256, 256, 64, 128, 64, 32, 1, 1, "NCS2"))
    out.append(_inst("f16", "f32", 128, 128, 64, 64, 64, 32, 1, 1, "CONV"))
    # A stored [k][m] (transA): register-staged instances, both B layouts
    for bsrc in ("KC", "NC"):
        for dt in ("f16", "bf16"):
            for (bm, bn, wm, wn, mb) in ((256, 256, 128, 64, 32), (256, 128, 64, 64, 32), (128, 256, 64, 64, 32), (128, 128, 64, 64, 32),
                                         (128, 128, 64, 64, 16), (64, 64, 32, 32, 32), (32, 32, 16, 16, 16)):
                out.append(_inst(dt, "f32", bm, bn, 64, wm, wn, mb, bsrc=bsrc, asrc="MC"))
            out.append(_inst(dt, "f32", 128, 128, 32, 64, 64, 32, bsrc=bsrc, asrc="MC"))
            out.append(_inst(dt, "f32", 128, 128, 64, 64, 64, 32, 1, 1, bsrc=bsrc, asrc="MC"))
            out.append(_inst(dt, "f32", 64, 64, 32, 32, 32, 16, bsrc=bsrc, vec=0, asrc="MC"))
            out.append(_inst(dt, dt, 128, 128, 64, 64, 64, 32, bsrc=bsrc, asrc="MC"))
            out.append(_inst(dt, dt, 64, 64, 32, 32, 32, 16, bsrc=bsrc, vec=0, asrc="MC"))
        for (bm, bn, wm, wn, mb) in ((128, 128, 64, 64, 32), (64, 64, 32, 32, 32), (64, 64, 32, 32, 16), (32, 32, 16, 16, 16)):
            out.append(_inst("f32", "f32", bm, bn, 32, wm, wn, mb, bsrc=bsrc, asrc="MC"))
        out.append(_inst("f32", "f32", 64, 64, 32, 32, 32, 32, 1, 1, bsrc=bsrc, asrc="MC"))
        out.append(_inst("f32", "f32", 64, 64, 16, 32, 32, 16, bsrc=bsrc, vec=0, asrc="MC"))
    # three-stage rings for an n-contiguous B (the mid-size eight-wave tiles), like the k-contiguous ones above
    for dt in ("f16", "bf16"):
        for (bm, bn) in ((128, 256), (256, 128)):
            out.append(_inst(dt, "f32", bm, bn, 64, 64, 64, 32, bsrc="NC", stages=3, direct=1))
    # operands at any alignment and with any extents (vec = 0), register-staged: the tiles a large problem wants, beside
    # the 64x64x32 ones above
    for bsrc, asrc in product(("KC", "NC"), ("KC", "MC")):
        for dt in ("f16", "bf16"):
            for odt in ("f32", dt):
                for (bm, bn, wm, wn) in ((128, 128, 64, 64), (128, 64, 64, 32), (64, 64, 32, 32)):
                    out.append(_inst(dt, odt, bm, bn, 64, wm, wn, 32, bsrc=bsrc, vec=0, asrc=asrc))
        for (bm, bn, wm, wn) in ((128, 128, 64, 64), (64, 64, 32, 32)):
            out.append(_inst("f32", "f32", bm, bn, 32, wm, wn, 32, bsrc=bsrc, vec=0, asrc=asrc))
    # A stored [k][m] staged directly, as an n-contiguous B is: two stages, and rings of three for the mid-size tiles
    for bsrc in ("KC", "NC"):
        for dt in ("f16", "bf16"):
            for (bm, bn, wm, wn) in ((256, 256, 128, 64), (256, 128, 64, 64), (128, 256, 64, 64), (128, 128, 64, 64), (128, 128, 64, 32)):
                out.append(_inst(dt, "f32", bm, bn, 64, wm, wn, 32, bsrc=bsrc, direct=1, asrc="MC"))
            for (bm, bn) in ((128, 256), (256, 128)):
                out.append(_inst(dt, "f32", bm, bn, 64, 64, 64, 32, bsrc=bsrc, stages=3, direct=1, asrc="MC"))
    # row-staged convolution: (BM filters, BN pixels, WM, WN); channels per stage are chosen per problem
    for dt, odt in (("f16", "f32"), ("f16", "f16"), ("bf16", "f32"), ("bf16", "bf16"), ("f32", "f32")):
        for (bm, bn, wm, wn) in ((64, 256, 64, 64), (64, 256, 32, 64), (32, 256, 32, 32), (32, 128, 32, 32)):
            out.append(_inst(dt, odt, bm, bn, 16 if dt != "f32" else 8, wm, wn, 32, 1, 1, "CONV", vec=0, stages=1, direct=1))
    # rings of three with output in the input type, for the mid-size tiles: what these shapes had ended in was a
    # register-staged tile (8192 x 3072 x 768 bf16, row-major B: 46-52 -> 42.4 us; 8192 x 768 x 3072, column-major B:
    # 42.4 -> 38.1 us; 2119 x 2816 x 704 f16: 13.8 -> 12.3 us)
    for dt in ("f16", "bf16"):
        for bsrc in ("KC", "NC"):
            for (bm, bn) in ((128, 256), (256, 128)):
                out.append(_inst(dt, dt, bm, bn, 64, 64, 64, 32, bsrc=bsrc, stages=3, direct=1))
        out.append(_inst(dt, dt, 256, 256, 64, 128, 64, 32, bsrc="NC", direct=1))
    # 256x256 tiles of eight waves of 16x16 blocks whose two halves alternate
    for dt in ("f16", "bf16"):
        for bsrc, asrc in product(("KC", "NC"), ("KC", "MC")):
            for odt in ("f32", dt):
                if odt == "f32" or asrc == "KC":
                    out.append(_inst(dt, odt, 256, 256, 64, 128, 64, 16, bsrc=bsrc, direct=1, asrc=asrc))
    # rings of four stages for the 128x128 tiles of eight 64x32 waves: launches of about one tile per compute unit, where one
    # k tile in flight does not cover the latency (1280 x 1792 x 2048 f16 20.5 -> 17.1 us, 1536 x 2304 x 3072 32.5 -> 27.9,
    # 1856 x 1280 x 3264 30.8 -> 25.6, 1024 x 3072 x 768 row-major B 11.9 -> 10.0, 3072 x 768 x 4096 transA 34.0 -> 32.3).  Five stages
    # are within 3 % either way.  Four 64x64 waves are 6-15 % slower on whole tiles (1216 x 2880 x 3456 f16 35.7 against 32.4 us, 4093 x 512 x
    # 2048 18.4 against 16.7) and within 8 % either way on parts (376 x 528 x 32512 in 16 26.9 both, 392 x 448 x 26688 in 16 22.5 against 24.3).
    for dt in ("f16", "bf16"):
        for bsrc, asrc in product(("KC", "NC"), ("KC", "MC")):
            for odt in ("f32", dt):
                if odt == "f32" or asrc == "KC":
                    out.append(_inst(dt, odt, 128, 128, 64, 64, 32, 32, bsrc=bsrc, stages=4, direct=1, asrc=asrc))
        # They are compiled where both operands are k-contiguous: there the walks reach the eight-wave state less often, and what such
        # shapes took without them is slower still (1216 x 2880 x 3456 37.6, 4093 x 512 x 2048 21.7, 392 x 448 x 26688 28.0)
        for odt in ("f32", dt):
            out.append(_inst(dt, odt, 128, 128, 64, 64, 64, 32, stages=4, direct=1))
    # the rings of 16x16 blocks (the kernel's RING_16).  128x128 tiles only where neither operand is transposed while it is read, of which
    # 16x16 blocks need more: m-contiguous A 2048^3 22.9 against 23.9 us, 1536 x 2304 x 3072 29.1 against 30.9; n-contiguous B within 5 %
    # either way (1600 x 1216 x 3776 32.0 against 33.6, 1280 x 1664 x 1664 16.7 against 17.5, 2048^3 23.8 against 22.7).  128x256 tiles are taken by a
    # tenth as many of 4800 drawn products as 256x128 ones, three quarters of them weight gradients of 576 to 960 rows (576 x 2304 x 6192 transA
    # 36.9 -> 34.0, 896 x 3584 x 4720 51.8 -> 47.0), the others where they leave fewer partial tiles (2688 x 3072 x 1088 25.0 -> 23.1,
    # 2049 x 3840 x 960 with 16-bit output 21.5 -> 20.8; pointwise 6 x 304 x 52 x 52 -> 336 10.1 -> 9.3).
    for dt in ("f16", "bf16"):
        for bsrc, asrc in product(("KC", "NC"), ("KC", "MC")):
            for odt in ("f32", dt):
                if odt == "f32" or asrc == "KC":
                    for (bm, bn) in ((256, 128), (128, 256)):
                        out.append(_inst(dt, odt, bm, bn, 64, 64, 64, 16, bsrc=bsrc, stages=3, direct=1, asrc=asrc))
                if asrc == "KC" and bsrc == "KC":
                    out.append(_inst(dt, odt, 128, 128, 64, 64, 32, 16, stages=4, direct=1))
    # Small products, whose k loop is a chain of waits (request, LDS, barrier, fragments, products on one wave per SIMD): twice the
    # k depth per barrier (512^3 fp32 6.9 -> 6.0 us, 671 x 2304 x 576 f16 13.1 -> 10.7), and at any alignment tiles small enough for a workgroup on
    # every compute unit (311 x 535 x 487 fp32 11.4 -> 8.2, 1277 x 1923 x 165 f16 12.6 -> 9.6).  64x64 tiles of that depth were 4-8 % faster than
    # their halves where a compute unit holds one workgroup and 10-28 % slower where it holds more (704 x 2816 x 1480 transA 17.7 against 20.1).
    for bsrc, asrc in product(("KC", "NC"), ("KC", "MC")):
        for dt in ("f16", "bf16"):
            out.append(_inst(dt, "f32", 32, 32, 128, 16, 16, 16, bsrc=bsrc, asrc=asrc))
            for odt in ("f32", dt):
                out.append(_inst(dt, odt, 32, 32, 128, 16, 16, 16, bsrc=bsrc, vec=0, asrc=asrc))
        out.append(_inst("f32", "f32", 32, 32, 64, 16, 16, 16, bsrc=bsrc, asrc=asrc))
        out.append(_inst("f32", "f32", 32, 32, 64, 16, 16, 16, bsrc=bsrc, vec=0, asrc=asrc))
        out.append(_inst("f32", "f32", 64, 32, 64, 32, 16, 16, bsrc=bsrc, vec=0, asrc=asrc))
    # eight 64x32 waves for the large any-alignment tile: one wave per SIMD covers none of its waits (2039 x 1511 x 1003 bf16 19.2 -> 17.3 us,
    # 1533 x 2041 x 1999 f16 31.9 -> 28.0)
    for bsrc, asrc in product(("KC", "NC"), ("KC", "MC")):
        for dt in ("f16", "bf16"):
            for odt in ("f32", dt):
                out.append(_inst(dt, odt, 128, 128, 64, 64, 32, 32, bsrc=bsrc, vec=0, asrc=asrc))
    # Patch-staged convolution with twice (and four times) the channels per stage.  A stage is a round trip to memory, which a compute
    # unit with one or two workgroups does not cover, and the smaller tiles fill a quarter to half of the staging units their threads have.
    # Best with 16 channels -> best, us: 24 x 248 x 17 x 17, 112 filters, stride 2, f16 26.2 -> 15.2; 8 x 224 x 17 x 17, 192 filters, stride 2, bf16 20.3
    # -> 13.6; 8 x 56 x 15 x 15, 208 filters 10.1 -> 7.2; 35 x 152 x 19 x 19, 72 filters 19.2 -> 14.3.  (64x256 tiles gain 3 % on inputs that stay and
    # lose 2 on ones that change, 32 x 64 x 56 x 56, 64 filters.)
    for dt in ("f16", "bf16"):
        for odt in ("f32", dt):
            for (bm, bn, wm, wn) in ((32, 128, 32, 32), (32, 256, 32, 64), (64, 128, 32, 64), (64, 64, 32, 32)):
                out.append(_convp(dt, odt, bm, bn, 32, wm, wn, 1, stages=1))
            out.append(_convp(dt, odt, 32, 128, 64, 32, 32, 1, stages=1))
    for (bm, bn, wm, wn) in ((32, 128, 32, 32), (64, 64, 32, 32), (64, 128, 32, 64)):
        out.append(_convp("f32", "f32", bm, bn, 16, wm, wn, 1, stages=1))
    # Small aligned tiles with output in the input type, which ended in large tiles or split ones: 495 x 512 x 2048 f16 12.5 -> 7.5 us, 908 x 512
    # x 2048 bf16 14.1 -> 9.7, 330 x 704 x 2816 13.0 -> 9.6, 410 x 2048 x 512 7.0 -> 5.9, 49 x 920 x 64 x 920 20.2 -> 18.5.
    for dt in ("f16", "bf16"):
        for bsrc in ("KC", "NC"):
            out.append(_inst(dt, dt, 32, 32, 128, 16, 16, 16, bsrc=bsrc))
            out.append(_inst(dt, dt, 64, 64, 64, 32, 32, 32, bsrc=bsrc))
    for i, d in enumerate(out):
        d["id"] = i
    keys = [(d["dt"], d["out"], d["bm"], d["bn"], d["bk"], d["wm"], d["wn"], d["mb"], d["vm"], d["vn"], d["bsrc"], d["vec"],
             d["stages"], d["direct"], d["units"], d["asrc"]) for d in out]
    assert len(set(keys)) == len(keys), "duplicate instance"
    return out


def cfg_type(d):
    if conv_rows(d):
        return "ConvRowsCfg<%s, %s, %d, %d, %d, %d>" % (CT[d["dt"]], CT[d["out"]], d["bm"], d["bn"], d["wm"], d["wn"])
    if d["units"]:
        return "ConvCfg<%s, %s, %d, %d, %d, %d, %d, %d, %d, %d>" % (
            CT[d["dt"]], CT[d["out"]], d["bm"], d["bn"], d["bk"], d["wm"], d["wn"], d["mb"], d["units"], d["stages"])
    return ("Cfg<%s, %s, %d, %d, %d, %d, %d, %d, %d, %d, %d, %s, %d, %s, %d>" % (
        CT[d["dt"]], CT[d["out"]], d["bm"], d["bn"], d["bk"], d["wm"], d["wn"], d["mb"], d["vm"], d["vn"],
        BSRC[d["bsrc"]], "true" if d["vec"] else "false", d["stages"], "true" if d["direct"] else "false", ASRC[d["asrc"]]))


if __name__ == "__main__":
    L = lattice()
    print(len(L), "instances")
