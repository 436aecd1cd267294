"""Register counts that rules in the kernels rely on, read from the compiler's own figures for this repository's kernels."""
import os
import re
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

sys.path.insert(0, os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_11407_amd", "csrc"))
import build as kernel_build  # noqa: E402
import lattice  # noqa: E402


def _counts(tmp_path, insts, launcher, extra=()):
    """(instance, registers, spilled registers) of every kernel the launches of these instances instantiate."""
    src, out = tmp_path / "k.hip", tmp_path / "k.s"
    lines = ['#include "registry.hpp"', "namespace gensor {"]
    for d in insts:
        lines.append("typedef %s C_%d;" % (lattice.cfg_type(d), d["id"]))
        for j, call in enumerate(launcher):
            lines.append("hipError_t l%d_%d(const KernelArgs& a, hipStream_t st) { return %s(a, st); }" % (d["id"], j, call % ("C_%d" % d["id"])))
    src.write_text("\n".join(lines + ["}\n"]))
    r = subprocess.run([kernel_build.HIPCC] + kernel_build.FLAGS + list(extra) + ["-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(out)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    text = out.read_text()
    regs = [int(x) for x in re.findall(r"\.vgpr_count:\s+(\d+)", text)]
    spills = [int(x) for x in re.findall(r"\.vgpr_spill_count:\s+(\d+)", text)]
    assert len(regs) == len(spills) >= len(insts)
    return list(zip(re.findall(r"\.name:\s+(_ZN6gensor\S+)", text), regs, spills))


def test_large_tiles_of_16x16_blocks_keep_two_waves_per_simd(tmp_path):
    """Their LDS leaves two workgroups of four waves per CU; more than 256 registers would leave one."""
    insts = [d for d in lattice.lattice() if d["dt"] == "f16" and d["mb"] == 16 and d["bm"] == 128 and d["vec"] == 1 and d["bsrc"] in ("KC", "NC")]
    assert len(insts) >= 4
    for name, regs, spilled in _counts(tmp_path, insts, ("launch_instance<%s>", "launch_instance<%s, true>")):
        assert regs <= 256 and spilled == 0, (name, regs, spilled)


def test_alternating_groups_keep_two_waves_per_simd(tmp_path):
    """256x256 tiles of eight waves, 254-256 registers a lane: one more would leave one wave per SIMD, or spill.  The launch of a whole
    tile instantiates the 192-column form, too."""
    insts = [d for d in lattice.lattice() if lattice.alternate(d)]
    assert len(insts) == 12

    def one(d):
        folder = tmp_path / str(d["id"])
        folder.mkdir()
        return _counts(folder, [d], ("launch_instance<%s>", "launch_instance<%s, true>"))

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        for kernels in ex.map(one, insts):
            assert len(kernels) == 3                       # wide, narrow, split
            for name, regs, spilled in kernels:
                assert regs <= 256 and spilled == 0, (name, regs, spilled)


def test_row_staged_convolution_does_not_spill(tmp_path):
    insts = [d for d in lattice.lattice() if lattice.conv_rows(d) and (d["dt"], d["out"]) in (("f16", "f32"), ("bf16", "bf16"), ("f32", "f32"))]
    assert len(insts) == 12
    for name, regs, spilled in _counts(tmp_path, insts, ("launch_conv_rows<%s>",), kernel_build.CONV_FLAGS):
        assert spilled == 0, (name, regs, spilled)


def test_tiles_of_several_sums_do_not_spill(tmp_path):
    """Rings of 16x16 blocks with 64x64 waves (one workgroup of eight waves a CU: 256 registers) and the any-alignment tiles that keep more sums in
    deep launches: 64x64 16-bit ones with three workgroups a CU (170 registers), 128x64 and fp32 ones with two."""
    insts = [d for d in lattice.lattice() if d["dt"] in ("f16", "f32") and d["out"] == "f32" and d["bsrc"] in ("KC", "NC") and not d["units"]]
    rings = [d for d in insts if d["direct"] and d["stages"] == 3 and d["mb"] == 16]
    loose = [d for d in insts if d["mb"] == 32 and lattice.chains(d) > 1]
    assert len(rings) == 8 and len(loose) == 12
    launches = ("launch_instance<%s>", "launch_instance<%s, true>")

    def one(item):
        d, extra = item
        folder = tmp_path / str(d["id"])
        folder.mkdir()
        return d, _counts(folder, [d], launches, extra)

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        for d, kernels in ex.map(one, [(d, ()) for d in rings] + [(d, kernel_build.CONV_FLAGS) for d in loose]):
            assert len(kernels) == 4                           # whole and split, each with one sum and with several
            most = 256 if d in rings or d["dt"] == "f32" or d["bm"] == 128 else 170
            for name, regs, spilled in kernels:
                assert regs <= most and spilled == 0, (d["id"], name, regs, spilled)
