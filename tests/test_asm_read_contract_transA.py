"""The wait contract of test_asm_read_contract.py (every LDS read issued from inline assembly is waited for before its
register is touched) on the instances with a directly staged m-contiguous A, whatever their B."""
import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

from test_asm_read_contract import _functions, check_function


def test_every_direct_staged_transA_instance_waits_for_its_reads(tmp_path):
    import build as kernel_build
    import lattice
    insts = [d for d in lattice.lattice() if d["asrc"] == "MC" and d["direct"] and d["dt"] == "f16"]
    assert len(insts) >= 10

    def one(d):
        src, out = tmp_path / ("t%d.hip" % d["id"]), tmp_path / ("t%d.s" % d["id"])
        src.write_text('#include "registry.hpp"\nnamespace gensor {\ntypedef %s C_X;\n'
                       "hipError_t l0(const KernelArgs& a, hipStream_t st) { return launch_instance<C_X>(a, st); }\n"
                       "hipError_t l1(const KernelArgs& a, hipStream_t st) { return launch_instance<C_X, true>(a, st); }\n}\n" % lattice.cfg_type(d))
        r = subprocess.run([kernel_build.HIPCC] + kernel_build.FLAGS + ["-x", "hip", "--cuda-device-only", "-S", str(src), "-o", str(out)],
                           capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-2000:]
        return d["id"], [check_function(fn) for fn in _functions(out.read_text())]

    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as ex:
        for idx, res in ex.map(one, insts):
            assert len(res) >= 2, idx
            for violations, reads in res:
                assert reads > 0 and not violations, "instance %d: %s" % (idx, violations[:3])
