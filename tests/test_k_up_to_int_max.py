"""Loop bounds of the GEMM kernels at reductions near INT32_MAX, evaluated by the compiler: a bound that overflows is no constant
expression, so the translation unit below does not compile."""
import os
import subprocess
import sys

import pytest

sys.path.insert(0, os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2502_11407_amd", "csrc"))
import build as kernel_build  # noqa: E402

SOURCE = """
#include "registry.hpp"
namespace gensor {
constexpr int walk(int bk, int beyond, int K, int from) {        // the first kt at which a step of two tiles no longer has four inside
  int kt = from;
  while (tiles_inside(kt, 4, bk, beyond, K)) kt += 2;
  return kt;
}
template <int BK, int BEYOND, int K> constexpr bool right() {
  constexpr int from = (K / BK - 40) / 2 * 2;
  constexpr int kt = walk(BK, BEYOND, K, from);
  return kt > from && kt * (long long)BK + 4ll * BK + BEYOND > K && (kt - 2) * (long long)BK + 4ll * BK + BEYOND <= K;
}
static_assert(right<64, 7, 0x7fffffff - 100>() && right<64, 0, 0x7fffffff>() && right<32, 7, 0x7fffffff - 63>() && right<32, 3, 0x7fffffff - 7>(), "");
static_assert(right<64, 7, 1 << 20>() && right<32, 0, 100003>(), "");
static_assert(!tiles_inside(0, 4, 64, 7, 1) && !tiles_inside(0, 4, 64, 7, 262) && tiles_inside(0, 4, 64, 7, 263) && tiles_inside(0, 4, 64, 0, 256), "");
}
"""


def test_inner_tiles_of_reductions_up_to_int_max(tmp_path):
    src = tmp_path / "bounds.hip"
    src.write_text(SOURCE)
    r = subprocess.run([kernel_build.HIPCC] + kernel_build.FLAGS + ["-x", "hip", "--cuda-device-only", "-fsyntax-only", str(src)],
                       capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("M,N", [(9, 7), (8, 8), (16, 24), (64, 32)])
@pytest.mark.parametrize("short", [200, 127, 100, 64, 40, 32])
def test_constructed_k_tiles_end_inside_32_bits(dtype, M, N, short):
    """An m-contiguous A beside a row-major B: K up to INT32_MAX with rows of a few elements.  Tiles whose last k tile would end beyond are not taken."""
    from paper_2502_11407_amd import binding as gs
    K = 2 ** 31 - short
    s = gs.construct(gs.gemm_problem(dtype, M, N, K, 1, 0))
    assert K + s.tile[2][0] - 1 <= 2 ** 31 - 1
    p = gs.gemm_problem(dtype, M, N, K, 1, 0)
    assert all(t is None or K + t.tile[2][0] - 1 <= 2 ** 31 - 1 for t in (gs.instance_schedule(i, p) for i in range(gs.num_instances())))


def test_k_beyond_every_tiles_last_end_is_refused():
    from paper_2502_11407_amd import binding as gs
    with pytest.raises(gs.GensorError):
        gs.construct(gs.gemm_problem("f16", 16, 24, 2 ** 31 - 31, 1, 0))
