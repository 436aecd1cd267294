"""The library's host code with every launch replaced by a recorder, built from source for the CPU tests of what a call is
dispatched to: nothing reaches a GPU, so operands may be made-up addresses, also on a machine that has one."""
import ctypes as C
import os
import subprocess
import sys

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2502_11407_amd", "csrc")

RECORDER = """
#include "registry.hpp"
namespace gensor {
static int32_t last[11];
static hipError_t record(int id, int split, const KernelArgs& a) {
  const int32_t v[11] = {last[0] + 1, id, split, a.narrow, a.tiles_m, a.tiles_n, a.batch, a.whole, a.split, a.paired, a.lds_stages};
  for (int i = 0; i < 11; ++i) last[i] = v[i];
  return hipErrorNotSupported;
}
%s
}
extern "C" const int32_t* last_launch(void) { return gensor::last; }
"""
FIELDS = ("count", "id", "split_launch", "narrow", "tiles_m", "tiles_n", "batch", "whole", "split", "paired", "lds_stages")
ACCEPTED = 5          # GENSOR_ERR_DEVICE: what the recorder's error becomes, once everything before the launch has passed
A, B, OUT, WORKSPACE = (1 << 40) * 1, (1 << 40) * 2, (1 << 40) * 3, (1 << 40) * 4


class Stub:
    def __init__(self, folder):
        sys.path.insert(0, CSRC)
        import build as kernel_build
        import lattice
        from paper_2502_11407_amd import binding as gs
        kernel_build.generate()
        body = []
        for d in lattice.lattice():
            body.append("hipError_t launch_%d(const KernelArgs& a, hipStream_t) { return record(%d, 0, a); }" % (d["id"], d["id"]))
            if lattice.splittable(d):
                body.append("hipError_t launch_split_%d(const KernelArgs& a, hipStream_t) { return record(%d, 1, a); }" % (d["id"], d["id"]))
        stubs = os.path.join(str(folder), "stubs.cpp")
        with open(stubs, "w") as f:
            f.write(RECORDER % "\n".join(body))
        flags = [x if x != "-O3" else "-O1" for x in kernel_build.FLAGS] + ["-ffp-contract=off", "-x", "hip"]
        jobs, objs = [], []
        for src in ("constructor.cpp", "gensor_api.cpp", "scan_kernels.cpp", os.path.join("_build", "registry.hip"), stubs):
            objs.append(os.path.join(str(folder), os.path.basename(src) + ".o"))
            jobs.append(subprocess.Popen([kernel_build.HIPCC] + flags + ["-c", os.path.join(CSRC, src), "-o", objs[-1]],
                                         stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True))
        for j in jobs:
            out = j.communicate()[0]
            assert j.returncode == 0, out[-3000:]
        path = os.path.join(str(folder), "libstub.so")
        subprocess.run([kernel_build.HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", path] + objs, check=True)
        self.gs, self.lib = gs, C.CDLL(path)
        for name in gs.EXPORTS:
            f, g = getattr(self.lib, name), getattr(gs.lib, name)
            f.restype, f.argtypes = g.restype, g.argtypes
        self.lib.last_launch.restype = C.POINTER(C.c_int32)

    def last(self):
        return dict(zip(FIELDS, self.lib.last_launch()[:len(FIELDS)]))

    def construct(self, p):
        s = self.gs.Schedule()
        assert self.lib.gensor_construct(C.byref(p), None, None, 0, C.byref(s)) == 0
        return s

    def workspace_bytes(self, p, s):
        return int(self.lib.gensor_workspace_bytes(C.byref(s), C.byref(p)))

    def call(self, p, s=None, lda=None, ldb=None, ldc=None, room=0, beta=0.0, static=False):
        """Status of one product on made-up addresses, and what it would have launched (None: nothing)."""
        before = self.last()["count"]
        lda, ldb, ldc = lda or (p.M if p.transA else p.K), ldb or (p.K if p.transB else p.N), ldc or p.N
        s = C.byref(s) if s is not None else None
        if static:
            st = self.lib.gensor_gemm_static_scratch(s, C.byref(p), 1.0, A, lda, B, ldb, beta, OUT, ldc, None)
        else:
            rows = lambda t, r, c, ld: (c if t else r) * ld
            st = self.lib.gensor_bmm(s, C.byref(p), 1.0, A, lda, rows(p.transA, p.M, p.K, lda), B, ldb, rows(p.transB, p.K, p.N, ldb),
                                     beta, OUT, ldc, p.M * ldc, WORKSPACE if room else None, room, None)
        last = self.last()
        return st, last if last["count"] != before else None
