"""The library's launch plans, for CPU tests: csrc/plan.h compiled with g++
into a small shared object and called through ctypes."""
import ctypes
import os
import shutil
import subprocess
from ctypes import POINTER, byref, c_int, c_int64

from paper_2609_05707_amd import _lib as L
from paper_2609_05707_amd import build as B

SOURCE = r"""
#include "plan.h"
extern "C" int step_plan(const ippd_batch_t* bt, int shared, int dense, int64_t* out) {
  ippd::StepPlan p;
  if (!ippd::plan_step(bt, shared != 0, &p, dense != 0)) return 0;
  const int64_t v[] = {p.waves, p.rb, p.nrg, p.chunk, p.max_chunks, p.n_groups, p.grid, p.ctx_blocks, p.seg_blocks,
                       p.seg_tpu, p.deep, p.n_igroups, p.nrg_i, p.max_ichunks, p.instr_blocks,
                       (int64_t)p.workspace_bytes};
  for (size_t i = 0; i < sizeof v / sizeof *v; ++i) out[i] = v[i];
  return 1;
}
extern "C" int segment_lds(int elem, int head_dim, int waves, int deep) {
  return ippd::segment_main_bytes(elem, head_dim, waves,
                                  ippd::ring_stages(elem, head_dim, deep != 0) * ippd::ring_stage_bytes(elem, head_dim));
}
"""
FIELDS = ["waves", "rb", "nrg", "chunk", "max_chunks", "n_groups", "grid", "ctx_blocks", "seg_blocks", "seg_tpu", "deep",
          "n_igroups", "nrg_i", "max_ichunks", "instr_blocks", "workspace_bytes"]


class Plans:
    def __init__(self, path):
        self.lib = ctypes.CDLL(path)
        self.lib.step_plan.argtypes = [POINTER(L.IppdBatch), c_int, c_int, POINTER(c_int64)]

    def step(self, bt, shared=True, dense=False):
        """Plan fields of a decode call, or None where it is refused."""
        out = (c_int64 * len(FIELDS))()
        if not self.lib.step_plan(byref(bt), int(shared), int(dense), out):
            return None
        return dict(zip(FIELDS, out))


def build(folder):
    src, so = os.path.join(folder, "plan_probe.cpp"), os.path.join(folder, "plan_probe.so")
    with open(src, "w") as f:
        f.write(SOURCE)
    cmd = [shutil.which("g++"), "-std=c++17", "-O1", "-Wall", "-Werror", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
           f"-I{B.INCLUDE}", f"-I{B.CSRC}", "-isystem", "/opt/rocm/include", src, "-o", so]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return Plans(so)
