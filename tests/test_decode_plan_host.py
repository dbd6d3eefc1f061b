"""The decode split rule on the host: a call never takes more partials than the
memory sized for it holds, and never other splits than that size stands
for but where more can pay.  The rule's source is compiled here
with a C interface of its own, without the kernels."""
import ctypes
import itertools
import os
import shutil
import subprocess

import pytest

from paper_2608_04771_amd.build import CSRC

SHIM = """
#include "decode_plan.hpp"
extern "C" int sized(int units, int cap, int cus) { return reco::decode_splits(units, cap, cus); }
extern "C" int launched(int splits, int units, int cap, int group, int dim, int elem, int cus) {
  return reco::decode_launch_splits(splits, units, cap, group, dim, elem, cus);
}
extern "C" int sized_static(int units, int cap, int dim, int cus) {
  return reco::decode_scratch_splits(units, cap, dim, cus);
}
extern "C" size_t written(int units, int splits, int group, int dim) {
  return reco::decode_partials_bytes(units, splits, group, dim);
}
extern "C" size_t static_bytes() { return reco::kDecodeScratchBytes; }
extern "C" size_t workspace(int units, int cap, int dim, int cus) {
  return reco::decode_workspace_bytes(units, cap, dim, cus);
}
"""


@pytest.fixture(scope="module")
def plan(tmp_path_factory):
    cxx = shutil.which("g++") or shutil.which("c++")
    if cxx is None:
        pytest.skip("no C++ compiler")
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "plan.so")
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(d / "shim.cpp"),
                    os.path.join(CSRC, "decode_plan.cpp"), "-o", so], check=True)
    lib = ctypes.CDLL(so)
    for f in (lib.written, lib.static_bytes, lib.workspace):
        f.restype = ctypes.c_size_t
    return lib


@pytest.mark.parametrize("cus", [1, 32, 64, 256, 304])
@pytest.mark.parametrize("dim,elem", [(64, 2), (64, 4), (128, 2), (128, 4)])
def test_partials_fit_and_splits_stay_in_range(plan, cus, dim, elem):
    caps = [1, 31, 255, 256, 4095, 5120, 9709, 10240, 16640, 32832, 65600, 1 << 20]
    units = sorted({1, 2, 3, 4, 7, 16, 31, 32, 96, 112, 127, 128, 129, 152, 200, 255, 256, 257, 512, 65535, cus,
                    cus + 1, max(1, 3 * cus // 8), max(1, cus // 2)})
    raised = 0
    for u, cap, group in itertools.product(units, caps, range(1, 17)):
        base = plan.sized(u, cap, cus)
        assert 1 <= base <= 128, (u, cap, group)
        s = plan.launched(base, u, cap, group, dim, elem, cus)
        # group x D outputs and 2 x group statistics a split, in the room of 16 x D + 32 a sized split
        assert s * group * (dim + 2) <= base * (16 * dim + 32), (u, cap, group)
        assert plan.written(u, s, group, dim) == (0 if s == 1 else u * s * group * (dim + 2) * 4)
        assert plan.written(u, s, group, dim) <= plan.workspace(u, cap, dim, cus), (u, cap, group)
        # the static array of allocation-free calls: what they launch fits it, and what they write is what is checked
        b = plan.sized_static(u, cap, dim, cus)
        t = plan.launched(b, u, cap, group, dim, elem, cus)
        assert b in (base, 1) and (t == s or b == 1), (u, cap, group)
        assert plan.written(u, t, group, dim) <= plan.static_bytes(), (u, cap, group)
        if s != base:
            raised += 1
            # a merge there is anyway, lengths that a wave holds, 1.5 to 2 workgroups a compute unit, long enough
            assert base == 2 and s in (4, 5) and u <= 128 and 3 * cus <= 2 * u * s <= 4 * cus, (u, cap, group)
            assert (cap + 32) // 32 >= 320, (u, cap, group)
            assert dim * elem == 256 or 5 * u * base <= 4 * cus, (u, cap, group)
    assert raised > 0 or cus == 1
