"""Scratch plans and launch shapes, checked on the host: programs that include the library's
sources are compiled without device code and run on the CPU."""
import os
import shutil
import subprocess

import pytest

from paper_2302_13529_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))
needs_hipcc = pytest.mark.skipif(not (os.path.exists(build.HIPCC) or shutil.which("hipcc")),
                                 reason="hipcc not available")


def run_host(tmp_path, program, sources):
    """The program's output; kernels are left undefined, none is launched."""
    objects = []
    for src in [os.path.join(HERE, program)] + [os.path.join(build.CSRC, s) for s in sources]:
        obj = str(tmp_path / (os.path.basename(src) + ".o"))
        subprocess.check_call([build.HIPCC, "-x", "hip", "--offload-arch=gfx950",
                               "--offload-host-only", "-O2", "-std=c++17", "-I",
                               os.path.join(build.ROOT, "include"), "-I", build.CSRC, "-c", src,
                               "-o", obj], stderr=subprocess.DEVNULL)
        objects.append(obj)
    exe = str(tmp_path / "check")
    subprocess.check_call([build.HIPCC, "-o", exe, *objects,
                           "-Wl,--unresolved-symbols=ignore-all"], stderr=subprocess.DEVNULL)
    res = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert res.returncode == 0, (res.returncode, res.stdout, res.stderr)
    return res.stdout


@needs_hipcc
def test_noalloc_plans(tmp_path):
    assert "plans ok" in run_host(tmp_path, "plan_check.cpp", ["api.cpp", "tree.hip"])


@needs_hipcc
def test_tree_shapes(tmp_path):
    assert "shapes ok" in run_host(tmp_path, "shape_check.cpp", [])
