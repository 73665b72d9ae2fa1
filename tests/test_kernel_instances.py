"""The kernels that the library holds are the ones that its launch plans can ask for
(tests/c/kernel_instances.cpp, host side only): none is missing and none is out of reach."""
import collections
import os
import re
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
PKG = os.path.join(ROOT, "paper_1111_1373_amd")


def test_every_planned_kernel_exists_and_no_other(tmp_path):
    lib = os.path.join(PKG, "libdtree.so")
    if shutil.which("g++") is None or not os.path.exists(lib):
        pytest.skip("needs g++ and the built library")
    import torch  # noqa: F401  (the HIP runtime that the library binds to)
    exe = str(tmp_path / "kernel_instances")
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                    "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(PKG, "csrc"),
                    os.path.join(ROOT, "tests", "c", "kernel_instances.cpp"),
                    "-L" + PKG, "-ldtree", "-Wl,-rpath," + PKG, "-o", exe],
                   check=True, capture_output=True, text=True)
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.startswith("ok "), r.stdout + r.stderr
    # kernel descriptors in the device code: one name per kernel, each as often as the others
    # (in a code object's two symbol tables); a kernel that several units hold appears more often
    with open(lib, "rb") as f:
        names = collections.Counter(re.findall(rb"[\w.$]+\.kd\0", f.read()))
    assert len(set(names.values())) == 1, names.most_common(1)
    tree_kernels = [n for n in names if b"copy_kernel" not in n and b"read_kernel" not in n]
    assert int(r.stdout.split()[1]) == len(tree_kernels)
