"""bench.py finds a kernel class's dispatches in a counter run by the kernel's name: every pattern
has to match a kernel of the built library."""
import os
import re
import shutil
import subprocess

import pytest

import bench

M = pytest.importorskip("paper_2505_00793_amd._lib")


@pytest.mark.skipif(shutil.which("nm") is None, reason="no nm")
def test_class_patterns_name_built_kernels():
    if not os.path.exists(M.LIB_PATH):
        pytest.skip("libmfmg.so not built")
    names = subprocess.run(["nm", "-C", M.LIB_PATH], capture_output=True, text=True,
                           check=True).stdout
    for cls, pattern in bench.CLASS_KERNEL.items():
        assert re.search(pattern, names), cls
