"""The kernels and the host side compile without a warning (among them stores
that claim more alignment than their type has)."""
import os
import subprocess

import pytest

from paper_1712_09789_amd import build as b


@pytest.mark.parametrize("source,defines", [
    ("ccl_kernels.hip", [f"-DCCL_TILE_ROWS={r}", f"-DCCL_SHAPE_NS=r{r}"]) for r in b.TILE_ROWS
] + [("ccl_api.cpp", [])])
def test_no_warnings(source, defines):
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    r = subprocess.run([hipcc, "-fsyntax-only", "-O3", "-std=c++17", "-Wall", "-Werror",
                        "-Wno-unused-command-line-argument", f"-I{b.INCLUDE}", f"-I{b.CSRC}",
                        *defines, "-x", "hip", f"--offload-arch={b.ARCH}",
                        os.path.join(b.CSRC, source)], capture_output=True, text=True)
    assert r.returncode == 0 and "warning" not in r.stderr, r.stderr[-3000:]
