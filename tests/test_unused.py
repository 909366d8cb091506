"""No function of the library's sources is left unused."""
import os
import subprocess

import pytest

from paper_2003_13493_amd import build


@pytest.mark.parametrize("name", build.HIP_SOURCES)
def test_no_unused_function(name):
    cmd = [build._hipcc(), "--offload-arch=gfx950", "-std=c++17", "-fsyntax-only", "-Wall", "-Wno-bitwise-instead-of-logical",
           "-Werror=unused-function", "-I", build.INCLUDE, "-I", build.CSRC, os.path.join(build.CSRC, name)]
    run = subprocess.run(cmd, capture_output=True, text=True)
    assert run.returncode == 0, run.stderr
