"""Which kernel takes a batch's regions: the rule's edges, evaluated by the
header that the runtime uses, on the host."""
import subprocess

import pytest

from paper_2003_13493_amd import build

GENERIC, GENERIC_WIDE, ANY, WHOLE = range(4)

# total, whole, single sub-tiles, threads, workgroups a CU, kernel
CASES = [(96, 77, 1, 256, 3, WHOLE), (96, 24, 1, 256, 3, WHOLE), (96, 23, 1, 256, 3, ANY), (97, 24, 1, 256, 3, ANY),
         (96, 0, 1, 256, 3, ANY), (1, 0, 1, 256, 1, ANY), (1, 1, 1, 256, 16, WHOLE),
         (96, 77, 1, 256, 4, WHOLE), (96, 77, 1, 320, 3, ANY), (96, 77, 1, 384, 2, ANY), (96, 77, 1, 448, 2, ANY),
         (96, 77, 1, 512, 2, ANY), (96, 77, 1, 512, 1, WHOLE), (96, 77, 1, 320, 1, WHOLE), (96, 0, 1, 512, 1, ANY),
         (96, 77, 0, 320, 2, GENERIC_WIDE), (96, 0, 0, 512, 16, GENERIC_WIDE), (96, 77, 0, 512, 1, GENERIC),
         (96, 77, 0, 256, 3, GENERIC), (96, 77, 1, 192, 3, GENERIC), (96, 0, 1, 64, 6, GENERIC),
         (1 << 30, 1 << 29, 1, 256, 3, WHOLE), (1 << 30, 1 << 27, 1, 256, 3, ANY)]

MAIN = """
#include <cstdio>
#include "fg_internal.h"
int main() {
    int total, whole, single, block, per_cu;
    while (std::scanf("%d %d %d %d %d", &total, &whole, &single, &block, &per_cu) == 5) {
        const fg_launch L{FG_SUB, 0, block, per_cu, 256};
        std::printf("%d\\n", (int)fg_choose_batch(fg_batch_work{total, whole, single != 0}, L));
    }
}
"""


@pytest.fixture(scope="module")
def chosen(tmp_path_factory):
    d = tmp_path_factory.mktemp("choice")
    (d / "main.hip").write_text(MAIN)
    subprocess.run([build._hipcc(), "--cuda-host-only", "-std=c++17", "-I", build.INCLUDE, "-I", build.CSRC,
                    "-o", str(d / "main"), str(d / "main.hip")], check=True)
    lines = "\n".join(" ".join(map(str, c[:5])) for c in CASES)
    out = subprocess.run([str(d / "main")], input=lines, capture_output=True, text=True, check=True).stdout
    return [int(x) for x in out.split()]


@pytest.mark.parametrize("i", range(len(CASES)))
def test_choice(chosen, i):
    assert chosen[i] == CASES[i][5], CASES[i]
