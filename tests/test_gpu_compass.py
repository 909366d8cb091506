"""The compass filter's byte thresholds at every pair of values: 8 x 8 blocks of
one value with another at their centre, all 65,536 pairs in one frame, at
thresholds of both parities and at the ends of their range, and for arc lengths
that ask for 1 to 4 compass points.  A point lost at its boundary would be a
score missing from the map."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2003_13493_amd import fastgrid  # noqa: E402


def pairs_frame():
    """2048 x 2048: block (i, j) is i all over, j at its centre."""
    img = np.repeat(np.repeat(np.arange(256, dtype=np.uint8)[:, None], 8, 0), 2048, 1)
    img = np.ascontiguousarray(img)
    img[4::8, 4::8] = np.arange(256, dtype=np.uint8)[None, :]
    return img


@pytest.mark.parametrize("t,n", [(0, 9), (1, 12), (2, 16), (9, 5), (10, 9), (127, 12), (128, 9), (254, 9), (255, 4)])
def test_every_pair_of_values(t, n):
    print(f"case compass pairs t={t} n={n}", flush=True)
    img = pairs_frame()
    ctx = fastgrid.Context(0, tuned=False)
    pyr, maps = fastgrid.Pyramid(2048, 2048, 1), fastgrid.ScoreMaps(2048, 2048, 1)
    pyr.upload(img)
    ctx.score_maps(pyr, t, n, maps)
    torch.cuda.synchronize()
    ctx.close()
    assert np.array_equal(maps.level(0), oracle.score_map(img, 2048, t, n))
