"""fast_pyr_build: up to five levels from one load.  Sizes around the 256 x 32
pixels a wave takes, odd at several levels, pitches past the width, all level
counts; bytes past a level's width stay as they were."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2003_13493_amd import fastgrid, synth  # noqa: E402

CASES = [(2, 2, 2), (17, 9, 2), (31, 40, 3), (255, 31, 4), (256, 32, 5), (257, 33, 6), (300, 511, 6), (1283, 719, 4),
         (520, 300, 7), (1027, 515, 8), (4096, 67, 6), (129, 1000, 7)]


@pytest.mark.parametrize("w,h,levels", CASES)
def test_pyramid(w, h, levels):
    print(f"case pyramid {w}x{h} L={levels}", flush=True)
    ctx = fastgrid.Context(0, tuned=False)
    img = synth.frame(w, h, seed=w * 7 + h, nshapes=60, sigma=9.0, pad_garbage=True)
    pyr = fastgrid.Pyramid(w, h, levels)
    pyr.upload(img)
    for t in pyr.tensors[1:]:
        t.fill_(0xA5)
    ctx.pyr_build(pyr)
    torch.cuda.synchronize()
    ctx.close()
    for k, (plane, wk) in enumerate(oracle.pyr_build(img, w, levels)):
        if k:
            got = pyr.tensors[k].cpu().numpy()
            assert np.array_equal(got[:, :wk], plane[:, :wk]), f"level {k}"
            assert (got[:, wk:] == 0xA5).all(), f"level {k}: padding written"
