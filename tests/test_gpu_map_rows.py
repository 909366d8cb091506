"""Score maps written eight scores at a time: rows at any even address, widths
around multiples of 8 and of the regions, odd pitches; what lies past a row's
width stays as it was."""
import ctypes

import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2003_13493_amd import fastgrid, synth  # noqa: E402


@pytest.mark.parametrize("w,h,levels,pad", [(64, 64, 1, 0), (71, 40, 1, 1), (73, 65, 3, 3), (129, 130, 4, 0), (640, 33, 3, 5),
                                            (33, 300, 2, 2), (321, 241, 5, 1)])
def test_rows(w, h, levels, pad):
    print(f"case map rows {w}x{h} L={levels} pad={pad}", flush=True)
    ctx = fastgrid.Context(0, tuned=False)
    img = synth.frame(w, h, seed=w + h, nshapes=80, sigma=6.0, pad_garbage=True)
    pyr = fastgrid.Pyramid(w, h, levels)
    pyr.upload(img)
    dev = [torch.full((1 + (h >> k) * ((w >> k) + pad),), 0x5A5A, dtype=torch.int16, device="cuda")
           for k in range(levels)]
    ptrs = (ctypes.c_void_p * levels)(*[t.data_ptr() + 2 for t in dev])
    pitches = (ctypes.c_int32 * levels)(*[(w >> k) + pad for k in range(levels)])
    fastgrid.fast_score_maps(ctx.handle, pyr.planes, levels, 10, 9, fastgrid.FAST_SCORE_SADB, ptrs, pitches)
    torch.cuda.synchronize()
    ctx.close()
    for k, (plane, wk) in enumerate(oracle.pyr_build(img, w, levels)):
        got = dev[k].cpu().numpy().view(np.uint16)
        assert got[0] == 0x5A5A
        got = got[1:].reshape(h >> k, -1)
        assert np.array_equal(got[:, :wk], oracle.score_map(plane, wk, 10, 9)), f"level {k}"
        assert (got[:, wk:] == 0x5A5A).all(), f"level {k}: written past the width"
