"""Levels past the third: built from the level below and detected by upper
regions (about 32 pixels of level 3 a side), three levels a pass.  Cells that
divide no power of two move the regions off the 16-pixel grid; frame sizes sit
around the regions' edges.  Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2003_13493_amd import fastgrid, synth  # noqa: E402

# width, height, levels, cell
CASES = [(256, 256, 4, 32), (257, 255, 4, 8), (513, 300, 5, 16), (511, 263, 5, 48), (700, 290, 4, 24),
         (600, 310, 4, 72), (560, 280, 4, 136), (1000, 520, 4, 248), (1030, 530, 6, 32), (777, 1025, 7, 64),
         (1100, 1030, 8, 128), (1040, 600, 7, 192), (520, 2100, 6, 256)]


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = fastgrid.Context(0, tuned=False)
    yield c
    torch.cuda.synchronize()
    c.close()


def frame_of(i):
    w, h, levels, cell = CASES[i]
    img = synth.frame(w, h, seed=700 + i, nshapes=200, sigma=5.0, pad_garbage=True)
    pyr, grid = fastgrid.Pyramid(w, h, levels), fastgrid.Grid(w, h, cell)
    pyr.upload(img)
    return img, pyr, grid


def check(i, img, pyr, grid, tag):
    w, h, levels, cell = CASES[i]
    want, planes = oracle.detect_grid(img, w, levels, 12, 9, cell)
    for k in range(1, levels):
        assert np.array_equal(pyr.level(k), planes[k][0][:, :planes[k][1]]), f"{tag} {CASES[i]} level {k}"
    assert np.array_equal(grid.fetch(), want), f"{tag} {CASES[i]} slots"
    assert (want["level"][want["score"] > 0] >= 3).any()


@pytest.mark.parametrize("i", range(len(CASES)), ids=["%dx%d_L%d_c%d" % c for c in CASES])
def test_one_frame(ctx, i):
    print(f"case upper {CASES[i]}", flush=True)
    img, pyr, grid = frame_of(i)
    ctx.detect(pyr, 12, 9, CASES[i][3], grid)
    torch.cuda.synchronize()
    check(i, img, pyr, grid, "plain")
    w, h, levels, _ = CASES[i]
    maps = fastgrid.ScoreMaps(w, h, levels)
    ctx.score_maps(pyr, 12, 9, maps)
    torch.cuda.synchronize()
    _, planes = oracle.detect_grid(img, w, levels, 12, 9, CASES[i][3])
    for k in range(levels):
        a, wk = planes[k]
        assert np.array_equal(maps.level(k), oracle.score_map(a, wk, 12, 9)), f"maps {CASES[i]} level {k}"


@pytest.mark.parametrize("shape", [(0, 256, 3), (256, 128, 4), (64, 512, 2)])
def test_batch_of_all(ctx, shape):
    print(f"case upper batch {shape}", flush=True)
    ctx.set_launch(*shape)
    frames = [frame_of(i) for i in range(len(CASES))]
    jobs = ctx.make_jobs((p, 12, 9, CASES[i][3], g) for i, (_, p, g) in enumerate(frames))
    assert ctx.wait(ctx.submit(jobs))
    for i, (img, p, g) in enumerate(frames):
        check(i, img, p, g, f"batch {shape}")
        g.tensor.zero_()
    ctx.submit_static(jobs, ticket=False)
    torch.cuda.synchronize()
    ctx.reset_launch()
    for i, (img, p, g) in enumerate(frames):
        check(i, img, p, g, f"static {shape}")
