"""Batches on both sides of the rule that picks their kernel, by the share of
their regions that are whole (64 x 64 pixels of three levels and more): none,
just under a quarter, a quarter, most.  With one workgroup a CU each takes several
regions, so that regions of several shapes and level counts follow each other.
Bit for bit against the oracle."""
import numpy as np
import pytest

import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2003_13493_amd import fastgrid, synth  # noqa: E402

# width, height, levels, cell, times
EDGES = [(65, 64, 1, 32, 2), (63, 129, 2, 16, 2), (257, 70, 1, 48, 1), (200, 190, 2, 24, 2), (191, 127, 3, 48, 1)]
MIXES = {
    "none": [(752, 480, 1, 32, 3), (640, 300, 2, 32, 3), (500, 410, 3, 48, 3), (333, 217, 3, 24, 4), (300, 64, 1, 16, 3)]
    + EDGES,
    "under": [(192, 128, 3, 32, 1), (192, 192, 1, 32, 1), (256, 64, 2, 16, 1), (384, 64, 1, 64, 1)],     # 6 whole of 25
    "quarter": [(192, 128, 3, 32, 1), (192, 192, 1, 32, 1), (256, 64, 2, 16, 1), (320, 64, 1, 64, 1)],   # 6 of 24
    "most": [(752, 480, 3, 32, 3), (640, 300, 1, 32, 2), (333, 217, 4, 16, 3), (320, 320, 5, 64, 2)] + EDGES,
}


@pytest.fixture(scope="module")
def ctx():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    c = fastgrid.Context(0, tuned=False)
    yield c
    torch.cuda.synchronize()
    c.close()


def frames_of(mix):
    out, i = [], 0
    for w, h, levels, cell, times in MIXES[mix]:
        for _ in range(times):
            i += 1
            img = synth.frame(w, h, seed=2000 + 31 * i + w, nshapes=60, sigma=5.0, pad_garbage=True)
            pyr, grid = fastgrid.Pyramid(w, h, levels), fastgrid.Grid(w, h, cell)
            pyr.upload(img)
            want, planes = oracle.detect_grid(img, w, levels, 12, 9, cell)
            out.append((pyr, grid, cell, want, planes))
    order = np.random.default_rng(len(out)).permutation(len(out))
    return [out[k] for k in order]


@pytest.mark.parametrize("shape", [(64, 256, 3), (64, 256, 1), (32, 256, 2), (64, 320, 1), (64, 384, 2), (64, 512, 2),
                                   (128, 256, 1), (128, 512, 2), (256, 320, 2), (256, 128, 4)], ids=lambda s: "%d_%d_%d" % s)
@pytest.mark.parametrize("mix", list(MIXES))
def test_batch(ctx, mix, shape):
    print(f"case batch regions {mix} {shape}", flush=True)
    frames = frames_of(mix)
    jobs = ctx.make_jobs((p, 12, 9, cell, g) for p, g, cell, _, _ in frames)
    ctx.set_launch(*shape)
    try:
        for r in range(2):
            for _, g, _, _, _ in frames:
                g.tensor.fill_(0x5A)
            assert ctx.wait(ctx.submit(jobs), 60_000)
            for i, (p, g, _, want, planes) in enumerate(frames):
                tag = f"{mix} {shape} frame {i} ({p.width}x{p.height} L={p.levels})"
                assert np.array_equal(g.fetch(), want), tag
                for k in range(1, p.levels):
                    assert np.array_equal(p.level(k), planes[k][0][:, :planes[k][1]]), f"{tag} level {k}"
    finally:
        ctx.reset_launch()


@pytest.mark.parametrize("graph", [False, True], ids=["direct", "graph"])
def test_plan_under_other_shapes(ctx, graph):
    """A resident batch keeps its regions; the workgroups that a launch uses, and
    with them the kernel, follow the context's shape of the moment (a captured
    launch keeps its own)."""
    print(f"case batch regions plan graph={graph}", flush=True)
    frames = frames_of("most")
    jobs = ctx.make_jobs((p, 12, 9, cell, g) for p, g, cell, _, _ in frames)
    pid = ctx.plan_create(jobs, graph=graph)
    try:
        for shape in [(0, 256, 3), (0, 512, 2), (0, 128, 4), (0, 512, 1), (0, 320, 2), (0, 256, 1)]:
            ctx.set_launch(*shape)
            for _, g, _, _, _ in frames:
                g.tensor.fill_(0x5A)
            ctx.plan_launch(pid, ticket=False)
            torch.cuda.synchronize()
            for i, (_, g, _, want, _) in enumerate(frames):
                assert np.array_equal(g.fetch(), want), f"{shape} frame {i}"
    finally:
        ctx.plan_destroy(pid)
        ctx.reset_launch()
