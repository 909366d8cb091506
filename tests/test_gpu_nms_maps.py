"""The standalone NMS on maps of its own: rows at any even address and of any
length (shorter than a load, one element past it), sparse and full maps, many
equal scores, sub-tiles at a map's edges, several sub-tiles a region.  Against
a restatement that compares every pixel with its window by shifting the map."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2003_13493_amd import fastgrid  # noqa: E402

# width, height, levels, cell, radius, pitch padding (elements), share of pixels that score, region
CASES = [(3, 40, 1, 16, 4, 0, 1.0, 0), (7, 9, 1, 16, 1, 1, 0.5, 0), (8, 64, 2, 2, 2, 0, 0.3, 0),
         (9, 65, 1, 32, 3, 2, 1.0, 0), (63, 66, 3, 4, 1, 1, 0.02, 0), (65, 129, 4, 8, 4, 3, 0.1, 64),
         (129, 131, 3, 16, 2, 0, 1.0, 128), (200, 131, 5, 16, 3, 1, 0.02, 256), (333, 190, 3, 24, 1, 5, 0.3, 0),
         (270, 260, 8, 128, 4, 0, 0.05, 0), (641, 77, 2, 40, 2, 0, 0.02, 32), (130, 300, 7, 64, 1, 1, 1.0, 256)]


def maps_of(i):
    w, h, levels, _, _, pad, share, _ = CASES[i]
    rng = np.random.default_rng(40 + i)
    out = []
    for k in range(levels):
        m = rng.integers(1, 9, size=(h >> k, w >> k)) * 500   # few values: ties everywhere
        m[rng.random(m.shape) >= share] = 0
        buf = rng.integers(1, 4000, size=(h >> k, (w >> k) + pad)).astype(np.uint16)   # padding scores if read
        buf[:, :w >> k] = m
        out.append(buf)
    return out


def survivors(m, r):
    """Where m > 0 is above every earlier pixel of its window and not below any later one."""
    h, w = m.shape
    p = np.zeros((h + 2 * r, w + 2 * r), dtype=np.int64)
    p[r:r + h, r:r + w] = m
    keep = m > 0
    for dy in range(-r, r + 1):
        for dx in range(-r, r + 1):
            other = p[r + dy:r + dy + h, r + dx:r + dx + w]
            if (dy, dx) < (0, 0):
                keep &= m > other
            elif (dy, dx) > (0, 0):
                keep &= m >= other
    return keep


def expected(maps, w, h, cell, r):
    gw, gh = -(-w // cell), -(-h // cell)
    best = {}
    for k, buf in enumerate(maps):
        m = buf[:, :w >> k].astype(np.int64)
        for y, x in zip(*np.nonzero(survivors(m, r))):
            c = ((y << k) // cell) * gw + (x << k) // cell
            key = (-m[y, x], k, y, x)
            if c not in best or key < best[c]:
                best[c] = key
    out = np.zeros(gw * gh, dtype=fastgrid.FEATURE_DTYPE)
    out["x"], out["y"], out["level"] = 0xFFFF, 0xFFFF, 0xFF
    for c, (s, k, y, x) in best.items():
        out[c] = (x, y, -s, k, 0)
    return out


@pytest.mark.parametrize("i", range(len(CASES)), ids=["%dx%d_L%d_c%d_r%d" % c[:5] for c in CASES])
def test_maps(i):
    w, h, levels, cell, radius, pad, _, region = CASES[i]
    print(f"case nms maps {CASES[i]}", flush=True)
    ctx = fastgrid.Context(0, tuned=False)
    ctx.set_launch(region, 256, 3)
    maps = maps_of(i)
    # each map two bytes past a 4-byte boundary, so its rows take both parities
    dev = [torch.from_numpy(np.concatenate([[7], m.ravel()]).astype(np.uint16).view(np.int16)).cuda() for m in maps]
    ptrs = (ctypes.c_void_p * levels)(*[t.data_ptr() + 2 for t in dev])
    pitches = (ctypes.c_int32 * levels)(*[m.shape[1] for m in maps])
    grid = fastgrid.Grid(w, h, cell)
    grid.tensor.fill_(0x77)
    fastgrid.fast_nms_grid(ctx.handle, ptrs, pitches, w, h, levels, radius, cell, grid.ptr)
    torch.cuda.synchronize()
    got, want = grid.fetch(), expected(maps, w, h, cell, radius)
    ctx.close()
    assert np.array_equal(got, want), f"{CASES[i]}: cells {np.nonzero(got != want)[0][:5]}"
