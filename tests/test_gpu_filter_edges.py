"""Inpainting across tile seams and the median at a wave's edges, against the
oracle bit for bit: regions that wind through many tiles (serpentine, comb,
spiral), that touch a seam by one cell, on maps of one tile, of exactly whole
tiles and one cell more, on a turned ring; median grids as narrow as a window
and around the columns that a wave gives."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_util import load_state, random_state

pytestmark = pytest.mark.gpu

F32 = np.float32


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_12876_amd import _emx
    _emx.lib()
    return torch.device("cuda:0")


def _bits(a):
    return np.ascontiguousarray(a, F32).view(np.uint32)


def _mask(kind, ny, nx, rng):
    """1 where the cell holds an estimate."""
    ok = np.ones((ny, nx), np.uint8)
    if kind == "serpentine":                # one hole region through every row pair
        ok[::2] = 0
        for k in range(1, ny, 2):
            ok[k, (nx - 1) if (k // 2) % 2 == 0 else 0] = 0
    elif kind == "comb":
        ok[0] = 0
        ok[:, ::2] = 0
    elif kind == "checker":
        ok[(np.add.outer(np.arange(ny), np.arange(nx)) % 2) == 0] = 0
    elif kind == "empty":
        ok[:] = 0
    elif kind == "one":
        ok[:] = 0
        ok[ny // 2, nx // 2] = 1
    elif kind == "spiral":
        y0, y1, x0, x1 = 0, ny - 1, 0, nx - 1
        while y0 <= y1 and x0 <= x1:
            ok[y0, x0:x1 + 1] = 0
            ok[y0:y1 + 1, x1] = 0
            ok[y1, x0:x1 + 1] = 0
            if y0 + 2 <= y1:
                ok[y0 + 2:y1 + 1, x0] = 0
            if y0 + 2 <= y1 and x0 + 1 <= x1:
                ok[y0 + 2, x0:x0 + 2] = 0
            y0, y1, x0, x1 = y0 + 2, y1 - 2, x0 + 2, x1 - 2
    elif kind == "random":
        ok = (rng.random((ny, nx)) < 0.55).astype(np.uint8)
    return ok


@pytest.mark.parametrize("kind", ["serpentine", "comb", "checker", "empty", "one", "spiral",
                                  "random", "full"])
@pytest.mark.parametrize("nx,ny", [(3, 3), (32, 32), (33, 32), (32, 33), (31, 97), (64, 65),
                                   (190, 130)])
def test_inpaint_regions(dev, kind, nx, ny):
    from paper_2204_12876_amd import ElevationMap
    print("[case] inpaint", kind, nx, ny, flush=True)
    rng = np.random.default_rng(nx * 7 + ny)
    params = dict(nx=nx, ny=ny, resolution=0.05)
    p = O.Params.from_dict(params)
    m = ElevationMap(params, 0.0, 0.0, 0, device=dev)
    m.move_map(0.05 * 2 + 0.01, -0.05 + 0.01)      # a turned ring
    st = random_state(p, rng)
    st.valid[:] = _mask(kind, ny, nx, rng)
    load_state(m, st)
    exp = O.inpaint_min(st.h, st.valid)
    for _ in range(2):                             # the second on used scratch
        g = m.inpaint_min().cpu().numpy()
        assert np.array_equal(np.isnan(g), np.isnan(exp))
        assert np.array_equal(_bits(g)[~np.isnan(g)], _bits(exp)[~np.isnan(exp)])
    m.close()


@pytest.mark.parametrize("k", [3, 5])
@pytest.mark.parametrize("nx", [3, 4, 59, 60, 61, 62, 63, 64, 65, 121, 125])
@pytest.mark.parametrize("ny", [3, 15, 16, 17])
def test_median_edges(dev, k, nx, ny):
    from paper_2204_12876_amd import smooth
    rng = np.random.default_rng(100 * nx + ny)
    for nans, few in ((0.0, True), (0.01, False), (0.0, False)):
        x = rng.normal(0.0, 1.0, (ny, nx)).astype(F32)
        if few:                                    # many equal values
            x = np.round(x * 2).astype(F32) + F32(10)
        x[rng.random(x.shape) < nans] = np.nan
        x[rng.integers(0, ny), rng.integers(0, nx)] = np.inf
        x[rng.integers(0, ny), rng.integers(0, nx)] = -np.inf
        g = smooth(torch.from_numpy(x).to(dev), "median", k).cpu().numpy()
        exp = O.smooth_median(x, k)
        assert np.array_equal(np.isnan(g), np.isnan(exp)), (k, nx, ny)
        assert np.array_equal(_bits(g)[~np.isnan(g)], _bits(exp)[~np.isnan(exp)]), (k, nx, ny)
