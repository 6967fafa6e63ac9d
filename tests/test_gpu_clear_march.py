"""The clearing march's pruning by blocks, superblocks and groups of samples,
against the oracle, which tests every sample: marks, state and upper bound bit
for bit.  Step lengths from a tenth of a cell (groups of 32 samples) to many
cells (groups of one, whose ends lie more than a block apart), sides on and
off the block sizes, a turned ring, sensors outside the map, axis-parallel rays
and rays along cell edges, points that cast no ray, and enough surviving groups
to fill a workgroup's list several times."""
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


def _points(rng, n, reach, flat):
    """Sensor-frame end points around the sensor, below it; some special ones."""
    ang = rng.uniform(0, 2 * np.pi, n)
    rad = rng.uniform(0.1, 1.0, n) * reach
    xs, ys = rad * np.cos(ang), rad * np.sin(ang)
    zs = -rng.uniform(0.0, 1.0, n) * (0.1 if flat else 1.5)
    k = np.arange(n)
    xs[k % 17 == 3] = 0.0                       # axis-parallel
    ys[k % 17 == 5] = 0.0
    ys[k % 29 == 7] = 1e-6                      # nearly so
    xs[k % 31 == 9] = np.nan                    # no ray
    zs[k % 37 == 11] = np.inf
    xs[k % 41 == 13] = 1e18                     # too long a ray
    return tuple(a.astype(F32) for a in (xs, ys, zs))


CASES = [
    # nx, ny, step / r, sensor (cells from the map's corner), reach (cells), n, valid, flat
    (32, 32, 1.0, (16.0, 16.0), 30, 256, 0.9, False),
    (31, 33, 1.0, (0.0, 33.0), 60, 257, 0.9, False),
    (97, 130, 0.11, (40.3, 70.7), 90, 255, 0.3, False),
    (97, 130, 3.3, (40.3, 70.7), 200, 1500, 0.9, False),
    (160, 64, 9.0, (80.0, 32.0), 300, 1500, 0.9, False),
    (160, 64, 40.0, (80.5, 31.5), 400, 700, 0.9, False),
    (200, 180, 1.0, (-25.0, 90.0), 260, 2000, 0.6, False),
    (200, 180, 1.0, (300.0, -40.0), 400, 2000, 0.6, True),
    (333, 290, 1.0, (150.0, 140.0), 330, 4000, 0.02, False),   # few cells to remove
    (500, 500, 1.0, (250.0, 250.0), 245, 1024, 0.8, True),     # lists fill up
    (3, 3, 1.0, (1.5, 1.5), 5, 1, 1.0, False),
    (200, 200, 1.0, (100.0, 100.0), 98, (3 << 14) + 1, 0.8, True),  # workgroups of 64 rays
    (200, 200, 1.0, (100.0, 100.0), 98, (1 << 17) + 1, 0.8, True),  # workgroups of 128 rays
]


@pytest.mark.parametrize("ub", [0, 1])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_march_equals_every_sample(dev, case, ub):
    from paper_2204_12876_amd import ElevationMap
    nx, ny, ratio, sensor, reach, n, valid, flat = CASES[case]
    print("[case] clear march", CASES[case], "ub", ub, flush=True)
    rng = np.random.default_rng(900 + 10 * case + ub)
    r = 0.05
    params = dict(nx=nx, ny=ny, resolution=r, noise_alpha=0.01, gate_k=2.0, min_range=0.05,
                  ray_step=ratio * r, clear_normal_alpha=0.1, clear_min_age_ms=200,
                  upper_bound=ub)
    p = O.Params.from_dict(params)
    m = ElevationMap(params, 0.0, 0.0, 0, device=dev)
    # a move turns the ring: layers and records differ in order from here on
    cx, cy = 5 * r + 0.01, -3 * r + 0.01
    m.move_map(cx, cy)
    st = random_state(p, rng, valid_frac=valid)
    st.cgx, st.cgy, _ = m.info()
    k = rng.integers(0, nx * ny, 5)
    st.h.reshape(-1)[k] = np.nan
    st.nrm.reshape(3, -1)[:, rng.integers(0, nx * ny, 5)] = np.nan
    load_state(m, st)
    ox, oy = (st.cgx - nx // 2) * r, (st.cgy - ny // 2) * r
    pose = np.zeros((3, 4))
    pose[:, :3] = np.eye(3)
    pose[:, 3] = (ox + sensor[0] * r, oy + sensor[1] * r, 0.3 if flat else 1.0)
    bound = np.full((ny, nx), np.inf, F32)
    xs, ys, zs = _points(rng, n, reach * r, flat)
    pts = tuple(torch.from_numpy(a).to(dev) for a in (xs, ys, zs))
    out = torch.full((nx * ny,), 9, dtype=torch.uint8, device=dev)
    for t_ms in (700, 800):     # the second call on the cleared map and lowered bound
        m.clear_visibility(*pts, pose, t_ms, out_cleared=out)
        torch.cuda.synchronize()
        marks = O.clear_visibility(p, st, xs, ys, zs, pose, t_ms)
        got = out.cpu().numpy().reshape(ny, nx)
        assert np.array_equal(got, marks.astype(np.uint8)), np.argwhere(got != marks)[:8]
        if ub:
            bound = O.upper_bound(p, st, bound, xs, ys, zs, pose)
            g = m.upper_bound().cpu().numpy()
            assert np.array_equal(g.view(np.uint32), bound.view(np.uint32))
        st = O.apply_clear(p, st, marks)
        g = m.state_numpy()
        for name in ("h", "v", "valid", "t_upd"):
            a, b = g[name], getattr(st, name)
            assert np.array_equal(a.view(np.uint8), b.view(np.uint8)), name
        print("[case]  ", int(marks.sum()), "cells removed", flush=True)
    m.close()
