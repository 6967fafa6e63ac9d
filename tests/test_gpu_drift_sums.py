"""The drift compensation's mean, bit for bit: the float64 sums are formed here in
the same fixed order (a thread's points in index order, a butterfly over the wave,
the waves in order; then the chunks' partials strided over one workgroup and
combined the same way), at frame sizes around a chunk, around one workgroup's eight
partials a thread, and where the shift takes fewer workgroups.  Every valid height
of maps with more and with fewer cells than threads is shifted once."""
import numpy as np
import pytest
import torch

from parity_util import load_state, random_state
import oracle as O

pytestmark = pytest.mark.gpu

F32 = np.float32
CHUNK = 1024


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_12876_amd import _emx
    _emx.lib()
    return torch.device("cuda:0")


def _workgroup(s):
    """[..., 256] partial sums of a workgroup's threads to their total."""
    s = s.reshape(s.shape[:-1] + (4, 64))
    lane = np.arange(64)
    for o in (32, 16, 8, 4, 2, 1):
        s = s + s[..., lane ^ o]
    w = s[..., 0]
    return ((w[..., 0] + w[..., 1]) + w[..., 2]) + w[..., 3]


def _fixed_sum(e):
    chunks = -(-e.size // CHUNK)
    a = np.zeros(chunks * CHUNK)
    a[:e.size] = e
    a = a.reshape(chunks, 4, 256)
    part = _workgroup(((a[:, 0] + a[:, 1]) + a[:, 2]) + a[:, 3])
    rows = np.zeros((-(-chunks // 256)) * 256)
    rows[:chunks] = part
    s = np.zeros(256)
    for row in rows.reshape(-1, 256):
        s = s + row
    return float(_workgroup(s))


@pytest.mark.parametrize("n,side", [(1, 40), (1023, 40), (1025, 40), (2047 * CHUNK, 40),
                                    (2048 * CHUNK + 1, 40), (2305 * CHUNK, 40), (30000, 900),
                                    (2100 * CHUNK + 7, 900)])
def test_mean_bitwise(dev, n, side):
    from paper_2204_12876_amd import ElevationMap
    print("[case] drift sums", n, side, flush=True)
    rng = np.random.default_rng(n + side)
    r = 0.1
    params = dict(nx=side, ny=side - 3, resolution=r, min_range=0.01)
    p = O.Params.from_dict(params)
    st = random_state(p, rng, valid_frac=0.95)
    m = ElevationMap(params, device=dev)
    load_state(m, st)
    half = 0.5 * r * (side - 4)
    xs, ys = (rng.uniform(-half, half, n).astype(F32) for _ in range(2))
    zs = rng.uniform(-2.0, -1.0, n).astype(F32)
    pose = np.eye(3, 4)
    pose[2, 3] = 1.25
    mean, count = m.compensate_drift(*(torch.from_numpy(a).to(dev) for a in (xs, ys, zs)), pose, 10,
                                     -0.5)
    torch.cuda.synchronize()
    d = O.point_decisions(p, st, xs, ys, zs, pose)
    c = d["cell"]
    use = (c >= 0) & (st.valid.reshape(-1)[c] != 0) & (st.trav.reshape(-1)[c] > F32(-0.5))
    e = np.where(use, d["zm"].astype(np.float64) - st.h.reshape(-1)[c].astype(np.float64), 0.0)
    want = _fixed_sum(e) / max(1, int(use.sum()))
    assert int(count) == int(use.sum())
    assert float(mean) == want
    g = m.state_numpy()
    h = np.where(st.valid != 0, st.h + F32(want), st.h) if use.any() else st.h
    assert np.array_equal(g["h"].view(np.uint32), h.astype(F32).view(np.uint32))
    m.close()
