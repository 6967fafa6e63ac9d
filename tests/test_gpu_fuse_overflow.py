"""Fusion terms past float32's range.  With a noise coefficient far below any
sensor's, w * rz of a valid point can overflow although its height and its noise
are ordinary numbers.  Such a term enters the fixed-point sum as 2^128 with its
sign, so that the cell's height stays finite, and is the same for any shape of
the launch.  Terms in range are compared in the same cells."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_util import load_state, random_state
from test_gpu_fuse_sums import _integers, _shifts, dev  # noqa: F401

pytestmark = pytest.mark.gpu

F32 = np.float32


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("n", [1, 40, 70000])
def test_overflowing_terms(dev, n, batched):  # noqa: F811
    from paper_2204_12876_amd import BatchEntry, ElevationMap, PipelineBatch, _emx
    print("[case] overflowing terms", n, "batched" if batched else "plain", flush=True)
    rng = np.random.default_rng(n)
    r = 0.5
    params = dict(nx=64, ny=64, resolution=r, noise_alpha=1e-40, gate_k=1e20, min_range=18.0)
    p = O.Params.from_dict(params)
    xs, ys = (rng.uniform(-15.0, 15.0, n).astype(F32) for _ in range(2))
    zs = (-20.0 - rng.uniform(0.0, 20.0, n)).astype(F32)
    xs[0], ys[0], zs[0] = 1.0, -1.0, -20.0       # overflows
    pose = np.eye(3, 4)
    pose[2, 3] = 4.0
    st = random_state(p, rng, valid_frac=0.7)
    st.v[:] = 1e3
    m = ElevationMap(params, 0.0, 0.0, 0, device=dev)
    load_state(m, st)
    pts = tuple(torch.from_numpy(q).to(dev) for q in (xs, ys, zs))
    if batched:
        pb = PipelineBatch(device=dev)
        pb.run([BatchEntry(m, *pts, pose, 900, stages=_emx.STAGE_FUSE)])
    else:
        m.fuse_points(*pts, pose, 900)
    torch.cuda.synchronize()
    d = O.point_decisions(p, st, xs, ys, zs, pose)
    a = np.nonzero(d["accept"])[0]
    assert a.size > 0.8 * n
    with np.errstate(all="ignore"):
        w = F32(1) / d["sp2"][a]
        u = w * zs[a]
    over = np.isinf(u)
    assert over.any() and (n == 1 or not over.all())
    u64 = np.where(over, -2.0 ** 128, u.astype(np.float64))
    Sw, Su = _shifts(p, d["R"], n)
    h, v = st.h.reshape(-1).copy(), st.v.reshape(-1).copy()
    cells = {}
    for c, iw, iu in zip(d["cell"][a].tolist(), _integers(w, Sw), _integers(u64, Su)):
        s = cells.setdefault(c, [0, 0, 0, 0])
        for k, x in enumerate((max(iw, 1) >> 32, max(iw, 1) & 0xFFFFFFFF, iu >> 32, iu & 0xFFFFFFFF)):
            s[k] += x
    for c, (wh, wl, zh, zl) in cells.items():
        sw = float(np.ldexp(float(wh) * 4294967296.0 + float(wl), -Sw))
        sz = float(np.ldexp(float(zh) * 4294967296.0 + float(zl), -Su))
        with np.errstate(all="ignore"):
            acc_w, acc_z = F32(sw), F32(sz + 4.0 * sw)
            v1 = F32(1) / (F32(1) / v[c] + acc_w)
            h[c], v[c] = (h[c] / v[c] + acc_z) * v1, v1
    g = m.state_numpy()
    assert np.array_equal(g["v"].reshape(-1).view(np.uint32), v.view(np.uint32))
    assert np.array_equal(g["h"].reshape(-1).view(np.uint32), h.view(np.uint32))
    m.close()
    if batched:
        pb.close()
