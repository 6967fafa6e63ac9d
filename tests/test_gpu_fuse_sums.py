"""The fusion's fixed-point sums, bit for bit.  The ABI fixes every step of a
fused cell: the points' float32 terms, their integers at the call's shifts, the
integer sums, and the float32 update from them.  Here the sums are formed in
Python integers from numpy float32 terms and the cells are compared as bits, at
frame sizes around the chunks of pass 1 (256 points in small frames, 1024 in
larger ones, and the batched call's, also with one workgroup for all chunks),
with one cell taking a whole chunk, with
more distinct cells than a chunk's table has slots, over the range of terms
(low words, rounding, negative heights, a term below half a unit), and after a
move in the same call."""
import math

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


def _exp_above(x):
    return math.frexp(x)[1]


def _shifts(p, R, n):
    c = O.f32_constants(p)
    rmin2, alpha = c["rmin2"], c["alpha"]
    wmax = float(F32(1) / F32(alpha * rmin2)) * (1 + 2.0 ** -10)
    l1 = sum(abs(float(v)) for v in R[2])
    zmax = (l1 if l1 > 0 else 1.0) / (float(alpha) * math.sqrt(float(rmin2))) * (1 + 2.0 ** -10)
    ln = 0
    while (1 << ln) < n:
        ln += 1
    return 93 - ln - _exp_above(wmax), 93 - ln - _exp_above(zmax)


def _integers(x, S):
    """round(x * 2^S), ties to even, as Python integers."""
    out = []
    for v in x:
        m, e = math.frexp(float(v))
        m, e = int(m * 2 ** 24), e - 24 + S      # v * 2^S = m * 2^e exactly
        if e >= 0:
            out.append(m << e)
        else:
            q, r = divmod(m, 1 << -e)
            half = 1 << (-e - 1)
            out.append(q + (1 if r > half or (r == half and q & 1) else 0))
    return out


def _expected(p, st, xs, ys, zs, pose):
    d = O.point_decisions(p, st, xs, ys, zs, pose)
    R, t = d["R"], d["t"]
    a = np.nonzero(d["accept"])[0]
    with np.errstate(all="ignore"):
        w = F32(1) / d["sp2"][a]
        rz = (R[2, 0] * xs[a] + R[2, 1] * ys[a]) + R[2, 2] * zs[a]
        u = w * rz
    Sw, Su = _shifts(p, R, len(xs))
    sums = {}
    for c, iw, iu in zip(d["cell"][a].tolist(), _integers(w, Sw), _integers(u, Su)):
        iw = max(iw, 1)
        s = sums.setdefault(c, [0, 0, 0, 0])
        s[0] += iw >> 32
        s[1] += iw & 0xFFFFFFFF
        s[2] += iu >> 32
        s[3] += iu & 0xFFFFFFFF
    h, v = st.h.reshape(-1).copy(), st.v.reshape(-1).copy()
    for c, (wh, wl, zh, zl) in sums.items():
        sw = math.ldexp(float(wh) * 4294967296.0 + float(wl), -Sw)
        sz = math.ldexp(float(zh) * 4294967296.0 + float(zl), -Su)
        acc_w, acc_z = F32(sw), F32(sz + float(t[2]) * sw)
        v1 = F32(1) / (F32(1) / v[c] + acc_w)
        h[c], v[c] = (h[c] / v[c] + acc_z) * v1, v1
    return h.reshape(st.h.shape), v.reshape(st.v.shape), d, len(sums)


def _frame(kind, rng, n, side, r):
    """Sensor-frame points of a sensor 1 m above the middle of the map."""
    if kind == "one cell":
        x, y = rng.uniform(0.0, r, n), rng.uniform(0.0, r, n)
    elif kind == "scattered":
        x, y = (rng.uniform(-0.5, 0.5, n) * side * r for _ in range(2))
    else:                               # rings, in scan order
        a = np.arange(n) * (2 * np.pi / 700)
        rad = 0.06 + (np.arange(n) // 700) / max(1, n // 700) * 0.7 * side * r
        x, y = rad * np.cos(a), rad * np.sin(a)
    z = -1.0 + rng.uniform(-0.4, 0.9, n)
    if kind == "range":                 # from the minimum range to far below, and near 0 height
        z = np.where(rng.random(n) < 0.3, rng.normal(0, 1e-6, n), z)
        z = np.where(rng.random(n) < 0.1, -10.0 ** rng.uniform(0, 4, n), z)
    return tuple(q.astype(F32) for q in (x, y, z))


CASES = [("rings", 1), ("rings", 255), ("rings", 256), ("rings", 257), ("rings", 3001),
         ("one cell", 1024), ("one cell", 66000), ("scattered", 4096), ("scattered", 70001),
         ("rings", 65536), ("rings", 65537), ("range", 5000)]


@pytest.mark.parametrize("batched", [False, True, '{"grid_chunk": 1}'])
@pytest.mark.parametrize("kind,n", CASES)
def test_fused_cells_bitwise(dev, kind, n, batched):
    from paper_2204_12876_amd import BatchEntry, ElevationMap, PipelineBatch, _emx
    print("[case] fusion sums", kind, n, "batched" if batched else "plain", batched, flush=True)
    rng = np.random.default_rng(n + len(kind))
    side, r = 300, 0.05
    params = dict(nx=side, ny=side - 11, resolution=r, noise_alpha=1e-4 if kind != "range" else 3e-3,
                  gate_k=3.0 if kind != "range" else 1e6, min_range=0.05)
    p = O.Params.from_dict(params)
    xs, ys, zs = _frame(kind, rng, n, side, r)
    yaw = 0.3
    pose = np.zeros((3, 4))
    pose[:, :3] = [[math.cos(yaw), -math.sin(yaw), 0.02], [math.sin(yaw), math.cos(yaw), -0.01],
                   [-0.02, 0.01, 0.9997]]
    pose[:, 3] = (0.01, -0.02, 1.0)
    st = random_state(p, rng, valid_frac=0.7)
    st.v[st.valid == 0] = 1e3
    m = ElevationMap(params, 0.0, 0.0, 0, device=dev)
    load_state(m, st)
    # the fused call moves the map first: some points fall in entering cells
    cx, cy = 7 * r + 0.01, -4 * r + 0.01
    moved = O.move_map(p, st, cx, cy)
    pts = tuple(torch.from_numpy(q).to(dev) for q in (xs, ys, zs))
    cell = torch.full((n,), -7, dtype=torch.int32, device=dev)
    acc = torch.full((n,), 7, dtype=torch.uint8, device=dev)
    if batched:
        pb = PipelineBatch(None if batched is True else batched, device=dev)
        pb.run([BatchEntry(m, *pts, pose, 900, center=(cx, cy), out_cell=cell, out_accept=acc,
                           stages=_emx.STAGE_MOVE | _emx.STAGE_FUSE)])
    else:
        m.move_fuse_points(cx, cy, *pts, pose, 900, out_cell=cell, out_accept=acc)
    torch.cuda.synchronize()
    h, v, d, fused = _expected(p, moved, xs, ys, zs, pose)
    assert np.array_equal(cell.cpu().numpy(), d["cell"].astype(np.int32))
    assert np.array_equal(acc.cpu().numpy().astype(bool), d["accept"])
    g = m.state_numpy()
    assert np.array_equal(g["h"].view(np.uint32), h.view(np.uint32))
    assert np.array_equal(g["v"].view(np.uint32), v.view(np.uint32))
    print("[case]  ", int(d["accept"].sum()), "points in", fused, "cells", flush=True)
    if batched:
        pb.close()
    m.close()
