"""The clearing march where its rays are spread and shared out: long rays in
workgroups of 32, 64 and 128 (one frame) and of 256 (a batch), consecutive or
from several parts of the frame, more spans than a workgroup has threads, rays
of more than one round of spans, and the batch's own records at every step
length.  Against the oracle, which tests every sample: marks, state and bound
bit for bit.  Large frames repeat a few thousand rays in another order, which
changes no result (removals are idempotent, the bound is a minimum), so the
oracle marches each ray once."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_util import load_state, random_state
from test_gpu_clear_march import CASES, _points, dev  # noqa: F401

pytestmark = pytest.mark.gpu

F32 = np.float32


def _check(dev, case, seed, ub, batched, repeat=1):  # noqa: F811
    from paper_2204_12876_amd import BatchEntry, ElevationMap, PipelineBatch, _emx
    nx, ny, ratio, sensor, reach, n, valid, flat = case
    print("[case] long rays", case, "ub", ub, "batched" if batched else "plain", "x", repeat,
          flush=True)
    rng = np.random.default_rng(seed)
    r = 0.05
    params = dict(nx=nx, ny=ny, resolution=r, noise_alpha=0.01, gate_k=2.0, min_range=0.05,
                  ray_step=ratio * r, clear_normal_alpha=0.1, clear_min_age_ms=200,
                  upper_bound=ub)
    p = O.Params.from_dict(params)
    m = ElevationMap(params, 0.0, 0.0, 0, device=dev)
    m.move_map(5 * r + 0.01, -3 * r + 0.01)      # turns the ring
    st = random_state(p, rng, valid_frac=valid)
    st.cgx, st.cgy, _ = m.info()
    st.h.reshape(-1)[rng.integers(0, nx * ny, 5)] = np.nan
    load_state(m, st)
    ox, oy = (st.cgx - nx // 2) * r, (st.cgy - ny // 2) * r
    pose = np.eye(3, 4)
    pose[:, 3] = (ox + sensor[0] * r, oy + sensor[1] * r, 0.3 if flat else 1.0)
    xs, ys, zs = _points(rng, n, reach * r, flat)
    order = np.argsort(np.arctan2(ys, xs), kind="stable")      # scan order
    more = np.concatenate([order if k % 2 == 0 else order[::-1] for k in range(repeat)])
    pts = tuple(torch.from_numpy(a[more]).to(dev) for a in (xs, ys, zs))
    out = torch.full((nx * ny,), 9, dtype=torch.uint8, device=dev)
    bound = np.full((ny, nx), np.inf, F32)
    pb = PipelineBatch(device=dev) if batched else None
    for t_ms in (700, 800):
        if batched:
            pb.run([BatchEntry(m, *pts, pose, t_ms, out_cleared=out, stages=_emx.STAGE_CLEAR)])
        else:
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
    if batched:
        pb.close()
    m.close()


@pytest.mark.parametrize("ub", [0, 1])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_batched_march_equals_every_sample(dev, case, ub):  # noqa: F811
    _check(dev, CASES[case], 3000 + 10 * case + ub, ub, True)


# nx, ny, step / r, sensor, reach, n, valid, flat; how often the frame is repeated
LONG = [
    ((600, 590, 1.0, (6.0, 8.0), 800, 3000, 0.5, True), 2),      # 32 rays, shared spans
    ((600, 590, 1.0, (6.0, 8.0), 800, 3000, 0.5, True), 20),     # 64 rays, shared spans
    ((600, 590, 1.0, (6.0, 8.0), 800, 3001, 0.5, True), 50),     # 128 rays, shared spans
    ((600, 590, 1.0, (6.0, 8.0), 800, 3001, 0.5, True), 90),     # 128 rays, runs of 64
    ((600, 590, 1.0, (6.0, 8.0), 800, 3001, 0.5, True), 200),    # 128 rays, consecutive
    ((300, 310, 1.0, (6.0, 8.0), 400, 3000, 0.5, True), 20),     # 64 rays, consecutive
    ((2300, 40, 1.0, (3.0, 20.0), 2290, 600, 0.5, True), 1),     # over 64 spans to a ray
    ((200, 190, 0.05, (3.0, 20.0), 260, 600, 0.5, True), 1),     # over 4000 samples to a ray
]


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("ub", [0, 1])
@pytest.mark.parametrize("k", range(len(LONG)))
def test_long_rays(dev, k, ub, batched):  # noqa: F811
    case, repeat = LONG[k]
    _check(dev, case, 4000 + 10 * k + ub, ub, batched, repeat)
