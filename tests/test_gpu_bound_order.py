"""The upper bound layer is a minimum, so it does not depend on the order of the
samples: not within a call, not between calls, and not in the sign of a zero (of
the two zeros the negative one is the lower).  The sensor is at height -0.0; rays
at height +0.0 and rays a denormal below, whose first samples round to -0.0,
cross the same cells without an estimate."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

F32 = np.float32


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_12876_amd import _emx
    _emx.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("ratio", [1.0, 4.0])
@pytest.mark.parametrize("batched", [False, True])
def test_zero_heights_have_no_order(dev, batched, ratio):
    from paper_2204_12876_amd import BatchEntry, ElevationMap, PipelineBatch, _emx
    print("[case] bound order", ratio, "batched" if batched else "plain", flush=True)
    r, side, n = 0.05, 96, 400
    params = dict(nx=side, ny=side, resolution=r, min_range=0.05, ray_step=ratio * r,
                  upper_bound=1)
    pose = np.eye(3, 4)
    pose[:, 3] = (0.01, 0.01, -0.0)
    a = np.linspace(0, 2 * np.pi, n, endpoint=False)
    x, y = ((2.2 * f(a)).astype(F32) for f in (np.cos, np.sin))
    plus, minus = np.zeros(n, F32), np.full(n, -1e-45, F32)
    pb = PipelineBatch(device=dev) if batched else None

    def bound(calls):
        m = ElevationMap(params, device=dev)
        for zs in calls:
            pts = [torch.from_numpy(np.concatenate([q] * len(zs))).to(dev) for q in (x, y)]
            pts.append(torch.from_numpy(np.concatenate(zs)).to(dev))
            if batched:
                pb.run([BatchEntry(m, *pts, pose, 100, stages=_emx.STAGE_CLEAR)])
            else:
                m.clear_visibility(*pts, pose, 100)
        out = m.upper_bound().cpu().numpy().view(np.uint32).copy()
        m.close()
        return out

    one = bound([(minus, plus)])
    assert (one == 0x80000000).sum() > 100            # -0.0
    assert (one == 1 << 31 | 1).sum() > 100            # the denormal
    for calls in ([(plus, minus)], [(minus,), (plus,)], [(plus,), (minus,)],
                  [(plus, plus, minus)], [(plus,), (plus,), (minus, plus)]):
        got = bound(calls)
        assert np.array_equal(got, one), int((got != one).sum())
    if batched:
        pb.close()
