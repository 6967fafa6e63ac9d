"""Clearing on maps and at ray steps at the edges of the march's forms, alone and
in a batch, against the oracle, which tests every sample: marks, state and bound
bit for bit."""
import pytest

from test_gpu_clear_long_rays import _check
from test_gpu_clear_march import dev  # noqa: F401

pytestmark = pytest.mark.gpu

# nx, ny, step / r, sensor (cells), reach (cells), n, valid, flat.  Maps of one row or
# column of 8 x 8 blocks, or of 32 x 32 superblocks, down to one block; the counts of
# blocks on both sides of the maxima's padding (64 to 256 bytes).
NARROW = [
    (8, 300, 1.0, (4.0, 20.0), 290, 700, 0.6, True),
    (300, 7, 1.0, (20.0, 3.0), 290, 700, 0.6, True),
    (5, 5, 1.0, (2.5, 2.5), 9, 300, 0.9, False),
    (8, 8, 0.3, (1.0, 7.0), 12, 300, 0.9, False),
    (9, 512, 1.0, (4.0, 500.0), 520, 700, 0.6, True),
    (3, 504, 1.0, (1.0, 10.0), 520, 500, 0.6, True),
    (4, 512, 1.0, (1.0, 10.0), 520, 500, 0.6, True),
    (512, 8, 0.25, (5.0, 4.0), 520, 500, 0.6, True),
    (2050, 8, 1.0, (1000.0, 4.0), 1100, 700, 0.6, True),
    (8, 2050, 1.0, (4.0, 1000.0), 1100, 50000, 0.6, True),
]


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("ub", [0, 1])
@pytest.mark.parametrize("k", range(len(NARROW)))
def test_narrow_maps(dev, k, ub, batched):  # noqa: F811
    _check(dev, NARROW[k], 5000 + 10 * k + ub, ub, batched)


# Ray steps around and above the length at which the march gives up its groups (three
# samples to 7 cells: 2.33), and groups of three, four and five samples; frames around
# the widths of its workgroups, and samples around whole runs of eight.
STEPS = [
    (160, 150, 1.39, (80.0, 70.0), 150, 900, 0.7, True),
    (160, 150, 1.41, (80.0, 70.0), 150, 900, 0.7, True),
    (160, 150, 1.76, (80.0, 70.0), 150, 900, 0.7, True),
    (160, 150, 2.33, (80.0, 70.0), 150, 900, 0.7, True),
    (160, 150, 2.34, (80.0, 70.0), 150, 900, 0.7, True),
    (160, 150, 5.0, (3.0, 4.0), 230, 31, 0.7, True),
    (160, 150, 5.0, (3.0, 4.0), 230, 33, 0.7, True),
    (160, 150, 3.0, (3.0, 4.0), 230, (3 << 14) + 1, 0.7, True),
    (160, 150, 3.0, (3.0, 4.0), 230, (1 << 17) + 1, 0.7, True),
    (1200, 1100, 2.5, (5.0, 4.0), 1500, 700, 0.6, True),
    (8, 300, 4.0, (4.0, 20.0), 290, 700, 0.6, True),
    (3, 3, 2.5, (1.5, 1.5), 6, 1, 1.0, False),
    (160, 150, 300.0, (80.0, 70.0), 400, 700, 0.7, True),
]


@pytest.mark.parametrize("batched", [False, True])
@pytest.mark.parametrize("ub", [0, 1])
@pytest.mark.parametrize("k", range(len(STEPS)))
def test_long_steps(dev, k, ub, batched):  # noqa: F811
    _check(dev, STEPS[k], 6000 + 10 * k + ub, ub, batched)


def test_batch_of_maps_with_short_and_long_steps(dev):  # noqa: F811
    """One batch holds items of both marches: each equals its plain call."""
    import numpy as np
    import torch
    from paper_2204_12876_amd import BatchEntry, ElevationMap, PipelineBatch, _emx
    import oracle as O
    from parity_util import load_state, random_state
    print("[case] batch of both marches", flush=True)
    rng = np.random.default_rng(71)
    pb = PipelineBatch(device=dev)
    plain, batch, entries, outs = [], [], [], []
    for k, (ratio, n) in enumerate([(1.0, 700), (4.0, 900), (0.5, 0), (3.0, 0), (9.0, 3000),
                                    (1.0, 5000), (2.4, 1)]):
        params = dict(nx=90 + k, ny=70 + 3 * k, resolution=0.05, ray_step=ratio * 0.05,
                      clear_normal_alpha=0.1, clear_min_age_ms=200, upper_bound=k % 2)
        p = O.Params.from_dict(params)
        st = random_state(p, rng, valid_frac=0.7)
        a = rng.uniform(0, 2 * np.pi, n)
        pts = [torch.from_numpy(q.astype(np.float32)).to(dev)
               for q in (3 * np.cos(a), 3 * np.sin(a), rng.uniform(-1.2, 0.0, n))]
        pose = np.eye(3, 4)
        pose[2, 3] = 0.6
        both = [ElevationMap(params, device=dev) for _ in range(2)]
        out = [torch.full((p.nx * p.ny,), 9, dtype=torch.uint8, device=dev) for _ in range(2)]
        for m in both:
            load_state(m, st)
        both[0].clear_visibility(*pts, pose, 900, out_cleared=out[0])
        entries.append(BatchEntry(both[1], *pts, pose, 900, out_cleared=out[1],
                                  stages=_emx.STAGE_CLEAR))
        plain.append(both[0])
        batch.append(both[1])
        outs.append(out)
    for _ in range(2):     # the second run replays the graph
        pb.run(entries)
    torch.cuda.synchronize()
    removed = 0
    for a, b, (oa, ob), e in zip(plain, batch, outs, entries):
        a.clear_visibility(e.x, e.y, e.z, e.pose, 900, out_cleared=oa)
        torch.cuda.synchronize()
        assert torch.equal(a.export_state(), b.export_state())
        assert torch.equal(oa, ob)
        if a.p.upper_bound:
            assert torch.equal(a.upper_bound().view(torch.int32), b.upper_bound().view(torch.int32))
        removed += int((a.state_numpy()["valid"] == 0).sum())
    assert removed > 100
    for m in plain + batch:
        m.close()
    pb.close()
