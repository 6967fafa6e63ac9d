"""Batches of any mix of robots share few captured graphs: a server that takes what
is ready forms batches of every size and mix, and each new set of grid sizes costs
a capture."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_12876_amd import _emx
    _emx.lib()
    return torch.device("cuda:0")


@pytest.mark.parametrize("most", [4, 8, 24])
def test_mixed_batches_share_graphs(dev, most):
    from paper_2204_12876_amd import BatchEntry, ElevationMap, PipelineBatch
    print("[case] mixed batches of up to", most, flush=True)
    rng = np.random.default_rng(most)
    side = rng.integers(64, 400, 24)
    n = np.exp(rng.uniform(np.log(2000), np.log(200000), 24)).astype(int)
    maps = [ElevationMap(dict(nx=int(s), ny=int(s), resolution=0.05), device=dev) for s in side]
    x = torch.linspace(-3, 3, int(n.max()), device=dev)
    w = torch.zeros(89, device=dev)
    pose = np.eye(3, 4)
    pose[2, 3] = 1.0
    pb = PipelineBatch(device=dev)
    entry = lambda i, k: BatchEntry(maps[i], x[:n[i]], -x[:n[i]], x[:n[i]] * 0 - 1, pose, 10 * k,
                                    center=(0.01 * k, 0.0), weights=w)
    pb.run([entry(i, 0) for i in range(24)])           # the scratch at its largest
    start = pb.stats()[1]
    for k in range(120):
        pick = rng.permutation(24)[:rng.integers(1, most + 1)]
        pb.run([entry(int(i), k + 1) for i in pick])
    torch.cuda.synchronize()
    runs, captures = pb.stats()
    assert runs == 121 and captures - start <= 16, captures
    pb.close()
    for m in maps:
        m.close()
