"""Normals and traversability at the edges of the stencil's tiles (62 columns, a
wave's rows, a workgroup's rows), on turned rings, with holes at the tile seams,
and with weights that start at any float: against the oracle, and the three
forms (normals, traversability, both; alone and batched) bit for bit against
each other."""
import numpy as np
import pytest
import torch

import oracle as O
from parity_util import (assert_normals_parity, assert_trav_parity, load_state, random_state)

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2204_12876_amd import _emx
    _emx.lib()
    return torch.device("cuda:0")


SHAPES = [(3, 3), (4, 9), (62, 8), (63, 7), (64, 17), (61, 16), (124, 33), (125, 1000), (187, 15),
          (500, 3), (3, 500)]


@pytest.mark.parametrize("nx,ny", SHAPES)
def test_tiles(dev, nx, ny):
    from paper_2204_12876_amd import BatchEntry, ElevationMap, PipelineBatch, _emx
    print("[case] stencil tiles", nx, ny, flush=True)
    rng = np.random.default_rng(1000 * nx + ny)
    params = dict(nx=nx, ny=ny, resolution=0.05)
    p = O.Params.from_dict(params)
    w = rng.normal(size=95).astype(np.float32)
    dw = torch.from_numpy(w).to(dev)
    for off, valid in ((0, 1.0), (1, 0.97), (3, 0.5)):
        m = ElevationMap(params, 0.0, 0.0, 0, device=dev)
        m.move_map(0.05 * (1 + off) + 0.01, -0.05 * off + 0.01)    # a turned ring
        st = random_state(p, rng, valid_frac=valid)
        st.cgx, st.cgy, _ = m.info()
        weights = dw[off:off + 89]
        outs = []
        for form in ("two", "one", "batch"):
            load_state(m, st)
            if form == "two":
                m.compute_normals()
                m.traversability(weights)
            elif form == "one":
                m.normals_traversability(weights)
            else:
                pb = PipelineBatch(device=dev)
                pb.run([BatchEntry(m, weights=weights,
                                   stages=_emx.STAGE_NORMALS | _emx.STAGE_TRAV)])
                torch.cuda.synchronize()
                pb.close()
            torch.cuda.synchronize()
            outs.append(m.state_numpy())
        g = outs[0]
        assert_normals_parity(g, O.compute_normals(p, st.h, st.valid))
        assert_trav_parity(g, *O.traversability(st.h, st.valid, w[off:off + 89]))
        for o in outs[1:]:
            for k in ("nrm", "trav", "h", "valid"):
                assert np.array_equal(g[k].view(np.uint8), o[k].view(np.uint8)), k
        m.close()
