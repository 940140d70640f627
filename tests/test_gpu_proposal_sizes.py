"""Proposal runs around the sizes at which the walk changes (2^19 rays, 128
voxels an axis): each against the run with a ledger, which always takes the
event walk.  Counts equal, sums within the parity bar."""
import numpy as np
import pytest

import workloads
from test_gpu_bundle import torch_cuda  # noqa: F401
from test_gpu_parity import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("size,n", [(40, 1000), (40, 2 ** 19), (127, 2 ** 19 + 1), (128, 2 ** 19 - 1), (128, 2 ** 19)])
def test_proposal_walks_agree(torch_cuda, size, n):  # noqa: F811
    import paper_2410_08747_amd as m
    torch = torch_cuda
    announce("proposal sizes", size, n)
    I = m.Instrument(workloads.edct_projection(workloads.make_phantom(size, 2), workloads.make_mu_tables(2), angle=0.4,
                                               strata=256, nx=64, ny=16, ne=16))
    lo, hi = (np.array(v) for v in I.proposal_box())
    rng = np.random.default_rng(3)
    gmm = np.empty((8, 7))
    gmm[:, 0] = 1 / 8
    gmm[:, 1:4] = lo + (hi - lo) * rng.uniform(0.2, 0.8, (8, 3))
    gmm[:, 4:7] = 0.3 * (hi - lo)
    I.set_proposal(torch.tensor(gmm.ravel(), device="cuda"), alpha=0.2)
    got, ref = I.run(n, seed=6)[0], I.run(n, seed=6, ledger=I.new_ledger())[0]
    torch.cuda.synchronize()
    assert int(ref["count"].sum()) > 100
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.abs(g - r) <= 1e-9 * np.abs(r)), k
