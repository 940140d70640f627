"""An opaque material (attenuation infinite) in the volume: the rays that meet it
arrive with weight 0, all others as if it were not there.  A run of it of no
length -- a ray that a walk looks at again behind the place where the run
closed, or whose path has ended -- must not turn 0 times infinity into NaN.
Plain runs (the wave's bundle walk) against runs with a ledger (one ray at a
time), whose sums are finite here."""
import numpy as np
import pytest

import workloads

from test_gpu_parity import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def volume():
    """Opaque blocks and single voxels among others, clear of the faces."""
    vol = workloads.make_phantom(112, seed=9)
    rng = np.random.default_rng(9)
    vol[vol == 7] = 2
    for _ in range(40):
        z, y, x = rng.integers(20, 90, 3)
        s = int(rng.integers(1, 6))
        vol[z:z + s, y:y + s, x:x + s] = 7
    return vol


MODELS = {"exact": {}, "voxel 0.8": {}, "steps": {"step": 0.4}, "long steps": {"step": 2.5}, "early-out": {"early_out": True},
          "scattered once": {"scatter_order": 1}}


@pytest.mark.parametrize("angle,strata,n", [(0.0, 256, 1_200_007), (0.7853981, 16, 100_003), (2.9, 1, 50_021)])
@pytest.mark.parametrize("model", sorted(MODELS))
def test_opaque_material(torch_cuda, model, angle, strata, n):
    import paper_2410_08747_amd as m
    announce("opaque material", model, angle, strata, n)
    mu = workloads.make_mu_tables(3)
    if model == "scattered once":
        mu = workloads.make_scatter_tables(mu)
        mu[0, 7] = np.inf
    else:
        mu[7] = np.inf
    ins = workloads.edct_projection(volume(), mu, angle=angle, strata=strata, nx=32, ny=16, ne=4, **MODELS[model])
    if "0.8" in model:
        ins["components"][1]["voxel"] = 0.8
    I = m.Instrument(ins)
    got, ref = I.run(n, seed=8)[0], I.run(n, seed=8, ledger=I.new_ledger())[0]
    torch_cuda.cuda.synchronize()
    assert int(ref["count"].sum()) > 1000
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.isfinite(r))
        assert np.all(np.abs(g - r) <= 1e-9 * np.abs(r)), (k, int(np.sum(~np.isfinite(g))))
