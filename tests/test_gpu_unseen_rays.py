"""Rays that the monitor will not see end before the phantom is walked: plain
and collecting runs of the cone-beam / absorbing-phantom / monitor chains
test the monitor's pixels first.  The image must be the one of the general
path, which carries every ray to the end (a run with a ledger): counts
equal, sums within the per-bin parity bar divided by a hundred, whatever part
of the cone the monitor covers -- none, a part, one pixel, turned, behind
the source -- and for every phantom model and source the shortcut serves."""
import numpy as np
import pytest

import workloads

from test_gpu_parity import announce

pytestmark = pytest.mark.gpu

N = 150_001


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def rot_x(a):
    c, s = np.cos(a), np.sin(a)
    return np.array([[1.0, 0.0, 0.0], [0.0, c, s], [0.0, -s, c]])


# monitor placements: name -> changes of the component
PLACES = {
    "as built": {},
    "half of the cone": {"xmin": 3.2, "xmax": 51.2},
    "one pixel": {"xmin": -1.0, "xmax": 1.0, "ymin": -1.0, "ymax": 1.0, "nx": 1, "ny": 1},
    "off the cone": {"pos": (4000.0, 0.0, 1200.0)},
    "behind the source": {"pos": (0.0, 0.0, -200.0)},
    "turned and shifted": {"pos": (20.0, -5.0, 1150.0), "rot": workloads.rot_y(0.4) @ rot_x(-0.2)},
    "a part of the spectrum": {"emin": 60.0, "emax": 90.0},
    "wavelength bins": {"wavelength": True, "emin": 0.08, "emax": 0.6},
}
MODELS = {"exact": {}, "exact, voxel 0.8": {}, "steps": {"step": 1.0 / 3.0}, "early-out": {"early_out": True}}


def build(model, place):
    ins = workloads.edct_projection(workloads.make_phantom(40, seed=2), workloads.make_mu_tables(2), angle=0.7, strata=48,
                                    nx=64, ny=16, ne=8, **MODELS[model])
    if "0.8" in model:
        ins["components"][1]["voxel"] = 0.8
    ins["components"][-1].update(PLACES[place])
    return ins


def compare(got, ref):
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.array_equal(g == 0, r == 0)
        assert np.all(np.abs(g - r) <= 1e-11 * np.abs(r)), k


@pytest.mark.parametrize("place", sorted(PLACES))
@pytest.mark.parametrize("model", sorted(MODELS))
def test_image_equals_the_ledger_runs(torch_cuda, model, place):
    import paper_2410_08747_amd as m
    announce("unseen rays", model, place)
    I = m.Instrument(build(model, place))
    got, ref = I.run(N, seed=5)[0], I.run(N, seed=5, ledger=I.new_ledger())[0]
    torch_cuda.cuda.synchronize()
    compare(got, ref)
    seen = int(ref["count"].sum())
    assert (seen == 0) == (place in ("off the cone", "behind the source"))


@pytest.mark.parametrize("place", ["half of the cone", "off the cone", "turned and shifted"])
def test_proposal_and_collection(torch_cuda, place):
    import paper_2410_08747_amd as m
    announce("unseen rays, proposal and collection", place)
    I = m.Instrument(build("exact", place))
    ref = I.run(N, seed=6, ledger=I.new_ledger())[0]
    hits = I.new_hits(N)
    got = I.collect(N, seed=6, context=np.zeros(6), hits=hits)[0]
    torch_cuda.cuda.synchronize()
    compare(got, ref)
    assert int(hits["count"].item()) == int(ref["count"].sum())
    g = np.zeros((8, 7))
    lo, hi = I.proposal_box()
    g[:, 0], g[:, 1], g[:, 2], g[:, 3] = 1.0, np.linspace(lo[0], hi[0], 8), 0.0, 80.0
    g[:, 4:] = 0.3 * hi[0], 0.3 * hi[1], 30.0
    I.set_proposal(torch_cuda.tensor(g.reshape(56), device="cuda"), alpha=0.2)
    got, ref = I.run(N, seed=7)[0], I.run(N, seed=7, ledger=I.new_ledger())[0]
    torch_cuda.cuda.synchronize()
    compare(got, ref)
