"""Tiles whose rays all miss the monitor end at once, and the tiles left keep a private
histogram: both from 2^23 rays on.  Monitors turned and shifted, covering a part of
the cone, one pixel of it, none of it, or standing behind the source; a wide cone, an
aperture before the phantom, a ray sink; strata from a tile's size down to a
fraction of it.  Against the run with a ledger: counts equal, sums within the
per-bin parity bar divided by a hundred."""
import numpy as np
import pytest

import workloads

from test_gpu_parity import announce
from test_gpu_unseen_rays import PLACES, compare

pytestmark = pytest.mark.gpu

N = (1 << 23) + 12_345


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def build(place, strata, half_angle=None, **kw):
    ins = workloads.edct_projection(workloads.make_phantom(40, seed=2), workloads.make_mu_tables(2), angle=0.7, strata=strata,
                                    nx=64, ny=16, ne=8, **kw)
    ins["components"][-1].update(PLACES[place])
    if half_angle is not None:
        ins["components"][0]["half_angle"] = half_angle
    return ins


def both_forms(torch, ins, n, seed):
    import paper_2410_08747_amd as m
    I = m.Instrument(ins)
    ref = I.run(n, seed=seed, ledger=I.new_ledger())[0]
    for occupancy in (4, 0):
        I.launch_shape = (occupancy, 1, 0, 1)
        got = I.run(n, seed=seed)[0]
        torch.cuda.synchronize()
        compare(got, ref)
    return int(ref["count"].sum())


@pytest.mark.parametrize("strata", [1, 37, 256, 1024])
@pytest.mark.parametrize("place", ["half of the cone", "one pixel", "off the cone", "behind the source", "turned and shifted"])
def test_monitors(torch_cuda, place, strata):
    announce("culled tiles", place, strata)
    seen = both_forms(torch_cuda, build(place, strata), N, 5)
    assert (seen == 0) == (place in ("off the cone", "behind the source"))


@pytest.mark.parametrize("half_angle", [0.6, 1.5, 2.6])
@pytest.mark.parametrize("place", ["as built", "turned and shifted"])
def test_wide_cones(torch_cuda, place, half_angle):
    announce("culled tiles, cone", place, half_angle)
    assert both_forms(torch_cuda, build(place, 1024, half_angle), N, 6) > 1000


def test_source_turned_away(torch_cuda):
    """The cone's axis at 1.2 rad to the monitor's: few of its tiles reach it."""
    announce("culled tiles, source turned")
    ins = build("as built", 512, 1.4)
    ins["components"][0]["rot"] = workloads.rot_y(1.2)
    assert both_forms(torch_cuda, ins, N, 7) > 1000


@pytest.mark.parametrize("strata", [64, 1024])
@pytest.mark.parametrize("model", [{"early_out": True}, {"step": 0.5}])
def test_chains(torch_cuda, model, strata):
    announce("culled tiles, chain", model, strata)
    for place in ("half of the cone", "turned and shifted"):
        both_forms(torch_cuda, build(place, strata, **model), N, 8)


@pytest.mark.parametrize("place", ["half of the cone", "turned and shifted"])
def test_collection(torch_cuda, place):
    import paper_2410_08747_amd as m
    announce("culled tiles, collection", place)
    I = m.Instrument(build(place, 1024))
    ref = I.run(N, seed=9, ledger=I.new_ledger())[0]
    hits = I.new_hits(N)
    got = I.collect(N, seed=9, context=np.zeros(6), hits=hits)[0]
    torch_cuda.cuda.synchronize()
    compare(got, ref)
    rows = int(hits["count"].item())
    assert rows == int(ref["count"].sum())
    bins = torch_cuda.bincount(hits["bin"][:rows], minlength=ref["count"].numel())
    assert torch_cuda.equal(bins, ref["count"])
