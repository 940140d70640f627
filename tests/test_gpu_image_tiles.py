"""Tiled image runs: every ray id is traced once, whatever the run's size, part
and strata, and the work-group's private histogram loses nothing, whether the
monitor's bins fit its window, collide in it or are too many for it.  The
reference is the run with a ledger (one ray per lane in the order of the ids,
tallied straight into the caller's arrays): counts equal, sums within the
per-bin parity bar divided by a hundred."""
import numpy as np
import pytest

import workloads

from test_gpu_parity import announce

pytestmark = pytest.mark.gpu

BIG = (1 << 23) + 12_345  # the fewest rays that give a tile two rounds, and a ragged end


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def same(got, ref, rtol=1e-11):
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.array_equal(g == 0, r == 0)
        assert np.all(np.abs(g - r) <= rtol * np.abs(r)), k


def instrument(strata, nx=64, ny=16, ne=8, **kw):
    import paper_2410_08747_amd as m
    return m.Instrument(workloads.edct_projection(workloads.make_phantom(64, seed=6), workloads.make_mu_tables(6), angle=0.4,
                                                  strata=strata, nx=nx, ny=ny, ne=ne, **kw))


@pytest.mark.parametrize("strata,n", [(1, 1), (1, 1000), (4096, 15), (4096, 257), (3, 1023), (37, 99_991), (500, 1_000_003)])
def test_every_ray_once(torch_cuda, strata, n):
    announce("image tiles, rays", strata, n)
    I = instrument(strata, nx=2, ny=2, ne=1)
    same(I.run(n, seed=1)[0], I.run(n, seed=1, ledger=I.new_ledger())[0])


@pytest.mark.parametrize("cuts", [(0, 1, 64, 5000, 200_001), (0, 100_000, 100_001, 200_001)])
def test_parts_of_a_run(torch_cuda, cuts):
    announce("image tiles, parts", cuts)
    I = instrument(200)
    n = cuts[-1]
    got = I.new_tallies()
    for a, b in zip(cuts[:-1], cuts[1:]):
        I.run(b - a, seed=2, first_ray=a, n_total=n, tallies=got)
    same(got[0], I.run(n, seed=2, ledger=I.new_ledger())[0])


@pytest.mark.parametrize("nx,ny,ne", [(64, 16, 8), (61, 17, 33), (256, 64, 128), (8, 4, 1024), (8, 4, 1025), (512, 256, 1), (1, 1, 1)])
def test_private_histogram(torch_cuda, nx, ny, ne):
    announce("image tiles, histogram", nx, ny, ne)
    I = instrument(1024, nx=nx, ny=ny, ne=ne)
    same(I.run(BIG, seed=3)[0], I.run(BIG, seed=3, ledger=I.new_ledger())[0])


def test_proposal_and_steps(torch_cuda):
    announce("image tiles, proposal and steps")
    I = instrument(1024, step=0.5)
    same(I.run(BIG, seed=4)[0], I.run(BIG, seed=4, ledger=I.new_ledger())[0])
    I = instrument(1024)
    lo, hi = I.proposal_box()
    g = np.zeros((8, 7))
    g[:, 0] = [1.0, 0.0, 3.0, 1e-9, 1.0, 1.0, 2.0, 0.5]  # an empty branch and one of next to no rays
    g[:, 1], g[:, 2], g[:, 3] = np.linspace(0.8 * lo[0], 0.8 * hi[0], 8), 0.1 * hi[1], 80.0
    g[:, 4:] = 0.3 * hi[0], 0.1 * hi[1], 30.0
    for alpha in (0.0, 0.1, 1.0):
        I.set_proposal(torch_cuda.tensor(g.reshape(56), device="cuda"), alpha=alpha)
        same(I.run(BIG, seed=5)[0], I.run(BIG, seed=5, ledger=I.new_ledger())[0])
