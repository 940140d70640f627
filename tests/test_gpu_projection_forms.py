"""Projections have two forms -- the rays of a wave as a bundle, in tiles, or each
ray by itself -- and which one a run takes depends on its size and its phantom.
Both, and the run's own choice, against the run with a ledger: counts equal, sums
within the per-bin parity bar divided by a hundred (scattered photons: within the
bar).  The volumes and views of the bundle walk's tests, and the monitors of the
unseen rays'."""
import numpy as np
import pytest

import workloads

from test_gpu_bundle import VIEWS, VOLUMES
from test_gpu_parity import announce
from test_gpu_unseen_rays import PLACES

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def check(torch, ins, n, seed, rtol=1e-11):
    import paper_2410_08747_amd as m
    I = m.Instrument(ins)
    ref = I.run(n, seed=seed, ledger=I.new_ledger())[0]
    for occupancy in (4, 6, 8, 0):
        I.launch_shape = (occupancy, 1, 0, 1)
        got = I.run(n, seed=seed)[0]
        torch.cuda.synchronize()
        assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy()), occupancy
        for k in ("sum_w", "sum_w2"):
            g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
            assert np.all(np.abs(g - r) <= rtol * np.abs(r)), (occupancy, k, np.max(np.abs(g - r) / np.where(r != 0, r, 1)))
    return int(ref["count"].sum())


def build(name, view, **kw):
    angle, voxel, strata, n = VIEWS[view]
    mu = workloads.make_mu_tables(3)
    if kw.get("scatter_order"):
        mu = workloads.make_scatter_tables(mu)
    if kw.get("step"):
        kw["step"] *= voxel
    ins = workloads.edct_projection(VOLUMES[name](), mu, angle=angle, strata=strata, nx=32, ny=16, ne=4, **kw)
    next(c for c in ins["components"] if c["type"] == "phantom")["voxel"] = voxel
    return ins, n


@pytest.mark.parametrize("view", range(len(VIEWS)))
@pytest.mark.parametrize("name", sorted(VOLUMES))
def test_exact(torch_cuda, name, view):
    announce("projection forms", name, view)
    ins, n = build(name, view)
    assert check(torch_cuda, ins, n, 8) > 1000


@pytest.mark.parametrize("view,step", [(0, 1.0 / 3.0), (1, 2.5), (2, 0.75), (3, 1.7)])
@pytest.mark.parametrize("name", sorted(VOLUMES))
def test_steps(torch_cuda, name, view, step):
    announce("projection forms, steps", name, view, step)
    ins, n = build(name, view, step=step)
    assert check(torch_cuda, ins, n, 8) > 1000


@pytest.mark.parametrize("view,order", [(0, 1), (1, 1), (2, 2), (3, 1)])
@pytest.mark.parametrize("name", ["luggage 96", "noise 64x65x63", "slabs x 129"])
def test_scattered(torch_cuda, name, view, order):
    announce("projection forms, scattered", name, view, order)
    ins, n = build(name, view, scatter_order=order)
    assert check(torch_cuda, ins, n // 4, 8, rtol=1e-9) > 100


@pytest.mark.parametrize("place", sorted(PLACES))
@pytest.mark.parametrize("model", [{}, {"step": 1.0 / 3.0}, {"early_out": True}])
def test_monitors(torch_cuda, model, place):
    announce("projection forms, monitors", model, place)
    ins, n = build("luggage 96", 0, **model)
    ins["components"][-1].update(PLACES[place])
    check(torch_cuda, ins, n // 2, 5)


@pytest.mark.parametrize("form", [(0, 0, 0, 0), (1, 2, 4096, 0), (2, 0, 0, 2)])
@pytest.mark.parametrize("name", ["luggage 96", "noise 64x65x63"])
def test_batches(torch_cuda, name, form):
    """A batch's grid walks phantoms in the one form or the other by its jobs."""
    import paper_2410_08747_amd as m
    announce("projection forms, batch", name, form)
    for n in (1023, 700_001):  # 6 x 700,001 rays of a 96^3 phantom go as bundles
        made = [m.Instrument(build(name, v)[0]) for v in (0, 2)]
        jobs = [(made[j % 2], n, 3, j, made[j % 2].new_tallies()) for j in range(6)]
        m.Batch(jobs, schedule=form).run()
        torch_cuda.cuda.synchronize()
        for I, _, seed, j, got in jobs:
            ref = I.run(n, seed=seed, job=j, ledger=I.new_ledger())[0]
            assert np.array_equal(got[0]["count"].cpu().numpy(), ref["count"].cpu().numpy())
            for k in ("sum_w", "sum_w2"):
                g, r = got[0][k].cpu().numpy(), ref[k].cpu().numpy()
                assert np.all(np.abs(g - r) <= 1e-11 * np.abs(r)), k
