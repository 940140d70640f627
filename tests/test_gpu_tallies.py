"""A run's new histograms are tensors of their own: each holds its memory alone (what
is kept or saved of one does not keep the others), and takes in-place updates that
autograd follows."""
import io

import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


@pytest.mark.parametrize("nx,ny,ne", [(1, 1, 1), (61, 17, 33), (256, 64, 128)])
def test_histograms_of_their_own(torch_cuda, nx, ny, ne):
    import paper_2410_08747_amd as m
    torch = torch_cuda
    I = m.Instrument(workloads.edct_projection(workloads.make_phantom(40, seed=2), workloads.make_mu_tables(2), nx=nx, ny=ny,
                                               ne=ne))
    junk = [torch.full((nx * ny * ne,), 7.0, dtype=torch.float64, device="cuda") for _ in range(6)]
    del junk  # freed memory that the new histograms may be given
    t = I.new_tallies()[0]
    bins = nx * ny * ne
    for k, dtype in (("count", torch.int64), ("sum_w", torch.float64), ("sum_w2", torch.float64)):
        assert t[k].dtype == dtype and t[k].shape == (bins,) and t[k].is_contiguous() and int(t[k].count_nonzero()) == 0
        assert t[k].untyped_storage().nbytes() == 8 * bins
        f = io.BytesIO()
        torch.save(t[k], f)
        assert len(f.getvalue()) < 8 * bins + 4096
    assert len({t[k].untyped_storage().data_ptr() for k in t}) == 3
    x = torch.full((bins,), 2.0, dtype=torch.float64, device="cuda", requires_grad=True)
    t["sum_w"].add_(x)
    t["sum_w"].sum().backward()
    assert torch.equal(x.grad, torch.ones_like(x))
