"""The Gaussian source's directions, whose logarithm, roots, quotients and circular
functions are evaluated for their known ranges, against extended precision on
the same uniforms.

Direction: tan(sigma r c), r = sqrt(-2 log u0), c = cos or sin of 2 pi u1, over
the norm.  Each of log, root, circular function, tan, product and quotient is
within about an ulp and the norm halves its argument's error, so the sum stays
below 8 ulp of sigma r (1 + tan^2 enters through the tangent's slope)."""
import numpy as np
import pytest

import oracle
import workloads
from test_gpu_parity import announce

pytestmark = pytest.mark.gpu

U = 2.0 ** -53


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


@pytest.mark.parametrize("sigma", [1e-9, 1e-4, 2e-3, 0.02])
def test_gaussian_directions(torch_cuda, sigma):
    import paper_2410_08747_amd as m
    announce("Gaussian source directions", sigma)
    ins = workloads.crl_focusing()
    src = dict(ins["components"][0], sigma_xp=sigma, sigma_yp=sigma / 3, pos=(0.0, 0.0, 0.0), rot=np.eye(3))
    det = dict(ins["components"][-1], pos=(0.0, 0.0, 1.0), rot=np.eye(3))
    ids = np.arange(40_000, dtype=np.uint64)
    out = m.Instrument({"components": [src, det]}).trace_rays(ids, seed=77, n_total=ids.size)
    torch_cuda.cuda.synchronize()
    L = np.longdouble
    u = np.array([[oracle.uniform(77, int(i), k) for k in (2, 3)] for i in ids[:4000]]).astype(L)
    r = np.sqrt(-2 * np.log(u[:, 0]))
    two_pi = L(2) * np.arctan2(L(0), L(-1))
    t = [np.tan(L(sigma) * r * np.cos(two_pi * u[:, 1])), np.tan(L(sigma / 3) * r * np.sin(two_pi * u[:, 1]))]
    nrm = np.sqrt(t[0] ** 2 + t[1] ** 2 + 1)
    for name, ref, scale in (("dx", t[0] / nrm, sigma * r), ("dy", t[1] / nrm, sigma / 3 * r), ("dz", 1 / nrm, 1 + sigma * r)):
        got = out[name].cpu().numpy()[:4000].astype(L)
        bound = 8 * U * scale * (1 + (sigma * r) ** 2)
        assert np.all(np.abs(got - ref) <= bound), (name, float(np.max(np.abs(got - ref) / bound)))
