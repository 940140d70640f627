"""Fixed steps: a path's last step ends behind the volume, up to its whole length,
and reads the voxel clamped into the last layer.  With the source inside the
volume the rays of a wave cross each other's places between the layers behind
the source and the last one, so the span they cover behind the last layer does
not follow from the spans at the volume's two ends alone.  Stripes of another
material in the last layers; long steps.  Plain runs against runs with a ledger
(one ray at a time)."""
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


def volume(width):
    """Clear but for a frame (so that the layers are looked at) and stripes in
    the first and last layers across z."""
    vol = np.zeros((128, 64, 64), np.uint8)
    vol[2:126, 0, 0] = 1
    stripes = (2 + (np.arange(64) // width) % 2).astype(np.uint8)
    vol[:3] = stripes
    vol[-3:] = stripes[::-1]
    return vol


@pytest.mark.parametrize("forward", [True, False])
@pytest.mark.parametrize("step,width,strata", [(8.0, 3, 400), (8.0, 5, 200), (2.5, 4, 300), (0.5, 3, 300), (300.0, 16, 300)])
def test_source_inside(torch_cuda, forward, step, width, strata):
    import paper_2410_08747_amd as m
    announce("last step, source inside", forward, step, width, strata)
    mu = np.zeros((4, 8))
    mu[0], mu[1], mu[2], mu[3] = 1e-3, 0.01, 0.2, 4.0
    ins = workloads.edct_projection(volume(width), mu, angle=0.0 if forward else np.pi, strata=strata, nx=64, ny=16, ne=2,
                                    step=step)
    src, ph, det = ins["components"]
    ph["pos"] = (0.3, 0.2, 7.0)
    I = m.Instrument(ins)
    n = 16 * strata * strata + 1001
    got, ref = I.run(n, seed=4)[0], I.run(n, seed=4, ledger=I.new_ledger())[0]
    torch_cuda.cuda.synchronize()
    assert int(ref["count"].sum()) > 1000
    assert np.array_equal(got["count"].cpu().numpy(), ref["count"].cpu().numpy())
    for k in ("sum_w", "sum_w2"):
        g, r = got[k].cpu().numpy(), ref[k].cpu().numpy()
        assert np.all(np.abs(g - r) <= 1e-11 * np.abs(r)), (k, np.max(np.abs(g - r) / np.where(r != 0, r, 1)))
