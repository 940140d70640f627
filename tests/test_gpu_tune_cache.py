"""Tuning caches: a line written by other kernels is not taken (its shape may
select a slow kernel now), and tuning on a share of the rays times whole runs of
that many rays, in the form that the full run takes."""
import re

import pytest

import workloads

from test_gpu_parity import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def instrument():
    import paper_2410_08747_amd as m
    vol = workloads.make_phantom(64, seed=1)
    return m.Instrument(workloads.edct_projection(vol, workloads.make_mu_tables(1), angle=0.5, strata=256, nx=32, ny=16, ne=8))


def without_version(path, value):
    """The cache file's only line as kernels without a version would have written it."""
    line = open(path).read().splitlines()[0]
    key = re.sub(r"^kernels \d+ ", "", line.split("\t")[0])
    open(path, "w").write(f"{key}\t{value}\n")


def test_instrument_cache_of_other_kernels(torch_cuda, tmp_path):
    announce("tuning cache, instrument")
    cache = str(tmp_path / "tune.txt")
    instrument().autotune(200_000, 0.5, cache_path=cache)
    without_version(cache, "8 1 0 2")
    shape = instrument().autotune(200_000, 0.5, cache_path=cache)
    lines = open(cache).read().splitlines()
    assert len(lines) == 2 and lines[0].endswith("8 1 0 2")
    assert instrument().autotune(200_000, 0.5, cache_path=cache) == shape
    assert len(open(cache).read().splitlines()) == 2


def test_batch_cache_of_other_kernels(torch_cuda, tmp_path):
    import paper_2410_08747_amd as m
    announce("tuning cache, batch")
    cache = str(tmp_path / "tune.txt")
    made = [instrument() for _ in range(2)]

    def batch():
        return m.Batch([(I, 50_000, 1, j, I.new_tallies()) for j, I in enumerate(made)])

    batch().autotune(0.5, cache_path=cache)
    without_version(cache, "1 8 65536 0")
    schedule = batch().autotune(0.5, cache_path=cache)
    assert len(open(cache).read().splitlines()) == 2
    assert batch().autotune(0.5, cache_path=cache) == schedule


def test_a_share_of_the_rays_is_a_whole_run(torch_cuda):
    announce("tuning, share of the rays")
    I = instrument()
    n, share = 400_000, 0.25
    tallies = I.new_tallies()
    I.autotune(n, share, tallies=tallies)
    one = I.run(int(n * share), seed=1)[0]["count"]
    got = tallies[0]["count"]
    torch_cuda.cuda.synchronize()
    runs = int(got.sum()) // int(one.sum())
    assert runs > 0 and torch_cuda.equal(got, one * runs)


@pytest.mark.parametrize("n,forms", [(100_000, (6, 8)), (1 << 24, (4,))])
def test_a_share_of_the_rays_takes_the_full_run_s_form(torch_cuda, n, forms):
    announce("tuning, form", n)
    assert instrument().autotune(n, 0.25)[0] in forms
