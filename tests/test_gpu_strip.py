"""The network's one-launch kernel at the edges of its work split (16 rows a
wave, 128 a work-group, 256 work-groups) and the training weights of more runs
than one launch serves.

Products are checked as in the layer-by-layer tests: on the GPU's own bfloat16
operands within Higham's bound for a float32 accumulation.  A work-group sums
at most 2 x 128 rows here and the reduction 256 work-groups, so gamma_{K + 1}
with K = 512 bounds the weight and bias gradients.
"""
import numpy as np
import pytest

from oracle import proposal as P

from test_gpu_mlp import box, check_product, data, f64, gamma, mxr, params, torch_cuda  # noqa: F401
from test_gpu_parity import announce

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 16, 127, 129, 32769])
def test_layers_and_gradient_at_the_edges(torch_cuda, n):  # noqa: F811
    torch = torch_cuda
    m = mxr()
    announce("network strip n", n)
    net = m.ProposalNet(params(15), batch=n)
    ctx, y, omega = data(n, 16 + n)
    lo, hi = box()
    tc, ty, tw = (torch.tensor(v, device="cuda") for v in (ctx, y, omega))
    net.ws.fill_(0xFF)
    out = f64(net.forward(tc))
    loss, _ = net.loss_grad(tc, ty, tw, lo, hi)
    torch.cuda.synchronize()
    W = P.unpack(f64(net.w))
    bf, f4, f8 = torch.bfloat16, torch.float32, torch.float64
    R = {k: f64(net.region(k, n, t, c)) for k, t, c in (
        ("X", bf, 6), ("Z1", f4, 128), ("H1", bf, 128), ("Z2", f4, 128), ("H2", bf, 128), ("O", f4, 56), ("DO", f4, 56),
        ("DOH", bf, 56), ("DZ2", f4, 128), ("DZ2H", bf, 128), ("DZ1", f4, 128), ("DZ1H", bf, 128), ("Y", f8, 3),
        ("W", f8, 1), ("ROWLOSS", f8, 1))}
    assert np.array_equal(R["X"], P.bf16_round(ctx)) and np.array_equal(R["O"], out)
    assert np.array_equal(R["Y"], y) and np.array_equal(R["W"][:, 0], omega)
    check_product(R["Z1"], R["X"], W["W1"], W["b1"], "layer 1")
    check_product(R["Z2"], R["H1"], W["W2"], W["b2"], "layer 2")
    check_product(R["O"], R["H2"], W["W3"], W["b3"], "layer 3")
    for a, b in (("DO", "DOH"), ("DZ2", "DZ2H"), ("DZ1", "DZ1H")):
        assert np.array_equal(R[b], P.bf16_round(R[a].astype(np.float32))), b
    assert abs(float(loss.item()) - R["ROWLOSS"].sum()) <= 1e-12 * np.abs(R["ROWLOSS"]).sum()
    wt = P.unpack(f64(net.w))
    off = m.mxr_mlp_workspace_layout(n)[m.WS_REGIONS.index("WT")]
    t = f64(net.ws[off:off + 2 * P.N_PARAMS].view(bf))
    at = 0
    for name, i, o in (("W1", 6, 128), ("W2", 128, 128), ("W3", 128, 56)):
        assert np.array_equal(t[at:at + i * o].reshape(o, i), wt[name].T), name
        at += i * o + o
    g = P.unpack(f64(net.grad))
    for name, A, B in (("W3", R["H2"].T, R["DOH"]), ("W2", R["H1"].T, R["DZ2H"]), ("W1", R["X"].T, R["DZ1H"])):
        assert np.all(np.abs(g[name] - P.gemm_bound(A, B)[0]) <= gamma(513) * (np.abs(A) @ np.abs(B)) + 1e-40), name
    for name, D in (("b3", R["DO"]), ("b2", R["DZ2"]), ("b1", R["DZ1"])):
        assert np.all(np.abs(g[name] - D.sum(0)) <= gamma(513) * np.abs(D).sum(0) + 1e-40), name


def test_training_weights_of_many_runs(torch_cuda):  # noqa: F811
    """19 runs, two of them without rows (null images), in one call against a
    call a run: the same rows bit for bit."""
    import workloads
    torch = torch_cuda
    m = mxr()
    announce("training weights of 19 runs")
    rng = np.random.default_rng(5)
    ins = m.Instrument(workloads.edct_projection(workloads.make_phantom(64, 1), workloads.make_mu_tables(1), nx=40, ny=8,
                                                 ne=16))
    lo, hi = (np.array(v) for v in ins.proposal_box())
    sizes = rng.integers(1, 700, 19)
    sizes[[4, 18]] = 0
    first = [0] + list(np.cumsum(sizes))
    n, bins = int(first[-1]), 40 * 8 * 16
    hits = dict(ctx=torch.tensor(rng.normal(size=(n, 6)).astype(np.float32), device="cuda"),
                y=torch.tensor(lo + (hi - lo) * rng.random((n, 3)), device="cuda"),
                w=torch.tensor(rng.uniform(0.1, 2, n), device="cuda"),
                bin=torch.tensor(rng.integers(0, bins, n), device="cuda"))
    images = [torch.tensor(np.where(rng.random(bins) < 0.3, 0.0, rng.random(bins)), device="cuda") for _ in range(19)]
    net = m.ProposalNet(params(17), batch=4096)
    omega = net.train_from_runs(ins, hits, [int(v) for v in first], images, epochs=1, lr=1e-4, seed=1)
    torch.cuda.synchronize()
    for r in range(19):
        a, b = int(first[r]), int(first[r + 1])
        if b > a:
            ref = m.train_weights({"w": hits["w"][a:b], "bin": hits["bin"][a:b]}, b - a, images[r])
            assert torch.equal(omega[a:b], ref), r
