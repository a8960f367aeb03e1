"""Natural-order filter (§4.3, Alg. 3 without the ancilla qubit): GPU against
the oracle, including the paper's printed N = 16 example."""
import numpy as np
import pytest
import torch

from conftest import read_golden
from gpu_util import COMPLEX, TOL, host64, make_inputs, rel_err, say
from oracle import gtt_oracle as O
from paper_2507_02420_amd import gtt as G
from paper_2507_02420_amd.inputs import u3

pytestmark = pytest.mark.gpu


def test_filter_paper_example_on_gpu():
    d = read_golden("filter_example.txt")
    W = u3(np.pi / 4, 0.0, np.pi).real
    psi = np.array(d["psi"])
    psi = psi / np.linalg.norm(psi)
    x = torch.from_numpy(psi).cuda().reshape(1, 16)
    Wt = torch.from_numpy(W).cuda()
    plan = G.Plan(2, 4, 1, torch.float64)
    lo, hi = plan.filter(Wt, x, 4)
    torch.cuda.synchronize()
    np.testing.assert_allclose(lo.cpu().numpy()[0], d["low"], atol=6e-5)
    np.testing.assert_allclose(hi.cpu().numpy()[0], d["high"], atol=6e-5)
    np.testing.assert_allclose(plan.forward(Wt, x).cpu().numpy()[0], d["spectrum"], atol=6e-5)


@pytest.mark.parametrize("dtype", [torch.float32, torch.complex64, torch.float64], ids=str)
@pytest.mark.parametrize("b,n,batch,cut", [(2, 12, 3, 100), (3, 9, 2, 5000), (4, 8, 2, 1), (8, 5, 2, 32767),
                                           (2, 16, 2, 1 << 15), (4, 8, 1, 0), (4, 8, 1, 1 << 30)])
def test_filter_matches_oracle(b, n, batch, cut, dtype):
    say(f"filter b={b} n={n} cut={cut} dtype={dtype}")
    x, W, x64, W64 = make_inputs(b, n, batch, dtype, seed=1300 + b + n)
    plan = G.Plan(b, n, batch, dtype)
    lo, hi = plan.filter(W, x, cut)
    torch.cuda.synchronize()
    for i in range(batch):
        rlo, rhi = O.natural_filter(W64, x64[i], n, cut)
        scale = np.linalg.norm(x64[i])
        assert np.linalg.norm(host64(lo[i]) - rlo) / scale < 3 * TOL[dtype]
        assert np.linalg.norm(host64(hi[i]) - rhi) / scale < 3 * TOL[dtype]


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float16, torch.float32], ids=str)
@pytest.mark.parametrize("b,n,batch,cut", [(16, 3, 2, 1000), (32, 2, 3, 1), (16, 4, 1, 40000), (32, 3, 1, 0),
                                           (32, 2, 2, 1 << 20)])
def test_filter_matrix_core(b, n, batch, cut, dtype):
    # radix 16 / 32: the natural-order mask is applied while the first
    # inverse group loads its tile on the matrix-core path
    say(f"filter mfma b={b} n={n} cut={cut} dtype={dtype}")
    x, W, x64, W64 = make_inputs(b, n, batch, dtype, seed=1400 + b + n)
    plan = G.Plan(b, n, batch, dtype)
    assert all(g["kind"] == "mfma" for g in plan.describe()["groups"])
    lo, hi = plan.filter(W, x, cut)
    torch.cuda.synchronize()
    for i in range(batch):
        rlo, rhi = O.natural_filter(W64, x64[i], n, cut)
        scale = np.linalg.norm(x64[i])
        assert np.linalg.norm(host64(lo[i]) - rlo) / scale < 3 * TOL[dtype]
        assert np.linalg.norm(host64(hi[i]) - rhi) / scale < 3 * TOL[dtype]


# the filter's middle pass on the register kernel (radix 2 and 4, float32 and
# complex64): one group (the whole filter in one launch) and two, cut-offs at
# the ends and inside a tile row, either part alone; against the oracle and the
# three-transform form (which a tuned tile budget selects)
@pytest.mark.parametrize("dtype", [torch.float32, torch.complex64], ids=str)
@pytest.mark.parametrize("b,n,batch", [(2, 2, 6), (2, 7, 37), (2, 13, 3), (2, 15, 2), (2, 18, 1), (4, 1, 6), (4, 3, 65),
                                       (4, 5, 9), (4, 6, 5), (4, 7, 3), (4, 9, 1)])
def test_filter_register_middle_pass(b, n, batch, dtype):
    x, W, x64, W64 = make_inputs(b, n, batch, dtype, seed=1500 + 31 * b + n)
    N = b ** n
    scale = np.linalg.norm(x64, axis=-1).max()
    plan = G.Plan(b, n, batch, dtype)
    for cut in sorted({0, 1, N // 2, N // 3 + 1, N - 1, N, 1 << 40}):
        say(f"filter register b={b} n={n} batch={batch} cut={cut} dtype={dtype}")
        lo, hi = plan.filter(W, x, cut)
        only_lo, none = plan.filter(W, x, cut, high=False)
        none2, only_hi = plan.filter(W, x, cut, low=False)
        torch.cuda.synchronize()
        assert none is None and none2 is None
        assert torch.equal(lo, only_lo) and torch.equal(hi, only_hi)
        for i in {0, batch - 1}:
            rlo, rhi = O.natural_filter(W64, x64[i], n, cut)
            assert np.linalg.norm(host64(lo[i]) - rlo) / scale < 3 * TOL[dtype]
            assert np.linalg.norm(host64(hi[i]) - rhi) / scale < 3 * TOL[dtype]
        G.set_tuning(b, dtype, 32768, 0, 0, n=n)
        try:
            tlo, thi = G.Plan(b, n, batch, dtype).filter(W, x, cut)
        finally:
            G.set_tuning(b, dtype, 0, 0, 0, n=n)
            G.load_tuning()
        # each within 3 TOL / 10 of the exact value
        assert np.linalg.norm(host64(lo) - host64(tlo)) / np.linalg.norm(x64) < 3 * TOL[dtype] / 5
        assert np.linalg.norm(host64(hi) - host64(thi)) / np.linalg.norm(x64) < 3 * TOL[dtype] / 5


# a filter of 64 MiB and more (descending tile order in every second group, the
# middle pass among them) against the same vectors in two halves, bit for bit
@pytest.mark.parametrize("b,n,batch,dtype", [(2, 14, 1100, torch.float32), (4, 7, 552, torch.complex64),
                                             (2, 14, 552, torch.complex64), (4, 7, 552, torch.float64)], ids=str)
def test_filter_descending_tile_order(b, n, batch, dtype):
    say(f"filter descending b={b} n={n} batch={batch} dtype={dtype}")
    gen = torch.Generator(device="cuda").manual_seed(1700 + b)
    x = torch.randn(batch, b ** n, generator=gen, device="cuda", dtype=dtype)
    _, W, _, _ = make_inputs(b, 1, 1, dtype, seed=1701 + b)
    cut = b ** n // 3 + 1
    lo, hi = G.Plan(b, n, batch, dtype).filter(W, x, cut)
    q = G.Plan(b, n, batch // 4, dtype)
    parts = [q.filter(W, h.clone(), cut) for h in x.chunk(4)]
    torch.cuda.synchronize()
    assert torch.equal(lo, torch.cat([p[0] for p in parts])) and torch.equal(hi, torch.cat([p[1] for p in parts]))
    rlo, rhi = O.natural_filter(host64(W), host64(x[-1]), n, cut)
    scale = np.linalg.norm(host64(x[-1]))
    assert np.linalg.norm(host64(lo[-1]) - rlo) / scale < 3 * TOL[dtype]
    assert np.linalg.norm(host64(hi[-1]) - rhi) / scale < 3 * TOL[dtype]
