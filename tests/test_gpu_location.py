"""Point location at the ends of its ranges: arguments whose ratio to a knot is
subnormal, zero or beyond the FP64 range, and location tables near and beyond
the size the fused Monte-Carlo kernel can hold in LDS."""
import numpy as np
import pytest

import oracle
from paper_2009_06635_amd import synth
from tolerance import check_f64, describe_failures, grid_L

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float64)).to(DEV)


@pytest.mark.parametrize("K", [1, 3])
def test_extreme_arguments(K):
    """Negative values take the linear continuations, whose error scale is the oracle's."""
    rng = np.random.default_rng(31 + K)
    g = synth.tiny_grid(rng, K=K, nx=7, nq=5, npid=3)
    g = g.with_values([-1.0 - np.abs(v) for v in g.values])
    xs = [5e-324, 1e-320, 1e-310, 2.3e-308, 1e-300, 1e-30, g.xknots[0][0], 0.3, 1.0]
    qs = [5e-324, 1e-310, 2.3e-308, 1e-20, g.q2knots[0][0], 5.0, g.q2knots[-1][-1], 1e30, 1e300, 1.7e308]
    x, q2 = (np.array(a).ravel() for a in np.meshgrid(xs, qs))
    m = pdfmi.load_synth(g)
    try:
        ora, scale = oracle.xfxq2(oracle.Grid(g.xknots, g.q2knots, g.values, g.pids), g.pids, x, q2, with_scale=True)
        out = pdfmi.xfxq2(m, g.pids, dev(x), dev(q2)).cpu().numpy()
        ok, _, _ = check_f64(out, ora, scale, grid_L(g))
        assert ok.all(), describe_failures(ok, out, ora, x, q2, g.pids)
    finally:
        pdfmi.unload(m)


@pytest.mark.parametrize("nx", [400, 2600, 2620, 2640, 2680, 4000])
@pytest.mark.parametrize("f32", [False, True])
def test_fused_sum_with_large_tables(nx, f32):
    """Tables in LDS, tables read from global memory, and tables refused: the
    accepted sums equal the separate calls' bit for bit."""
    rng = np.random.default_rng(nx)
    xk = np.exp(np.linspace(np.log(1e-5), 0.0, nx))
    xk[-1] = 1.0
    qk = np.array([2.0, 4.0, 9.0, 30.0, 90.0])
    m = pdfmi.load_grid([xk], [qk], [rng.uniform(-1.0, 2.0, (nx, 5, 2))], [21, 1])
    pdfmi.load_alphas(*synth.config1_alphas())
    try:
        x1, x2 = (dev(np.exp(rng.uniform(np.log(1e-6), 0.0, 5000))) for _ in range(2))
        q2 = dev(np.exp(rng.uniform(0.0, 6.0, 5000)))
        ev = pdfmi.xfxq2_f32 if f32 else pdfmi.xfxq2
        ref = pdfmi.mc_chunk_sum(ev(m, [21, 1], x1, q2), ev(m, [21, 1], x2, q2), pdfmi.alphas_q2(q2))
        try:
            s = pdfmi.mc_fused(m, [21, 1], x1, x2, q2, f32=f32)
        except pdfmi.PdfError as e:
            assert e.code == pdfmi.PDF_ERR_GRID and nx >= 2680
        else:
            assert nx <= 2640
            assert torch.equal(s.view(torch.int64), ref.view(torch.int64))
    finally:
        pdfmi.unload(m)
