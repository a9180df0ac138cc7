"""Grids around the LDS limit of the staged kernels, which take fewer waves per
workgroup where that lets the grid fit: bit-identical to the grid read from
global memory, for calls and plans, with points outside the grid and invalid
ones, on counts around a pass of a workgroup."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("nx,nq,P,f32", [(20, q, 13, False) for q in (18, 21, 24, 32, 40)] + [
    (50, 28, 13, True), (50, 35, 13, True), (50, 37, 11, True), (50, 46, 11, True), (50, 60, 11, True),
    (70, 72, 4, True), (70, 90, 4, True), (50, 50, 2, False)])
def test_blocks_equal_global(nx, nq, P, f32):
    print("lds block", nx, nq, P, f32, flush=True)
    rng = np.random.default_rng(nx * 100 + nq)
    xk = 10.0 ** (-6.0 + 6.0 * np.arange(nx) / (nx - 1))
    xk[-1] = 1.0
    g = synth.SynthGrid([xk], [synth.logspace_q2(1.65, 1e4, nq)], [rng.uniform(0.1, 1.0, (nx, nq, P))],
                        synth.PIDS_13[:P])
    pdfmi.load_alphas(*synth.config2_alphas())
    m = pdfmi.load_synth(g)
    ev = pdfmi.xfxq2_f32 if f32 else pdfmi.xfxq2
    bits = torch.int32 if f32 else torch.int64
    try:
        for n in (1, 767, 769, 100_003):
            x, q2 = synth.config1_queries(n=n, seed=n)
            x[::50] *= 1e-3
            q2[::70] *= 1e5
            if n > 5:
                x[3], q2[5] = -1.0, np.nan
            x, q2 = torch.from_numpy(x).to(DEV), torch.from_numpy(q2).to(DEV)
            for pids in (list(g.pids), [g.pids[-1], 6, g.pids[0]]):
                pdfmi.set_lds_policy(1)
                want = ev(m, pids, x, q2).view(bits)
                pdfmi.set_lds_policy(2)
                assert torch.equal(ev(m, pids, x, q2).view(bits), want)
                got, _ = pdfmi.xfxq2_alphas(m, pids, x, q2, f32=f32)
                assert torch.equal(got.view(bits), want)
                out = torch.zeros_like(got)
                plan = pdfmi.BatchPlan([(m, pids, x, q2, out)], out_f64=not f32)
                plan.run()
                assert torch.equal(out.view(bits), want)
                plan.destroy()
    finally:
        pdfmi.set_lds_policy(0)
        pdfmi.unload(m)
