"""Compacted copies of grids around the LDS limit, where packed rows fit and
rows of whole 16-byte groups do not: bit-identical to one lane per (point,
flavour), with and without alpha_s behind the staged rows."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"
N = (1 << 21) + 37   # enough points for the copy to be made by this call


@pytest.mark.parametrize("nx,nq,n_cols,f32", [
    (40, 30, 5, False), (41, 29, 5, False), (50, 36, 3, False), (50, 40, 9, True), (41, 41, 9, True),
    (57, 57, 1, False), (71, 73, 1, True), (70, 70, 2, True), (70, 70, 3, True)])
def test_rows_around_the_lds_limit(nx, nq, n_cols, f32):
    print("rows", nx, nq, n_cols, f32, flush=True)
    rng = np.random.default_rng(nx * 100 + nq)
    xk = 10.0 ** (-6.0 + 6.0 * np.arange(nx) / (nx - 1))
    xk[-1] = 1.0
    qk = synth.logspace_q2(1.65, 1e4, nq)
    g = synth.SynthGrid([xk], [qk], [rng.uniform(0.1, 1.0, (nx, nq, 13))], synth.PIDS_13)
    pids = [int(p) for p in rng.permutation(synth.PIDS_13)[:n_cols]]
    x, q2 = synth.config1_queries(n=N, seed=7)
    x[::50] *= 1e-3
    q2[::70] *= 1e5
    x[3], q2[5] = -1.0, np.nan
    x, q2 = torch.from_numpy(x).to(DEV), torch.from_numpy(q2).to(DEV)
    pdfmi.load_alphas(*synth.config1_alphas())
    m = pdfmi.load_synth(g)
    ev = pdfmi.xfxq2_f32 if f32 else pdfmi.xfxq2
    bits = torch.int32 if f32 else torch.int64
    try:
        pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, 0)
        want = ev(m, pids, x, q2)
        alphas = pdfmi.alphas_q2(q2)
        pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, 1)
        for _ in range(2):
            assert torch.equal(ev(m, pids, x, q2).view(bits), want.view(bits))
        got, al = pdfmi.xfxq2_alphas(m, pids, x, q2, f32=f32)
        assert torch.equal(got.view(bits), want.view(bits))
        assert torch.equal(al.view(torch.int64), alphas.view(torch.int64))
    finally:
        pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, 1)
        pdfmi.unload(m)
