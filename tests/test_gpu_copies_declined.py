"""PDF_TUNE_VECTOR_COLUMNS = 0 declines the copies that queries and plans keep
(device memory unchanged), with results identical to those from the copies."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


def test_declined():
    rng = np.random.default_rng(0)
    nx, nq = 200, 250
    xk = 10.0 ** (-6.0 + 6.0 * np.arange(nx) / (nx - 1))
    xk[-1] = 1.0
    g = synth.SynthGrid([xk], [synth.logspace_q2(1.65, 1e4, nq)], [rng.uniform(0.1, 1.0, (nx, nq, 13))], synth.PIDS_13)
    n = (1 << 21) + 1
    x, q2 = (torch.from_numpy(a).to(DEV) for a in synth.config1_queries(n=n, seed=1))
    outs = [torch.empty((n, 13), dtype=torch.float64, device=DEV) for _ in range(6)]
    pids = synth.PIDS_13[::-1]
    m = pdfmi.load_synth(g)
    try:
        used = []
        for k, vec in enumerate((0, 0, 1)):   # the first launches make the runtime allocate memory of its own
            pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, vec)
            before = torch.cuda.mem_get_info()[0]
            plan = pdfmi.BatchPlan([(m, pids, x, q2, outs[2 * k])], out_f64=True)
            plan.run()
            pdfmi.xfxq2(m, pids, x, q2, out=outs[2 * k + 1])
            torch.cuda.synchronize()
            used.append(before - torch.cuda.mem_get_info()[0])
            plan.destroy()
        assert used[1] < 4 << 20                 # tables of the plan only
        assert used[2] >= used[1] + (10 << 20)   # two copies of 50000 rows of 128 bytes
        assert all(torch.equal(o, outs[0]) for o in outs[1:])
    finally:
        pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, 1)
        pdfmi.unload(m)
