"""Which requests get a compacted copy: one that is asked for at many points
gets it after any number of other small requests on the same member."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


def test_copy_after_many_small_requests():
    rng = np.random.default_rng(0)
    nx, nq = 200, 250
    xk = 10.0 ** (-6.0 + 6.0 * np.arange(nx) / (nx - 1))
    xk[-1] = 1.0
    g = synth.SynthGrid([xk], [synth.logspace_q2(1.65, 1e4, nq)], [rng.uniform(0.1, 1.0, (nx, nq, 13))], synth.PIDS_13)
    n = (1 << 20) + 1
    x, q2 = (torch.from_numpy(a).to(DEV) for a in synth.config1_queries(n=n, seed=1))
    out = torch.empty((n, 13), dtype=torch.float64, device=DEV)
    m = pdfmi.load_synth(g)
    try:
        pids = synth.PIDS_13[::-1]                    # its copy: 50000 rows of 128 bytes
        for i in range(100):
            pdfmi.xfxq2(m, [int(p) for p in rng.permutation(synth.PIDS_13)[:1 + i % 12]], x[:1].clone(), q2[:1].clone())
        torch.cuda.synchronize()
        free = []
        for _ in range(4):
            pdfmi.xfxq2(m, pids, x, q2, out=out)
            torch.cuda.synchronize()
            free.append(torch.cuda.mem_get_info()[0])
        assert free[0] - free[1] >= 6 << 20           # made by the second call of 2^20 points
        assert free[1] == free[2] == free[3]          # and once only
    finally:
        pdfmi.unload(m)
