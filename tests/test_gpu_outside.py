"""Points outside the grid wait in a short list of their wave and are worked
off together: few and many of them per tile (the list fills up inside a tile),
one to 30 requested columns (repeated and absent ones too), tables read in
place and staged, single calls and batched plans, against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2009_06635_amd import synth
from tolerance import check_f32, check_f64, grid_L

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("fraction", [0.02, 0.3, 1.0])
@pytest.mark.parametrize("pids", [[21], [2, 6, -1], "all", [21, 1, 2, 6, 1, -1] * 5])
def test_outside_points(pids, fraction, f32):
    g = synth.config2_grid()
    m = pdfmi.load_synth(g)
    try:
        req = list(g.pids) if pids == "all" else pids
        n, k = 70_003, 600
        x, q2 = synth.config2_queries(n=n, seed=8, out_fraction=fraction)
        og = oracle.Grid(g.xknots, g.q2knots, g.values, g.pids)
        at = np.r_[0:k // 2, n - k // 2:n]
        ora, scale = oracle.xfxq2(og, req, x[at], q2[at], with_scale=True)
        xd, qd = torch.from_numpy(x).to(DEV), torch.from_numpy(q2).to(DEV)
        one = pdfmi.xfxq2_f32 if f32 else pdfmi.xfxq2
        full = one(m, req, xd, qd).cpu().numpy()
        ok = check_f32(full[at], ora, scale)[0] if f32 else check_f64(full[at], ora, scale, grid_L(g))[0]
        assert ok.all()
        # the same points in small calls, and in a plan
        ends = torch.from_numpy(at).to(DEV)
        assert np.array_equal(one(m, req, xd[ends].contiguous(), qd[ends].contiguous()).cpu().numpy(), full[at])
        out = torch.full((n, len(req)), -1.0, dtype=torch.float32 if f32 else torch.float64, device=DEV)
        plan = pdfmi.BatchPlan([(m, req, xd, qd, out)], out_f64=not f32)
        plan.run()
        assert np.array_equal(out.cpu().numpy(), full)
        plan.destroy()
    finally:
        pdfmi.unload(m)
