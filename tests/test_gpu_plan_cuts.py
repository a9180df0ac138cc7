"""Plans around the changes of their cut: one tile per half-size workgroup, one
or several per full-size one, requests cut finer than asked for, grids in LDS
and in global memory, many members and lists between the tiles of one
workgroup, points outside the grid and invalid ones, repeated runs --
bit-identical to the per-request calls."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"
LISTS = [synth.PIDS_13, [21, 2, -2, 1, -1], [3], [6, 21, 0, 1], synth.PIDS_13[::-1]]


@pytest.mark.parametrize("policy", [0, 1])
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("n_req,n,tile", [(1, 262144, 4096), (1, 262145, 4096), (255, 512, 4096), (256, 513, 4096),
                                          (257, 1025, 4096), (511, 512, 512), (513, 512, 512), (600, 700, 256),
                                          (40, 20_001, 4096), (900, 130, 64)])
def test_cuts_equal_per_request_calls(n_req, n, tile, f64, policy):
    print("cut", n_req, n, tile, f64, policy, flush=True)
    rng = np.random.default_rng(n_req * 31 + n)
    grids = [synth.tiny_grid(rng, K=k, nx=9, nq=5, npid=13, pids=synth.PIDS_13) for k in (1, 2, 1)]
    mids = [pdfmi.load_synth(g) for g in grids]
    ev, dt, bits = (pdfmi.xfxq2, torch.float64, torch.int64) if f64 else (pdfmi.xfxq2_f32, torch.float32, torch.int32)
    try:
        g = grids[0]
        x = np.exp(rng.uniform(np.log(g.xknots[0][0]) - 0.5, 0.0, n))
        q2 = np.exp(rng.uniform(np.log(g.q2knots[0][0]) - 0.3, np.log(g.q2knots[-1][-1]) + 0.3, n))
        x[n // 3] = -1.0
        x, q2 = torch.from_numpy(x).to(DEV), torch.from_numpy(q2).to(DEV)
        pdfmi.set_lds_policy(policy)
        want, reqs = {}, []
        for i in range(n_req):
            m, pids = mids[i % 3], LISTS[(i // 2) % 5]
            if (i % 3, (i // 2) % 5) not in want:
                want[i % 3, (i // 2) % 5] = ev(m, pids, x, q2).view(bits)
            short = n - i % 3      # the requests differ in length
            reqs.append((m, pids, x[:short], q2[:short], torch.full((short, len(pids)), 7.0, dtype=dt, device=DEV)))
        plan = pdfmi.BatchPlan(reqs, out_f64=f64)
        plan.configure(tile_points=tile, vector_cols=1)
        for _ in range(3):
            for r in reqs:
                r[4].fill_(7.0)
            plan.run()
            assert all(torch.equal(r[4].view(bits), want[i % 3, (i // 2) % 5][:r[4].shape[0]])
                       for i, r in enumerate(reqs))
        plan.destroy()
    finally:
        pdfmi.set_lds_policy(0)
        for m in mids:
            pdfmi.unload(m)
