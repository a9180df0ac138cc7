"""Batched plans whose requests are compacted to their columns in request order
(staged in LDS in FP32, copied with the plan in FP64): every group remainder, absent and repeated flavours, requests that
share a layout, members on both sides of the compacted row width, points of
every region -- bit-identical to the per-request calls."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"
P13 = synth.PIDS_13


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float64)).to(DEV)


def requests(n_stored, rng):
    """Lists of 1..14 flavours in random order (some absent), a repeated flavour, all in order, a list twice."""
    lists = [[int(p) for p in rng.permutation(P13)[:r]] for r in (1, 2, 3, 4, 5, 7, 8, 9, 11, 12, 13)]
    lists += [[21, 1, 0], P13 + [21], P13[:n_stored], lists[4], [6], [-6, 6]]
    return lists


@pytest.mark.parametrize("n_stored", [1, 4, 11, 12, 13])
@pytest.mark.parametrize("vec", [1, 0])
@pytest.mark.parametrize("f64", [False, True])
@pytest.mark.parametrize("policy", [0, 1])
def test_layouts_equal_per_request_calls(n_stored, vec, f64, policy):
    rng = np.random.default_rng(100 + n_stored)
    grids = [synth.tiny_grid(rng, K=k, nx=9, nq=5, npid=n_stored, pids=P13[:n_stored]) for k in (1, 2)]
    mids = [pdfmi.load_synth(g) for g in grids]
    try:
        reqs = []
        for i, pids in enumerate(requests(n_stored, rng)):
            n = (1, 63, 64, 65, 700)[i % 5]
            g = grids[i % 2]
            x = np.exp(rng.uniform(np.log(g.xknots[0][0]) - 1.0, 0.0, n))
            q2 = np.exp(rng.uniform(np.log(g.q2knots[0][0]) - 1.0, np.log(g.q2knots[-1][-1]) + 1.0, n))
            if n > 1:
                x[n // 2] = -1.0
            out = torch.full((n, len(pids)), 7.0, dtype=torch.float64 if f64 else torch.float32, device=DEV)
            reqs.append((mids[i % 2], pids, dev(x), dev(q2), out))
        pdfmi.set_lds_policy(policy)
        plan = pdfmi.BatchPlan(reqs, out_f64=f64)
        plan.configure(tile_points=128, vector_cols=vec)
        bits = torch.int64 if f64 else torch.int32
        want = [(pdfmi.xfxq2 if f64 else pdfmi.xfxq2_f32)(m, pids, x, q2) for m, pids, x, q2, _ in reqs]
        for _ in range(3):   # every run leaves the tile counter as it found it
            for r in reqs:
                r[4].fill_(7.0)
            plan.run()
            for r, w in zip(reqs, want):
                assert torch.equal(r[4].view(bits), w.view(bits)), r[1]
        plan.destroy()
    finally:
        pdfmi.set_lds_policy(0)
        for m in mids:
            pdfmi.unload(m)
