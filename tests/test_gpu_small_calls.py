"""Calls around the points where the tile of a small call changes (8, 16, 32
and 64 points, tables read in place, then staged): whatever the tile, a point's
values are the same, so each call equals the same points in calls of 8."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("pids", ["all", [2, 21, 2, 6], [21]])
def test_every_tile_size_gives_the_same_values(pids, f32):
    g = synth.config2_grid()
    m = pdfmi.load_synth(g)
    pdfmi.load_alphas(*synth.config2_alphas())
    try:
        req = g.pids if pids == "all" else pids
        x, q2 = synth.config2_queries(n=70_001, out_fraction=0.05)
        x[:3], q2[:3] = [2.0, np.nan, 1e-12], [10.0, 10.0, 1e-3]
        x, q2 = torch.from_numpy(x).to(DEV), torch.from_numpy(q2).to(DEV)
        parts = [pdfmi.xfxq2_alphas(m, req, x[i:i + 8], q2[i:i + 8], f32=f32) for i in range(0, 4096, 8)]
        want = torch.cat([p[0] for p in parts]).cpu().numpy()
        was = torch.cat([p[1] for p in parts]).cpu().numpy()
        cu = torch.cuda.get_device_properties(0).multi_processor_count
        for n in [1, 7, 8, 9, 63, 64, 65] + [cu * 4 * t + d for t in (16, 32, 64) for d in (-1, 0, 1)]:
            out, a = [t.cpu().numpy() for t in pdfmi.xfxq2_alphas(m, req, x[:n], q2[:n], f32=f32)]
            only = (pdfmi.xfxq2_f32 if f32 else pdfmi.xfxq2)(m, req, x[:n], q2[:n]).cpu().numpy()
            k = min(n, 4096)
            assert np.array_equal(out[:k], want[:k], equal_nan=True) and np.array_equal(a[:k], was[:k], equal_nan=True)
            assert np.array_equal(only, out, equal_nan=True), n
            # the end of the call: its last tile, against the same points in a call of their own
            tail, ta = [t.cpu().numpy() for t in pdfmi.xfxq2_alphas(m, req, x[max(0, n - 70):n], q2[max(0, n - 70):n], f32=f32)]
            assert np.array_equal(out[-len(tail):], tail, equal_nan=True) and np.array_equal(a[-len(ta):], ta, equal_nan=True)
    finally:
        pdfmi.unload(m)
