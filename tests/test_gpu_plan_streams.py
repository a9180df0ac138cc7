"""Runs of one plan on two streams, with more tiles than workgroups and with
fewer: every run evaluates every tile, whatever the other run does."""
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("n", [1000, 70_001])
def test_runs_on_two_streams(n, graph):
    g = synth.config1_grid()
    m = pdfmi.load_synth(g)
    try:
        x, q2 = [torch.from_numpy(a).to(DEV) for a in synth.config1_queries(n=n, seed=3)]
        want = pdfmi.xfxq2_f32(m, g.pids, x, q2)
        out = torch.empty_like(want)
        plan = pdfmi.BatchPlan([(m, g.pids, x, q2, out)])
        plan.configure(tile_points=64, vector_cols=1, use_graph=graph)
        s = [torch.cuda.Stream(), torch.cuda.Stream()]
        for k in range(4):
            out.fill_(-1.0)
            torch.cuda.synchronize()
            for i in range(3):
                plan.run(stream=s[(i + k) % 2])
            torch.cuda.synchronize()
            assert torch.equal(out, want), k
        plan.destroy()
    finally:
        pdfmi.unload(m)
