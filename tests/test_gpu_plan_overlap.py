"""Overlapping runs of one plan: the outputs of a run are complete when its
own stream has passed it, whatever the other run does.  The plan's cheap tiles
come first and its few costly ones (points outside the grid) last: a run that
shared its tiles with the other would end while the other still evaluates
them.  Recorded runs the same, more of them than keep a counter."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


def requests(m, g, f64, tile):
    """About 600 tiles inside the grid, then 300 a little smaller outside it."""
    reqs, want = [], []
    for k, n in enumerate((600 * tile, 300 * (tile - 64))):
        x, q2 = synth.config1_queries(n=n, seed=3 + k)
        if k == 1:
            x *= 1e-7
        x, q2 = torch.from_numpy(x).to(DEV), torch.from_numpy(q2).to(DEV)
        w = (pdfmi.xfxq2 if f64 else pdfmi.xfxq2_f32)(m, g.pids, x, q2)
        for i in range(1 if k == 0 else 300):
            s = slice(None) if k == 0 else slice(i * (tile - 64), (i + 1) * (tile - 64))
            reqs.append((m, g.pids, x[s], q2[s], torch.empty_like(w[s])))
            want.append(w[s])
    return reqs, want


@pytest.mark.parametrize("graph", [0, 1])
@pytest.mark.parametrize("f64", [True, False])
def test_outputs_complete_on_each_stream(f64, graph):
    print("overlap f64=%s graph=%d" % (f64, graph), flush=True)
    g = synth.config1_grid()
    m = pdfmi.load_synth(g)
    try:
        reqs, want = requests(m, g, f64, 4096)
        plan = pdfmi.BatchPlan(reqs, out_f64=f64)
        plan.configure(tile_points=4096, vector_cols=1, use_graph=graph)
        streams = [torch.cuda.Stream() for _ in range(10)]
        for pair in ((0, 1), (1, 0), *((k, k + 1) for k in range(2, 9))):
            for r in reqs:
                r[4].fill_(-1.0)
            torch.cuda.synchronize()
            got = []
            for k in pair:
                plan.run(stream=streams[k])
                with torch.cuda.stream(streams[k]):
                    got.append([r[4].clone() for r in reqs])
            torch.cuda.synchronize()
            for outs in got:
                assert all(torch.equal(o, w) for o, w in zip(outs, want)), pair
        plan.destroy()
    finally:
        pdfmi.unload(m)


def test_recorded_runs():
    """Two recorded runs replayed on two streams beside direct runs; then more recorded runs than keep a counter."""
    g = synth.config1_grid()
    m = pdfmi.load_synth(g)
    try:
        reqs, want = requests(m, g, True, 128)
        plan = pdfmi.BatchPlan(reqs, out_f64=True)
        plan.configure(tile_points=128, vector_cols=1, use_graph=0)
        graphs = []
        for _ in range(2):
            graphs.append(torch.cuda.CUDAGraph())
            with torch.cuda.graph(graphs[-1]):
                plan.run()
        streams = [torch.cuda.Stream() for _ in range(3)]
        for _ in range(3):
            for r in reqs:
                r[4].fill_(-1.0)
            torch.cuda.synchronize()
            got = []
            for k, s in enumerate(streams):
                with torch.cuda.stream(s):
                    graphs[k].replay() if k < 2 else plan.run(stream=s)
                    got.append([r[4].clone() for r in reqs])
            torch.cuda.synchronize()
            for outs in got:
                assert all(torch.equal(o, w) for o, w in zip(outs, want))
        many = torch.cuda.CUDAGraph()
        with torch.cuda.graph(many):
            for _ in range(1100):
                plan.run()
        for r in reqs:
            r[4].fill_(-1.0)
        many.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(r[4], w) for r, w in zip(reqs, want))
        plan.destroy()
    finally:
        pdfmi.unload(m)
