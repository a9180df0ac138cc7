"""A query on one stream, served from a compacted copy that is not known to be
complete yet, while another stream records a graph in the mode that forbids
most calls of every thread: the query succeeds and the recording stays whole."""
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"


@pytest.mark.parametrize("made", [True, False])
def test_query_beside_a_recording(made):
    g = synth.config2_grid()
    n = (1 << 21) + 5
    x, q2 = (torch.from_numpy(a).to(DEV) for a in synth.config2_queries(n=n, seed=11))
    pids, pids2 = [21, 2, -2, 1, -1], [1, 2]
    m = pdfmi.load_synth(g)
    try:
        want, want2 = (pdfmi.xfxq2(m, p, x[:4096].clone(), q2[:4096].clone()) for p in (pids, pids2))
        out, rec = torch.zeros((n, 5), dtype=torch.float64, device=DEV), torch.zeros((4096, 2), dtype=torch.float64, device=DEV)
        xs, qs = x[:4096].clone(), q2[:4096].clone()
        side = torch.cuda.Stream()
        if made:                       # the copy is made here; nothing has looked at its event since
            pdfmi.xfxq2(m, pids, x, q2, out=out)
        torch.cuda.synchronize()
        out.zero_()
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, capture_error_mode="global"):
            pdfmi.xfxq2(m, pids2, xs, qs, out=rec)
            pdfmi.xfxq2(m, pids, x, q2, out=out, stream=side)
        torch.cuda.synchronize()
        assert torch.equal(out[:4096], want)
        for _ in range(2):
            rec.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(rec, want2)
    finally:
        pdfmi.unload(m)
