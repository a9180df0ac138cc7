"""Requests served from a compacted copy of the member's values (made once
enough points have asked for the same flavours) against the same requests with
one lane per (point, flavour): bit-identical, for every group remainder, order,
absent and repeated flavours, with the copy in LDS and in global memory, with
points of every region; the first call of another stream and calls recorded
in a graph."""
import numpy as np
import pytest

from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)

from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"
N = (1 << 21) + 37          # enough points for the copy to be made by this call
LISTS = {"1": [3], "2": [2, -2], "3": [21, 1, -1], "4": [4, -4, 1, 21], "5": [21, 2, -2, 1, -1],
         "absent": [21, 6, -6, 5, 0], "reversed": synth.PIDS_13[::-1], "repeat": [21, 0, 1, 1, 2, 21, -5],
         "max": (synth.PIDS_13 * 5)[:40]}


def points(grid, n):
    if grid == "three":
        g, (x, q2) = synth.config2_grid(), synth.config2_queries(n=n, seed=5, out_fraction=0.02)
    else:
        g, (x, q2) = synth.config1_grid(), synth.config1_queries(n=n, seed=5)
        x[::50] *= 1e-3
        q2[::70] *= 1e5
    x[3], q2[5] = -1.0, np.nan
    return g, torch.from_numpy(x).to(DEV), torch.from_numpy(q2).to(DEV)


def same(a, b):
    t = torch.int64 if a.dtype == torch.float64 else torch.int32
    return torch.equal(a.view(t), b.view(t))


@pytest.mark.parametrize("grid", ["one", "three"])
@pytest.mark.parametrize("f32", [False, True])
@pytest.mark.parametrize("name", sorted(LISTS))
def test_layout_equals_general_path(grid, f32, name):
    g, x, q2 = points(grid, N if name != "max" else 300_000)
    pdfmi.load_alphas(*(synth.config2_alphas() if grid == "three" else synth.config1_alphas()))
    m = pdfmi.load_synth(g)
    ev = pdfmi.xfxq2_f32 if f32 else pdfmi.xfxq2
    try:
        pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, 0)
        pdfmi.error_count(reset=True)
        want = ev(m, LISTS[name], x, q2)
        errs = pdfmi.error_count(reset=True)
        pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, 1)
        for _ in range(1 if name != "max" else 8):
            got = ev(m, LISTS[name], x, q2)
        assert same(got, want)
        assert pdfmi.error_count(reset=True) == errs * (1 if name != "max" else 8)
        for n in (1, 65, 1000, 40_000):
            assert same(ev(m, LISTS[name], x[:n].clone(), q2[:n].clone()), want[:n])
        got, _ = pdfmi.xfxq2_alphas(m, LISTS[name], x, q2, f32=f32)
        assert same(got, want)
    finally:
        pdfmi.set_tuning(pdfmi.TUNE_VECTOR_COLUMNS, 1)
        pdfmi.unload(m)


def test_other_streams_and_capture():
    g, x, q2 = points("three", N)
    m = pdfmi.load_synth(g)
    try:
        small = slice(0, 5000)
        pids, other = [21, 2, -2, 1, -1], [1, 2, 3]
        want = pdfmi.xfxq2(m, pids, x[small].clone(), q2[small].clone())
        want_other = pdfmi.xfxq2(m, other, x, q2, out=None)  # makes this request's copy
        torch.cuda.synchronize()
        streams = [torch.cuda.Stream() for _ in range(3)]
        outs = []
        for s in streams:                                    # the first call makes the copy, the others follow it
            with torch.cuda.stream(s):
                outs.append(pdfmi.xfxq2(m, pids, x, q2))
        torch.cuda.synchronize()
        assert all(same(o, outs[0]) for o in outs) and same(outs[0][small], want)
        # recorded calls: a request with its copy made, and one whose copy may not be made while recording
        fresh = [5, 4, -4]
        out1, out2 = torch.zeros_like(want_other), torch.empty((N, 3), dtype=torch.float64, device=DEV)
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            pdfmi.xfxq2(m, other, x, q2, out=out1)
            pdfmi.xfxq2(m, fresh, x, q2, out=out2)
        for _ in range(3):
            out1.zero_()
            out2.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert same(out1, want_other)
            assert same(out2, pdfmi.xfxq2(m, fresh, x, q2))
    finally:
        pdfmi.unload(m)
