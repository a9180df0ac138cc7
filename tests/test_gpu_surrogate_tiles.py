"""Fused surrogate inference at the edges of its 64-point tiles and 32-point
sub-tiles, for an even and an odd number of envelope knots (the envelope is
read 16 bytes at a time), with repeated, absent and more than 16 requested
flavours: network points against the FP64 network within the bound of the
operand splits, fallback points equal to the FP32 interpolator bit for bit."""
import numpy as np
import pytest

from oracle import mlp
from paper_2009_06635_amd import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402
from test_gpu_surrogate import dev, envelope, forward_bound, normalise, trusted_mask  # noqa: E402


@pytest.mark.parametrize("nx", [12, 13])
@pytest.mark.parametrize("n", [1, 16, 31, 32, 33, 64, 65, 1000])
def test_inference_tile_edges(n, nx):
    rng = np.random.default_rng(100 * n + nx)
    g = synth.tiny_grid(rng, nx=nx, nq=9, npid=5)
    m = pdfmi.load_synth(g)
    s = pdfmi.Surrogate(m, seed=4)
    try:
        p = rng.normal(0, 0.3, mlp.NPARAMS).astype(np.float32)
        s.set_params(p)
        x = synth.loguniform(rng, g.xknots[0][0], g.xknots[0][-1], n)
        q2 = synth.loguniform(rng, g.q2knots[0][0], g.q2knots[0][-1], n)
        req = [g.pids[j] for j in (3, 0, 3)] + [next(q for q in synth.PIDS_13 if q not in g.pids)] + list(g.pids) * 3
        out = s.xfxq2(dev(x), dev(q2), req).cpu().numpy()
        ref = pdfmi.xfxq2_f32(m, req, dev(x), dev(q2)).cpu().numpy()
        tm = trusted_mask(g, x, q2)
        assert np.array_equal(out[~tm], ref[~tm])
        inp = normalise(g, x, q2).astype(np.float64)
        y = mlp.forward_device(p.astype(np.float64), inp)
        bound = forward_bound(p.astype(np.float64), inp, y)
        E, Es = envelope(g, x, with_scale=True)
        for j, pid in enumerate(req):
            if pid not in g.pids:
                assert np.all(out[:, j] == 0.0)
                continue
            c = g.pids.index(pid)
            assert np.all(np.abs(out[:, j] - y[:, c] * E[:, c])[tm] <= (bound[:, c] * Es[:, c])[tm]), pid
    finally:
        s.destroy()
        pdfmi.unload(m)
