"""FK contraction at the edges of its member tiles: every tile height, the
change of kernel, K around the register step and the waves' ranges."""
import numpy as np
import pytest

from oracle import fk as ofk

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"
EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("nrep", [1, 16, 17, 33, 48, 49, 64, 65, 96, 97, 112, 113])
@pytest.mark.parametrize("ndat,K", [(1, 16), (31, 15), (32, 17), (33, 64), (70, 255), (33, 1027), (100, 4099)])
def test_tiles_match_oracle(nrep, ndat, K):
    rng = np.random.default_rng(nrep * 7919 + ndat * 31 + K)
    pdf, table = rng.normal(size=(nrep, K)), rng.normal(size=(ndat, K))
    d_pdf, d_table = (torch.from_numpy(a).to(DEV) for a in (pdf, table))
    out = pdfmi.fk_contract(d_pdf, d_table)
    same = torch.full_like(out, float("nan"))
    pdfmi.fk_contract(d_pdf, d_table, out=same, noalloc=True)
    assert torch.equal(out.view(torch.int64), same.view(torch.int64))
    tol = 2.0 * K * EPS * ofk.abs_scale(pdf, table)
    assert np.all(np.abs(out.cpu().numpy() - ofk.contract(pdf, table)) <= tol)
