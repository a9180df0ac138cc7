"""FK contraction around the size of table and the member counts at which the
kernel changes, against FP64 matrix products."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("needs a GPU", allow_module_level=True)
from paper_2009_06635_amd import pdfmi  # noqa: E402

DEV = "cuda:0"
EPS = np.finfo(np.float64).eps


@pytest.mark.parametrize("ndat,K", [(1023, 32249), (1023, 32263), (4099, 8192), (4020, 8192), (1433, 31395), (1434, 31395)])
def test_large_tables(ndat, K):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(ndat + K)
    table = torch.randn((ndat, K), dtype=torch.float64, device=DEV, generator=gen)
    for nrep in (16, 24, 25, 48, 49, 65, 80, 81, 112):
        print("fk table", nrep, ndat, K, flush=True)
        pdf = torch.randn((nrep, K), dtype=torch.float64, device=DEV, generator=gen)
        want = torch.mm(pdf, table.t())
        tol = 2.0 * 2.0 * K * EPS * torch.mm(pdf.abs(), table.abs().t())   # both sums within K eps of sum |a b|
        got = pdfmi.fk_contract(pdf, table)
        assert bool(((got - want).abs() <= tol).all())
        same = torch.full_like(got, float("nan"))
        pdfmi.fk_contract(pdf, table, out=same, noalloc=True)
        assert torch.equal(got.view(torch.int64), same.view(torch.int64))
