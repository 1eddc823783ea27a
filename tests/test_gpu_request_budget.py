"""The memory that one served request takes does not grow: servers whose budget
held exactly one request register the pattern and serve it (run on an MI355X).

The figures are arena bytes of one request (values, panels, update matrices,
descriptors, staging) for stages of four to nine variables under the default
analysis; a budget below what a request takes is refused with BUDGET.
"""
import numpy as np
import pytest

import kktgen
from oracle import dense as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

REQUESTS = [(3, 3, 1, 12800), (10, 3, 1, 25600), (50, 8, 1, 387328)]


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("N,nx,nu,need", REQUESTS)
def test_request_fits_its_budget(N, nx, nu, need):
    from paper_2403_15913_amd import kkt
    pat = kktgen.nmpc_pattern(N, nx, nu)
    v = kktgen.nmpc_values(pat, kktgen.rng_for(11, N), 1e-2, 1e2)
    srv = kkt.Server(hbm_budget=need, max_wave=4, workers=1)
    pid = srv.register(kkt.Symbolic.from_pattern(pat))
    x = torch.zeros(pat.n, dtype=torch.float64, device="cuda")
    res = srv.wait(srv.submit(pid, dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), dev(v.sigma_s), dev(v.b), x))
    assert res["status"] == 0, res
    be = D.backward_errors(D.condensed(pat, v, v.sigma_s), x.cpu().numpy(), v.b)
    assert be["eta"] <= 1e-10, be
    srv.close()
