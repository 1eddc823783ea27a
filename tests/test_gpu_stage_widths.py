"""Stage widths at the edges of the stage-structured solver's triangular
substitutions (blocks of 16 columns; a lane's second row from 65 on), against
the oracle (run on an MI355X). Seven stages: chains of one, two and three left
over on the levels. Gates as in test_gpu_stagewise (backward error 1e-10,
forward error 1e-8 entry by entry at Sigma in [1e-2, 1e2]).
"""
import numpy as np
import pytest

import checks
import kktgen
from oracle import dense as D
from oracle import sparse as S

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("width", [3, 15, 16, 17, 49, 63, 64, 65, 67, 79, 80])
def test_stage_width(width):
    from paper_2403_15913_amd import kkt
    print(f"stage width {width}", flush=True)
    pat = kktgen.nmpc_pattern(7, width - 1, 1)
    v = kktgen.nmpc_values(pat, kktgen.rng_for(9, width), 1e-2, 1e2)
    s = pat.meta["stage"] if "stage" in pat.meta else width
    W = kkt.Stagewise([kkt.Symbolic.from_pattern(pat)], [np.arange(0, pat.n + 1, s, dtype=np.int32)])
    W.refactor(dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), dev(v.sigma_s))
    st, bad = W.status()
    assert (st == 0).all(), (st, bad)
    x = torch.zeros(pat.n, dtype=torch.float64, device="cuda")
    infos = W.solve(dev(v.b), x, tol=1e-14)
    xq = x.cpu().numpy()
    be = D.backward_errors(D.condensed(pat, v, v.sigma_s), xq, v.b)
    assert be["eta"] <= 1e-10 and infos[0]["eta"] <= 1e-10, (be, infos)
    xo, oinfo = S.lifted_solve(pat, v, v.b)
    assert oinfo["spd"]
    checks.assert_well_conditioned(xq, xo, width)
