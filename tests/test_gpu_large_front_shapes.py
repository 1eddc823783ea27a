"""Large fronts (assembled, factored and solved in HBM) at the edges of their
kernels' splits, against the oracle (run on an MI355X).

Branches of c variables coupled densely to a hub of u (natural order, no
amalgamation) under an LDS budget that makes every branch and the hub large
fronts: one column, the 16-column blocks' edges and the widest large front; row
counts to either side of the 256 rows a workgroup takes, of the 512 rows a wave
keeps in flight in a dot product and of 2,048 entries of a child in flight; one
child and three. Gates as in test_gpu_large_fronts (forward and entrywise error
1e-8 at Sigma in [1e-2, 1e2]).
"""
import numpy as np
import pytest

import checks
import kktgen
from oracle import dense as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 255), (4, 252), (15, 242), (17, 496), (33, 223), (63, 64), (64, 449), (2, 2060)]


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("c,u", SHAPES)
def test_large_front_shape(c, u, k):
    from paper_2403_15913_amd import kkt
    print(f"large front c={c} u={u} k={k}", flush=True)
    pat = kktgen.hub_pattern(k, c, u, 5)
    v = kktgen.hub_values(pat, kktgen.rng_for(8, c, u), 1e-2, 1e2)
    sym = kkt.Symbolic.from_pattern(pat, ordering=kkt.ORDER_NATURAL, max_super=64, relax_small=-1, relax_frac=0.0,
                                    front_lds_max=8192)
    _, _, rows = sym.supernodes()
    assert rows[0] == c + u
    f = kkt.Factor(sym)
    f.refactor(dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), dev(v.sigma_s))
    st, bad = f.status()
    assert st == 0, bad
    x = torch.zeros(pat.n, dtype=torch.float64, device="cuda")
    f.solve(dev(v.b), x)
    checks.assert_well_conditioned(x.cpu().numpy(), D.lifted_solution(pat, v, v.b)[0], (c, u, k))
