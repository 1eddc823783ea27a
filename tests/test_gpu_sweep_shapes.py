"""Dense fronts at the edges of the sweep kernels' splits, against the oracle
(run on an MI355X).

Branches of c variables coupled densely to a hub of u rows (natural order, no
amalgamation): fronts of c columns and c + u rows, and a hub front with k
children. Sizes to either side of 64 and 128 columns (one or two columns per
lane in the backward substitution, four or two lanes per dot product), of 128,
256 and 512 rows (rows held by one, two and four waves, and the rows past
them), an odd and an even number of rows (a lane holds two), and one, three and
five children (two at a time). Gates as in test_gpu_random_patterns (forward
and entrywise error 1e-8 at Sigma in [1e-2, 1e2]); the queue schedule gives
the same bits.
"""
import numpy as np
import pytest

import checks
import kktgen
from oracle import dense as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 126), (1, 128), (3, 520), (5, 252), (16, 239), (16, 241), (17, 14), (31, 97), (32, 97), (63, 65),
          (64, 64), (65, 63), (66, 66), (81, 40), (112, 17), (127, 1), (128, 2)]


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("k", [1, 3, 5])
@pytest.mark.parametrize("c,u", SHAPES)
def test_sweep_shape(c, u, k):
    from paper_2403_15913_amd import kkt
    print(f"sweep shape c={c} u={u} k={k}", flush=True)
    pat = kktgen.hub_pattern(k, c, u, 5)
    v = kktgen.hub_values(pat, kktgen.rng_for(7, c, u), 1e-2, 1e2)
    sym = kkt.Symbolic.from_pattern(pat, ordering=kkt.ORDER_NATURAL, max_super=128, relax_small=-1, relax_frac=0.0)
    _, _, rows = sym.supernodes()
    assert rows[0] == c + u
    f = kkt.Factor(sym)
    xs, got = D.lifted_solution(pat, v, v.b)[0], []
    for sched in (kkt.SCHEDULE_LEVELS, kkt.SCHEDULE_QUEUE):
        f.set_schedule(sched)
        f.refactor(dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), dev(v.sigma_s))
        st, bad = f.status()
        assert st == 0, (bad, sched)
        x = torch.zeros(pat.n, dtype=torch.float64, device="cuda")
        f.solve(dev(v.b), x)
        got.append(x.cpu().numpy())
    checks.assert_well_conditioned(got[0], xs, (c, u, k))
    np.testing.assert_array_equal(got[1], got[0])
