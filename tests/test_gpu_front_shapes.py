"""Dense fronts at the edges of the front kernel's tiles, against the oracle
(run on an MI355X).

One branch of c variables coupled densely to a hub of u (natural order, no
amalgamation): the branch's supernode is a front of c columns and c + u rows,
then the hub's own. Sizes: one column, multiples of 16 and one to either
side, the widest supernode, the tallest fronts whose panel the panel waves of
the four- and eight-or-more-wave kernels cover (208 and 272 rows once columns
and update rows are padded to 16) and one row past them. With four branches
the hub's front has four children. Gates as in test_gpu_random_patterns
(forward and entrywise error 1e-8 at Sigma in [1e-2, 1e2]); the four-wave
kernel, the queue schedule and the tiled update give the same bits.
"""
import numpy as np
import pytest

import checks
import kktgen
from oracle import dense as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 1), (1, 33), (15, 17), (16, 16), (17, 15), (31, 48), (33, 47), (48, 160), (48, 161), (64, 1),
          (32, 240), (32, 241), (90, 60), (96, 100), (128, 15)]


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("k", [1, 4])
@pytest.mark.parametrize("c,u", SHAPES)
def test_front_shape(c, u, k):
    from paper_2403_15913_amd import kkt
    pat = kktgen.hub_pattern(k, c, u, 5)
    v = kktgen.hub_values(pat, kktgen.rng_for(6, c, u), 1e-2, 1e2)
    sym = kkt.Symbolic.from_pattern(pat, ordering=kkt.ORDER_NATURAL, max_super=128, relax_small=-1, relax_frac=0.0)
    cols, _, rows = sym.supernodes()
    assert cols[1] == c and rows[0] == c + u, (cols[:3], rows[:3])
    f = kkt.Factor(sym)
    xs, got = D.lifted_solution(pat, v, v.b)[0], []
    for small, split, sched in ((0, (140, 64), kkt.SCHEDULE_LEVELS), (128, (140, 64), kkt.SCHEDULE_LEVELS),
                                (0, (0, 0), kkt.SCHEDULE_LEVELS), (128, (0, 0), kkt.SCHEDULE_LEVELS),
                                (0, (0, 0), kkt.SCHEDULE_QUEUE)):
        f.set_small_fronts(small)
        f.set_update_split(*split)
        f.set_schedule(sched)
        f.refactor(dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), dev(v.sigma_s))
        st, bad = f.status()
        assert st == 0, (bad, small, split, sched)
        x = torch.zeros(pat.n, dtype=torch.float64, device="cuda")
        f.solve(dev(v.b), x)
        got.append(x.cpu().numpy())
    checks.assert_well_conditioned(got[0], xs, (c, u, k))
    for g in got[1:]:
        np.testing.assert_array_equal(g, got[0])
