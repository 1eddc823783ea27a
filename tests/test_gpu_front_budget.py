"""Fronts whose blocked panel is over a small LDS budget although the analysis counts
them within it, against the oracle (run on an MI355X).

Branches of c variables coupled densely to a hub of u (natural order, no
amalgamation), the budget being what the analysis counts for the branch's front, at
least 4 KiB: one column, a column or a few past a multiple of 16, one and several
update rows.
Gates as in test_gpu_front_shapes (forward and entrywise error 1e-8 at Sigma in
[1e-2, 1e2]); the four-wave kernel, the queue schedule and the tiled update give
the same bits.
"""
import numpy as np
import pytest

import checks
import kktgen
from oracle import dense as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

SHAPES = [(1, 17), (16, 65), (17, 1), (17, 15), (17, 40), (32, 1), (33, 1), (33, 33), (49, 1), (49, 17)]


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def counted(r, c):
    cp = (c + 15) // 16 * 16
    return max((r | 1) * cp * 8 + r * 4 + 16, ((((r | 1) * c + 1) // 2 * 2) + r + c) * 8)


def blocked(r, c):
    nbc = (c + 15) // 16
    rt = 16 * (nbc + (r - c + 15) // 16)
    return 128 * (nbc * rt - 8 * nbc * (nbc - 1))


@pytest.mark.parametrize("k", [1, 4])
@pytest.mark.parametrize("c,u", SHAPES)
def test_front_budget(c, u, k):
    from paper_2403_15913_amd import kkt
    print(f"front budget c={c} u={u} k={k}", flush=True)
    budget = max(4096, counted(c + u, c))
    assert blocked(c + u, c) > budget
    pat = kktgen.hub_pattern(k, c, u, 5)
    v = kktgen.hub_values(pat, kktgen.rng_for(12, c, u), 1e-2, 1e2)
    sym = kkt.Symbolic.from_pattern(pat, ordering=kkt.ORDER_NATURAL, max_super=128, relax_small=-1, relax_frac=0.0,
                                    front_lds_max=budget)
    cols, _, rows = sym.supernodes()
    assert cols[1] == c and rows[0] == c + u and sym.stats()["large_fronts"] == 0
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
