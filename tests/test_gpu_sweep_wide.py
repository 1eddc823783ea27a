"""Levels of more fronts than compute units whose panels fill a unit's LDS: the
backward sweep with only the triangle in LDS (run on an MI355X).

260 branches of c variables coupled to a hub of u: one level of 260 fronts of c
columns and c + u rows (panels over 79 KiB). At the edges of the splits (16,
32, 64 columns; odd and even row counts; rows that leave one, two or three to a
lane's first strand, and more rows than are kept in flight), the solution has
the same bits as the queue schedule's, whose backward step stages the panel,
and a backward error of at most 1e-10.
"""
import numpy as np
import pytest

import kktgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


@pytest.mark.parametrize("c,u", [(16, 641), (17, 590), (32, 290), (33, 280), (48, 171), (64, 98), (64, 101), (65, 97),
                                 (66, 103), (80, 60)])
def test_sweep_wide(c, u):
    from paper_2403_15913_amd import kkt
    print(f"wide level c={c} u={u}", flush=True)
    pat = kktgen.hub_pattern(260, c, u, 5)
    v = kktgen.hub_values(pat, kktgen.rng_for(10, c, u), 1e-2, 1e2)
    sym = kkt.Symbolic.from_pattern(pat, ordering=kkt.ORDER_NATURAL, max_super=128, relax_small=-1, relax_frac=0.0)
    _, _, rows = sym.supernodes()
    assert rows[0] == c + u
    f = kkt.Factor(sym)
    got = []
    for sched in (kkt.SCHEDULE_LEVELS, kkt.SCHEDULE_QUEUE):
        f.set_schedule(sched)
        f.refactor(dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), dev(v.sigma_s))
        st, bad = f.status()
        assert st == 0, (bad, sched)
        x = torch.zeros(pat.n, dtype=torch.float64, device="cuda")
        info = f.solve(dev(v.b), x)
        assert info["eta"] <= 1e-10, info
        got.append(x.cpu().numpy())
    np.testing.assert_array_equal(got[1], got[0])
