"""Sweep launches on either side of 512 fronts a level, in a tree with taller fronts
(run on an MI355X).

Leaves of c variables, each coupled to u variables of a dense hub of 150: one
level of 511 or 512 fronts of at most 128 rows and light panels, below the hub's
fronts. From 512 on the level takes the one-wave forward kernel and, where the
hub's panel fills the LDS, the four-wave backward kernel; below that the hub's forms. The solution has the same bits as the
queue schedule's, which has one form, and a backward error of at most 1e-10.
"""
import numpy as np
import pytest

import kktgen

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

HUB = 150


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def pattern(leaves, c, u):
    hub0, n = leaves * c, leaves * c + HUB
    w_rows = [np.arange(q * c, q * c + r + 1) for q in range(leaves) for r in range(c)]
    w_rows += [np.arange(hub0, hub0 + r + 1) for r in range(HUB)]
    j_rows = [np.concatenate([np.arange(q * c, (q + 1) * c), hub0 + (5 * q) % (HUB - u) + np.arange(u)])
              for q in range(leaves)]

    def csr(rows):
        ptr = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
        return ptr, np.concatenate(rows).astype(np.int32)

    return kktgen.Pattern(n, leaves, *csr(w_rows), *csr(j_rows))


@pytest.mark.parametrize("c,u", [(4, 3), (17, 111), (40, 25)])
@pytest.mark.parametrize("leaves", [511, 512])
def test_sweep_many(leaves, c, u):
    from paper_2403_15913_amd import kkt
    print(f"{leaves} leaves of {c} x {c + u}", flush=True)
    pat = pattern(leaves, c, u)
    v = kktgen.general_values(pat, kktgen.rng_for(15, c, u), 1e-2, 1e2)
    sym = kkt.Symbolic.from_pattern(pat, ordering=kkt.ORDER_NATURAL, max_super=128, relax_small=-1, relax_frac=0.0)
    cols, _, rows = sym.supernodes()
    assert (rows[:leaves] == c + u).all() and (np.diff(cols)[:leaves] == c).all() and rows[leaves:].max() > 128
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
