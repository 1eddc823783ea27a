"""Columns of J around the lengths where the J^T v kernels change hands,
against the oracle (run on an MI355X).

Each row of J holds a variable of its own and the shared variables whose
column is longer than the row's number, so the shared columns hold exactly the
lengths listed: up to 8 entries go to one lane, more to a 16-lane group that
takes 64 entries a round. HyKKT (gamma 1e4; f_gamma, the CG direction, the dx
right-hand side) and the augmented solve at Sigma in [1e-2, 1e2], within 1e-8
of the saddle-point and augmented-system solutions, as in
test_gpu_random_patterns and test_gpu_inertia_augmented.
"""
import numpy as np
import pytest

import checks
import kktgen
from oracle import dense as D

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

LENGTHS = [[8], [9], [7, 8, 9, 10], [15, 16, 17], [63, 64, 65], [80, 81, 128, 129]]


def dev(a):
    return torch.tensor(np.asarray(a), dtype=torch.float64, device="cuda")


def pattern(lengths):
    m = max(lengths)
    n = m + len(lengths)
    rows = [np.array([r] + [m + s for s, ln in enumerate(lengths) if r < ln]) for r in range(m)]
    rp = np.concatenate([[0], np.cumsum([len(r) for r in rows])]).astype(np.int32)
    return kktgen.Pattern(n, m, np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), rp,
                          np.concatenate(rows).astype(np.int32))


@pytest.mark.parametrize("lengths", LENGTHS, ids=[str(x) for x in LENGTHS])
def test_long_columns(lengths):
    from paper_2403_15913_amd import kkt
    pat = pattern(lengths)
    v = kktgen.general_values(pat, kktgen.rng_for(7, len(lengths), max(lengths)), 1e-2, 1e2)
    f = kkt.Factor(kkt.Symbolic.from_pattern(pat))
    x, y, z = (torch.zeros(k, dtype=torch.float64, device="cuda") for k in (pat.n, pat.m, pat.m))
    f.refactor(dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), None, 1e4)
    info = f.cg_schur(dev(v.f), dev(v.g), x, y, tol=1e-12)
    assert info["status"] == 0, info
    dx, dy, _ = D.hykkt_solution(pat, v, v.f, v.g, 0.0)
    assert D.forward_error(x.cpu().numpy(), dx) <= 1e-8 and D.forward_error(y.cpu().numpy(), dy) <= 1e-8
    f.keep_augmented(True)
    f.refactor(dev(v.w_vals), dev(v.j_vals), dev(v.sigma_x), dev(v.sigma_s))
    r4 = np.flip(v.g).copy()
    assert f.solve_augmented(dev(v.f), dev(v.g), dev(r4), x, y, z)["status"] == 0
    want = np.linalg.solve(D.lifted_augmented(pat, v), -np.concatenate([v.f, v.g, r4]))
    for got, ref in ((x, want[:pat.n]), (y, want[pat.n:pat.n + pat.m]), (z, want[pat.n + pat.m:])):
        checks.assert_well_conditioned(got.cpu().numpy(), ref, lengths)
