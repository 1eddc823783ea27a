"""The shapes of test_gpu_large_front_shapes are large fronts under its LDS budget
(no GPU): the k branches and the hub's first chunk of 64 columns. (The hub's last
rows may fit the budget at one column and then go to the LDS kernels.)
"""
import numpy as np
import pytest

import kktgen
import test_gpu_large_front_shapes as shapes
from test_abi_cpu import _front_lds

BUDGET = 8192


@pytest.mark.parametrize("k", [1, 3])
@pytest.mark.parametrize("c,u", shapes.SHAPES)
def test_shapes_are_large_fronts(c, u, k):
    from paper_2403_15913_amd import kkt
    sym = kkt.Symbolic.from_pattern(kktgen.hub_pattern(k, c, u, 5), ordering=kkt.ORDER_NATURAL, max_super=64,
                                    relax_small=-1, relax_frac=0.0, front_lds_max=BUDGET)
    cols, _, rows = sym.supernodes()
    width = np.diff(cols)
    large = [_front_lds(int(r), int(w)) > BUDGET for r, w in zip(rows, width)]
    assert rows[:k].tolist() == [c + u] * k and width[:k].tolist() == [c] * k
    assert all(large[:k + 1]) and sum(large) == sym.stats()["large_fronts"] >= k + 1
    assert width[k] == min(64, u + 5)
