"""The solver evaluates eight tokens at a time with a sorting network per split count: token counts
that are no multiple of eight, split counts with and without a network of their own, and inner
budgets from none to all, against the reference that evaluates Eq. 4 from scratch."""
import numpy as np
import pytest

from oracle import partition_oracle as PO
from paper_2510_19366_amd import binding as B


@pytest.mark.parametrize("rows,C,S", [(1, 6, 3), (7, 8, 2), (9, 24, 12), (17, 32, 8), (3, 64, 64), (12, 5, 1)])
def test_solver_equals_reference_on_ragged_shapes(rows, C, S):
    # multiples of 2^-6: every sum is exact whatever its order, so decisions and losses must agree bit for bit
    A = (np.round(np.random.default_rng(rows + C).standard_normal((rows, C)) * 64.0) / 64.0).astype(np.float32)
    g0 = PO.greedy(A, S)
    assert np.array_equal(B.moe_prism_partition_greedy(A, S), g0)
    for k_in in sorted({0, 1, S // 2, S}):
        assert B.moe_prism_partition_objective(A, g0, S, k_in) == PO.objective(A, g0, S, k_in)
        for t in (2.0, 1e-9):                       # mostly accepting, and descending only
            ref = PO.anneal(A, g0, S, k_in, steps=200, t0=t, t1=t, seed=S)
            got = B.moe_prism_partition_anneal(A, g0, S, k_in, 200, t, t, S)
            assert np.array_equal(got[0], ref[0]) and got[1] == ref[1]


@pytest.mark.parametrize("t0,t1", [(4.0, 1e-3), (1e-3, 4.0), (0.25, 0.25)])
@pytest.mark.parametrize("equal", [False, True])
def test_decisions_inside_and_outside_the_bounds_of_an_unordered_sum(t0, t1, equal):
    # a cooling, a heating and a constant schedule; with equal activations every proposal leaves the loss as it is, which no
    # bound of a sum can tell
    rng = np.random.default_rng(3)
    A = (np.round(rng.standard_normal((13, 24)) * 64.0) / 64.0).astype(np.float32)
    if equal:
        A[:] = A[:, :1]
    g0 = PO.greedy(A, 4)
    ref = PO.anneal(A, g0, 4, 2, steps=400, t0=t0, t1=t1, seed=9)
    got = B.moe_prism_partition_anneal(A, g0, 4, 2, 400, t0, t1, 9)
    assert np.array_equal(got[0], ref[0]) and got[1] == ref[1]
