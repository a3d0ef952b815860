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


def plain_anneal(A, group_of, S, k_in, steps, t0, t1, seed):
    """The solver's own arithmetic without bounds: group sums updated per kept swap, every loss its tokens' losses added
    up in order."""
    B_tok, C = A.shape
    a = np.abs(A.astype(np.float64)).T
    g, L = np.array(group_of, np.int32), np.zeros((S, B_tok))
    for c in range(C):
        L[g[c]] += a[c]

    def loss_of(L):
        tok = np.zeros(B_tok)
        for v in np.sort(L, axis=0)[:S - k_in]:
            tok = tok + v
        return float(np.cumsum(tok)[-1])                     # one addition after the other

    loss = loss_of(L)
    for step in range(steps):
        r = [PO.splitmix64((seed + 3 * step + n) & PO.MASK) for n in range(3)]
        i, j = r[0] % C, r[1] % C
        if g[i] == g[j]:
            continue
        new = L.copy()
        new[g[i]] = L[g[i]] - a[i] + a[j]
        new[g[j]] = L[g[j]] - a[j] + a[i]
        new_loss = loss_of(new)
        delta, temp = new_loss - loss, t0 * (t1 / t0) ** (step / (steps - 1))
        if delta <= 0.0 or (r[2] >> 11) * 2.0 ** -53 < np.exp(-delta / temp):
            g[i], g[j] = g[j], g[i]
            L, loss = new, new_loss
    return g, loss


@pytest.mark.parametrize("t", [1e-300, 1e-9, 1.0])
@pytest.mark.parametrize("columns", ["twice", "equal"])
@pytest.mark.parametrize("S", [2, 3, 4, 8])
def test_decisions_that_the_order_of_a_sum_makes(t, columns, S):
    # activations of 2^-25 to 2^25, so that sums are rounded, with equal neurons, so that a loss changes by roundings only:
    # the sum in another order says something else about many of these swaps
    for seed in range(6):
        rng = np.random.default_rng(seed)
        A = rng.standard_normal((61, 24)) * 2.0 ** rng.integers(-25, 26, (61, 1))
        A[:, 12:] = A[:, :12]
        if columns == "equal":
            A[:] = A[:, :1]
        A = A.astype(np.float32)
        g0 = PO.greedy(A, S)
        ref = plain_anneal(A, g0, S, S // 2, 300, t, t, seed)
        got = B.moe_prism_partition_anneal(A, g0, S, S // 2, 300, t, t, seed)
        assert np.array_equal(got[0], ref[0]) and got[1] == ref[1]


@pytest.mark.parametrize("rows", [15, 16, 17, 256, 257])    # vectors of 16 tokens, 16 of them to a binary32 sum
@pytest.mark.parametrize("scale", [1.0, 1e-42, 1e33, 1e36])  # subnormal; below and beyond what binary32 sums may reach
@pytest.mark.parametrize("S,k_in", [(2, 1), (3, 1), (4, 2), (8, 5)])
def test_decisions_behind_a_binary32_sum(rows, scale, S, k_in):
    # hot enough to take swaps, then so cold that the binary32 bound leaves many open
    A = np.random.default_rng(rows).standard_normal((rows, 24)) * scale
    A = A.astype(np.float32)
    g0 = PO.greedy(A, S)
    for t0, t1 in ((scale, 1e-3 * scale), (1e-4 * scale, 1e-9 * scale)):
        ref = plain_anneal(A, g0, S, k_in, 250, t0, t1, rows)
        got = B.moe_prism_partition_anneal(A, g0, S, k_in, 250, t0, t1, rows)
        assert np.array_equal(got[0], ref[0]) and got[1] == ref[1]
