"""The kernel that writes the new population and prepares the next generation
in one pass, against the oracle generation by generation, at the sizes where
its work is cut: 512 slots (and 512 row-list entries) per workgroup,
fewer individuals than vectors (rows to spare), an odd number of offspring, an
adaptation every generation, and both sides of the rule that chooses it; and
small populations' reproduction."""
import numpy as np
import pytest

from parity import lockstep, new_stats

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def P():
    if not torch.cuda.is_available():
        pytest.skip("no HIP device")
    import paper_2404_01159_amd as P

    return P


@pytest.fixture(scope="module")
def O():
    import oracle as O

    O.lib()
    return O


# (problem, m, d, N, K): slots at the edges of one to four workgroups (any
# count is a lattice of two objectives), list entries at multiples of 512 +- 1
@pytest.mark.parametrize("shape", [(1, 2, 6, 1, 2), (1, 2, 5, 511, 512), (2, 2, 4, 512, 513), (2, 2, 5, 1023, 1023), (1, 2, 4, 1024, 1024),
                                   (3, 2, 7, 1000, 1025), (1, 2, 5, 23, 1001), (2, 3, 9, 511, 528),
                                   (1, 2, 4, 2047, 2049), (2, 8, 9, 33, 36)])
def test_turn_matches_oracle(P, O, shape):
    problem, m, d, N, K = shape
    prm = P.default_params(t_max=6, fr=1 / 6)  # adapts after every generation
    run = P.Run(problem, m, d, N, K, seed=K + N, params=prm)
    stats = lockstep(O, run, prm, 4, new_stats())
    run.close()
    assert stats["generations"] == 4
    assert stats["near_ties"] <= 1e-4 * stats["vectors"] + 1


@pytest.mark.parametrize("K", [16383, 16384, 16385])
def test_rule_edges_match_oracle(P, O, K):
    prm = P.default_params(t_max=4, fr=0.5)
    run = P.Run(1, 2, 4, K - 3, K, seed=K, params=prm)
    stats = lockstep(O, run, prm, 3, new_stats())
    run.close()
    assert stats["near_ties"] <= 1e-4 * stats["vectors"] + 1


def test_state_set_back_and_forward(P):
    """A run set back to an earlier state (either parity of the generation)
    repeats what it did, and its last offspring are not readable until then."""
    prm = P.default_params(t_max=20, fr=0.2)
    run = P.Run(2, 3, 14, 90, 105, seed=3, params=prm)
    states = [run.get_state()]
    for _ in range(7):
        run.run(1)
        states.append(run.get_state())
    for t in (5, 2, 4, 0):
        s = states[t]
        run.set_state(s["X"], s["F"], s["valid"], s["V"], s["gamma"], t)
        with pytest.raises(Exception):
            run.get_offspring()
        run.run(7 - t)
        got = run.get_state()
        for k in ("X", "F", "valid", "V", "gamma"):
            assert np.array_equal(got[k], states[7][k], equal_nan=True), (t, k)
    run.close()


# few pairs of long rows: the parts' distance sums of a child over 16 lanes,
# part counts below, at and above 16; few pairs of short rows: 16 lanes a pair
@pytest.mark.parametrize("shape", [(1, 3, 1024, 5, 6), (3, 2, 7681, 7, 8), (2, 3, 8192, 33, 36),
                                   (1, 5, 8704, 14, 15), (2, 3, 3, 9, 10), (1, 2, 17, 301, 301),
                                   (3, 4, 31, 4, 4)])
def test_few_pairs_match_oracle(P, O, shape):
    problem, m, d, N, K = shape
    prm = P.default_params(t_max=6, fr=0.5)
    run = P.Run(problem, m, d, N, K, seed=d, params=prm)
    lockstep(O, run, prm, 3, new_stats())
    run.close()


# every segment width of the reproduction kernel (4, 8, 16, 32 and 64 lanes a
# pair): the mutation sites' prefix sums and counts over 2 to 32 lanes a child,
# up to four sites a child expected
@pytest.mark.parametrize("shape", [(1, 2, 12, 4200, 4200), (2, 2, 25, 4199, 4200), (3, 2, 60, 4101, 4200),
                                   (1, 3, 100, 251, 253), (2, 3, 300, 989, 990)])
@pytest.mark.parametrize("p_m", [1.0, 4.0])
def test_segment_widths_match_oracle(P, O, shape, p_m):
    problem, m, d, N, K = shape
    prm = P.default_params(t_max=6, fr=0.5, p_m=p_m)
    run = P.Run(problem, m, d, N, K, seed=d, params=prm)
    stats = lockstep(O, run, prm, 2, new_stats())
    run.close()
    assert stats["straddles"] <= 1e-6 * stats["genes"] + 1
