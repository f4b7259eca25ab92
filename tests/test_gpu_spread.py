"""The crossover's spread factor over the distribution indices whose power is
a product (eta_c + 1 an integer up to 64): children against the oracle's, gene
by gene, in a box wide enough that no child is clipped, so that the rare
variates next to 0, 1/2 and 1 (spreads far from one) show in the genes."""
import numpy as np
import pytest

from parity import gene_mismatches, ora_params

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


# 1,024 pairs of 4,096 genes: 4 million variates of 24 bits, so spreads up to
# (2^23)^(1/(eta_c + 1)) / 4 or so are met
@pytest.mark.parametrize("eta_c,batched", [(0, False), (1, False), (1, True), (2, False), (3, True),
                                           (4, False), (5, False), (6, False), (7, False),
                                           (20, False), (20, True), (63, False)])
def test_children_match_oracle(P, O, eta_c, batched):
    K, d, seed = 2048, 4096, 40 + eta_c
    prm = P.default_params(t_max=10, fr=0.5, eta_c=float(eta_c), p_m=0.0, lb=-2.0 ** 24, ub=2.0 ** 24)
    run = P.Run(2, 2, d, K, K, seed=seed, params=prm)
    r = np.random.default_rng(eta_c)
    X = (r.random((K, d)) - 0.5).astype(np.float32)
    valid = np.ones(K, np.uint8)
    run.set_state(X, r.random((K, 2)).astype(np.float32), valid, t=0)
    if batched:
        batch = P.Batch(1)
        batch.admit(run)
        batch.step()
        off = run.get_offspring()
        batch.retire(run)
        batch.close()
    else:
        run.step()
        off = run.get_offspring()
    run.close()
    parents, _ = O.mate(seed, 1, valid, K)
    assert np.array_equal(off["parents"], parents)
    want, pre = O.reproduce(ora_params(O, prm), seed, 1, X, parents, K, with_pre=True)
    assert np.abs(want).max() < 2.0 ** 24  # no child at the box
    straddles = gene_mismatches(off["X"], want, pre)
    assert straddles <= 1e-6 * want.size
