"""Workspaces sized by an earlier build go on sufficing: no shape needs more
device memory than it did (small and large vector counts, few and many
individuals, both sides of the layouts' rules)."""
import os

HERE = os.path.dirname(os.path.abspath(__file__))


def test_footprints_are_no_larger():
    import paper_2404_01159_amd as P

    rows = [line.split() for line in open(os.path.join(HERE, "golden", "footprints.txt"))
            if line.strip() and not line.startswith("#")]
    assert len(rows) > 150
    larger = []
    for m, d, N, K, op, was in rows:
        prm = P.default_params(op)
        now = P.footprint(1, int(m), int(d), int(N), int(K), prm)
        if now > int(was):
            larger.append((m, d, N, K, op, was, now))
    assert not larger, larger[:5]
