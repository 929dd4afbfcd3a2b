"""What one max-flow says about other candidates of its sink, shown with the oracle's max-flow alone (CPU): F(U, k) is concave in U / k once
divided by k, a demand that arrives in full arrives at every larger U / k, and the sink's own cut, where a flow meets it, is the
value at every smaller U / k."""
from fractions import Fraction

import numpy as np
import pytest

import oracle as o
import workloads as w


@pytest.mark.parametrize("seed", range(12))
def test_lines_between_candidates(seed):
    topo = w.random_tiny(seed, n_vertices=9)
    rng = np.random.default_rng(seed)
    inb = o.in_bandwidths(topo)
    N = topo.n_compute
    cand = sorted({(int(rng.integers(1, 40)), int(rng.integers(1, 7))) for _ in range(24)}, key=lambda c: Fraction(*c))
    for t in topo.compute_nodes:
        F = [int(o.aux_maxflow(topo, int(t), U, k)) for U, k in cand]
        phi = [Fraction(f, k) for f, (_, k) in zip(F, cand)]
        r = [Fraction(U, k) for U, k in cand]
        for i in range(len(cand)):
            own = cand[i][1] + cand[i][0] * int(inb[t])
            for j in range(len(cand)):
                if r[j] >= r[i] and F[i] == N * cand[i][1]:
                    assert F[j] == N * cand[j][1]
                if r[j] <= r[i] and F[i] == own:
                    assert F[j] == cand[j][1] + cand[j][0] * int(inb[t])
        for a in range(len(cand)):
            for c in range(a + 1, len(cand)):
                if r[a] == r[c]:
                    assert phi[a] == phi[c]
                    continue
                for b in range(a + 1, c):
                    assert phi[b] >= phi[a] + (phi[c] - phi[a]) * (r[b] - r[a]) / (r[c] - r[a])
