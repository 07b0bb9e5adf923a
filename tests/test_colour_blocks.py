"""The block form of the colour matrix (24 and 120 flows): on integer jamps, where every sum is
exact, it equals the full quadratic form, and the blocks' vectors form an orthogonal basis."""
import numpy as np
import pytest

from paper_2210_11122_amd.gen import colour


@pytest.mark.parametrize("n", [4, 5])
def test_block_form_equals_the_colour_matrix(n):
    _, C = colour.colour_matrix_quark_line(n)
    den = colour.common_denominator(C)
    num = np.array([[int(x * den) for x in row] for row in C], dtype=object)
    blocks, table = colour.block_form(n, num.tolist())
    nc = len(num)
    assert sum(len(b) for b in blocks) == nc
    basis = np.zeros((nc, nc), dtype=int)
    for k, v in enumerate(v for b in blocks for v in b):
        for f, w in v.items():
            basis[k, f] = w
    gram = basis @ basis.T
    assert np.array_equal(gram, np.diag(np.diag(gram))) and set(np.diag(gram)) <= {4, 8}
    rng = np.random.default_rng(5)
    for _ in range(3):
        J = rng.integers(-1000, 1000, nc)
        z = (basis @ J).astype(object)
        q, t, at = 0, 0, 0
        for b in blocks:
            for i in range(len(b)):
                for j in range(i, len(b)):
                    q += table[t] * z[at + i] * z[at + j]
                    t += 1
            at += len(b)
        assert t == len(table)
        J = J.astype(object)
        assert q == 64 * (J @ num @ J)
