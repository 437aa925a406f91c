"""Block form of the colour matrix (gen.emit.colour_blocks), CPU.

The butterflies and the block matrix reproduce the quadratic form of the
colour matrix exactly (integers), and leave at most 4 x 4 blocks for the 24
colour flows of g g -> t t~ g g.
"""
import random

from paper_2106_12631_amd.gen import emit
from paper_2106_12631_amd.gen.diagrams import ProcessDiagrams, colour_matrix


def test_blocks_reproduce_the_quadratic_form():
    pd = ProcessDiagrams('ggttgg')
    basis = pd.colour_basis()
    cnum, _ = colour_matrix(basis, len(pd.gluons))
    fly, D, scale = emit.colour_blocks(basis, cnum)
    n = len(basis)
    rng = random.Random(5)
    for _ in range(3):
        x = [rng.randrange(-1000, 1000) for _ in range(n)]
        y = list(x)
        for i, j, s in fly:
            y[i], y[j] = y[i] + s * y[j], y[i] - s * y[j]
        want = sum(cnum[i][j] * x[i] * x[j] for i in range(n) for j in range(n))
        got = sum(D[i][j] * y[i] * y[j] for i in range(n) for j in range(n))
        assert got == scale * want
    assert max(sum(1 for v in row if v) for row in D) <= 4
