"""The composed sweeps (FP64: several transfer levels per launch, with the
products of the transfers between them formed at load) on deep trees of any
arity, with empty leaves, shared and separate bases, ranks that differ per
level and between rows and columns, and rows of more columns than one
source-row table: both ops, every pass width, bit for bit the oracle's
integers (entries in {-1, 0, 1}, every product of transfers an integer below
2^53).  On built operators of a few thousand points, whose sweeps fall into
one to four stages, both ops are within 1e-12 * B of the oracle, the bar of
the other FP64 parity tests."""
import numpy as np
import pytest

import h2gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def run(g, X, op):
    Y = g.gemv(torch.from_numpy(np.asfortranarray(X)).cuda(), op=op)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


CASES = [
    dict(q=5, max_children=2, max_leaf=6, max_rank=4, p_adm=0.1),
    dict(q=6, max_children=2, max_leaf=4, max_rank=3, p_adm=0.15, separate=False),
    dict(q=4, max_children=3, max_leaf=9, max_rank=5, p_adm=0.1, allow_empty=True),
    dict(q=7, max_children=1, max_leaf=20, max_rank=4, p_adm=0.2),
    dict(q=3, max_children=4, max_leaf=60, ranks=([7, 20, 33, 17], [5, 36, 18, 40]), p_adm=0.05),
    dict(q=3, max_children=3, max_leaf=70, ranks=([64, 70, 66, 65], [64, 70, 66, 65]), p_adm=0.1, separate=False),
    dict(q=2, max_children=7, max_leaf=61, ranks=([5] * 3, [7] * 3), p_adm=0.02),
]


@pytest.mark.parametrize("ci", range(len(CASES)))
def test_composed_sweeps_integer_bitwise(ci):
    from paper_2109_05451_amd import H2Operator
    for seed in range(4):
        buf = h2gen.random_rep(9000 + 10 * ci + seed, integer=True, int_range=1, **CASES[ci])
        ref = oracle.Oracle(buf)
        g = H2Operator(buf)
        for nv in (1, 3, 7, 20, 40, 64):
            X = np.random.default_rng(nv).integers(-1, 2, size=(g.n, nv)).astype(np.float64)
            for op in "NT":
                assert ref.gemv(X, op=op, absval=True).max(initial=0.0) < 2.0 ** 53
                assert np.array_equal(run(g, X, op), ref.gemv(X, op=op)), (ci, seed, nv, op)
        g.close()
        ref.close()


@pytest.mark.parametrize("n,dim,leaf,p", [(700, 2, 30, 4), (4096, 2, 64, 4), (9000, 2, 40, 6), (6000, 3, 48, 3),
                                          (30000, 2, 33, 5)])
def test_composed_sweeps_built_operators(n, dim, leaf, p):
    from paper_2109_05451_amd import H2Operator
    buf = np.array(h2gen.build(h2gen.points(n, dim, 51), leaf=leaf, p=p, eta=0.7,
                               kernel="exp" if dim == 2 else "laplace").array, copy=True)
    ref = oracle.Oracle(buf)
    g = H2Operator(buf)
    stages = [line for line in g.plan_info().splitlines() if line.startswith("up ")]
    assert 1 <= len(stages) < g.stats()["depth"]  # fewer launches than levels
    for nv in (1, 4, 17, 64):
        X = h2gen.vectors(n, nv, nv)
        for op in "NT":
            want, B = ref.gemv(X, op=op), ref.gemv(X, op=op, absval=True)
            assert np.all(np.abs(run(g, X, op) - want) <= 1e-12 * B), (nv, op)
    g.close()
    ref.close()
