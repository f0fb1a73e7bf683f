"""Dense near-field rows of operators of few leaves on the multi-vector path:
a workgroup per row, the columns split over its four waves.  Leaf sizes at the
edges of the row tiles (every form, and the fallback past 64 rows), rows of
fewer columns than waves and of more than one source-row table per wave, both
row orders, XCD ranges and a persistent grid smaller than the rows; bit for
bit the oracle's integers (entries in {-1, 0, 1}, sums below 2^53)."""
import numpy as np
import pytest

import h2gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kw", [
    dict(q=2, max_children=3, max_leaf=3, max_rank=2, p_adm=0.1, allow_empty=True),
    dict(q=2, max_children=4, max_leaf=16, max_rank=3, p_adm=0.2),
    dict(q=2, max_children=4, max_leaf=33, max_rank=3, p_adm=0.1),
    dict(q=2, max_children=4, max_leaf=36, max_rank=3, p_adm=0.1, allow_empty=True),
    dict(q=2, max_children=4, max_leaf=50, max_rank=3, p_adm=0.1),
    dict(q=2, max_children=3, max_leaf=64, max_rank=3, p_adm=0.1),
    dict(q=2, max_children=3, max_leaf=75, max_rank=3, p_adm=0.1),
    dict(q=3, max_children=6, max_leaf=61, max_rank=3, p_adm=0.01),
], ids=lambda kw: str(kw["max_leaf"]))
def test_dense_split_integer_bitwise(kw):
    from paper_2109_05451_amd import H2Operator
    for seed in range(3):
        buf = h2gen.random_rep(7100 + seed, integer=True, int_range=1, **kw)
        ref = oracle.Oracle(buf)
        g = H2Operator(buf)
        for nv in (5, 30, 48, 64):
            X = np.random.default_rng(nv).integers(-1, 2, size=(g.n, nv)).astype(np.float64)
            assert ref.gemv(X, absval=True).max(initial=0.0) < 2.0 ** 53
            want, Xd = ref.gemv(X), torch.from_numpy(np.asfortranarray(X)).cuda()
            for xcd, tree, grid in ((0, False, -1), (1, True, -1), (0, False, 3), (1, True, 8)):
                g.tune_set("fp64", 9, 0, xcd, tree)
                g.set_dense_grid(grid)
                Y = g.gemv(Xd)
                torch.cuda.synchronize()
                assert np.array_equal(Y.cpu().numpy(), want), (seed, nv, xcd, tree, grid)
        g.close()
        ref.close()
