"""The wave-per-row kernels at the edges of their forms: ranks and leaf sizes
around the 16-row tiles and the four-row tails (one and two of them), rows of
one column, rows of more columns than one source-row table (1024), blocks of
odd width (four-column steps that straddle blocks) and empty leaves, for every
pass width, in both forms (codes 9-12), from the column-major matrices and
from the fragment-ordered copies, and untuned; and the transposed rows of op
'T' at the same edges.  Integer representations: every partial sum
is an integer below 2^53, so the products are the oracle's bit for bit."""
import numpy as np
import pytest

import h2gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

# (row rank, column rank, largest leaf, seed of a tree with blocks of both kinds)
SHAPES = [(1, 1, 2, 541), (4, 16, 16, 564), (16, 17, 17, 556), (17, 20, 20, 517), (20, 21, 25, 560),
          (24, 33, 33, 584), (25, 36, 36, 525), (33, 25, 40, 673), (36, 41, 41, 556), (40, 48, 49, 560),
          (48, 52, 52, 568), (52, 56, 56, 572), (56, 57, 57, 596), (57, 64, 64, 557), (64, 64, 64, 584)]


def run(g, X, prec, op="N"):
    Y = g.gemv(torch.from_numpy(np.asfortranarray(X)).cuda(), op=op, alpha=2.0, precision=prec)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


@pytest.mark.parametrize("kr,kc,leaf,seed", SHAPES)
def test_wave_rows_integer_bitwise(kr, kc, leaf, seed):
    from paper_2109_05451_amd import H2Operator
    buf = h2gen.random_rep(seed, q=2, max_children=3, max_leaf=leaf, ranks=([kr] * 3, [kc] * 3), p_adm=0.3,
                           integer=True, int_range=1)
    ref = oracle.Oracle(buf)
    g = H2Operator(buf)
    X = np.random.default_rng(0).integers(-1, 2, size=(g.n, 64)).astype(np.float64)
    assert np.array_equal(run(g, X, "fp64"), ref.gemv(X, alpha=2.0))  # untuned
    for prec in ("fp64", "fp32"):
        g.set_sweeps(prec, False)
    for nv in (5, 32, 40, 64):
        X = np.random.default_rng(nv).integers(-1, 2, size=(g.n, nv)).astype(np.float64)
        want = ref.gemv(X, alpha=2.0)
        assert np.array_equal(run(g, X, "fp64", "T"), ref.gemv(X, op="T", alpha=2.0)), nv
        # FP32 is exact only while every partial sum stays below 2^24
        small = ref.gemv(X, alpha=2.0, absval=True).max() < 2.0 ** 24
        for prec in ("fp64", "fp32") if small else ("fp64",):
            for fl in (False, True):
                g.set_fragment_order(prec, fl)
                for code in (9, 10, 11, 12):
                    g.tune_set(prec, code, 0, code == 10, 0)
                    if not fl:
                        g.set_fragment_order(prec, False)  # tune_set lets launches read the copies
                    assert np.array_equal(run(g, X, prec), want), (nv, prec, fl, code)
    g.close()
    ref.close()


@pytest.mark.parametrize("nv", [16, 64])
def test_wave_rows_of_several_tables(nv):
    """Dense rows of more than 1024 columns: several source-row tables."""
    from paper_2109_05451_amd import H2Operator
    buf = h2gen.random_rep(82, q=2, max_children=7, max_leaf=61, ranks=([5] * 3, [7] * 3), p_adm=0.02, integer=True,
                           int_range=1)
    ref = oracle.Oracle(buf)
    g = H2Operator(buf)
    assert g.stats()["csp_dense"] == g.stats()["nleaves"] and g.n > 1024  # a row with every leaf's columns
    X = np.random.default_rng(3).integers(-1, 2, size=(g.n, nv)).astype(np.float64)
    want = ref.gemv(X, alpha=2.0)
    for code in (9, 10, 11, 12):
        g.tune_set("fp64", code, 8 if code == 11 else 0)
        assert np.array_equal(run(g, X, "fp64"), want), code
    g.close()
    ref.close()
