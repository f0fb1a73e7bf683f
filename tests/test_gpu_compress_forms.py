"""Recompression at the edges of its QR and eigenvalue kernels' forms: QR
operands of each LDS size (up to 2560, 4608 and 8192 elements), of fewer rows
than columns and of more than 128 rows, eigenproblems of order 1, odd, and at
the sizes the matrix is stored in (32, 33, 48, 49, 64).  With tau = 0 the
operator is the same matrix: its product is within 1e-8 of the absolute-value
bound, the tolerance of the other recompression tests (eps / tau^2 does not
enter; eps times the products of ranks and levels is below 1e-11)."""
import numpy as np
import pytest

import h2gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ranks,leaf,kids", [
    ([1, 1, 1], 7, 2), ([3, 5, 7], 2, 3), ([9, 17, 31], 40, 3), ([32, 32, 32], 80, 2), ([20, 33, 30], 70, 4),
    ([47, 48, 48], 96, 2), ([40, 49, 63], 128, 2), ([20, 42, 64], 120, 3), ([20, 20, 63], 60, 6),
], ids=str)
def test_compress_forms_keep_the_matrix(ranks, leaf, kids):
    from paper_2109_05451_amd import H2Operator
    for seed, separate in ((1, False), (2, True)):
        buf = np.array(h2gen.random_rep(5200 + seed, integer=False, q=2, max_children=kids, max_leaf=leaf,
                                        ranks=(ranks, ranks), separate=separate, p_adm=0.4), copy=True)
        ref = oracle.Oracle(buf)
        X = np.random.default_rng(seed).standard_normal((ref.n, 3))
        want, B = ref.gemv(X), ref.gemv(X, absval=True)
        g = H2Operator(buf)
        c, info = g.compress(0.0)
        Y = c.gemv(torch.from_numpy(np.asfortranarray(X)).cuda())
        torch.cuda.synchronize()
        assert np.all(np.abs(Y.cpu().numpy() - want) <= 1e-8 * B + 1e-300), (seed, separate)
        c.close()
        g.close()
        ref.close()


def test_compress_refuses_operands_past_the_largest_form():
    """Three children of rank 64 under a parent of rank 64: 12 288 elements."""
    from paper_2109_05451_amd import H2Error, H2Operator
    buf = np.array(h2gen.random_rep(5202, integer=False, q=2, max_children=3, max_leaf=120,
                                    ranks=([42, 64, 64], [42, 64, 64]), separate=True, p_adm=0.4), copy=True)
    g = H2Operator(buf)
    with pytest.raises(H2Error):
        g.compress(0.0)
    g.close()
