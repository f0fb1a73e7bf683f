"""The streamed transposed rows (op 'T', one to four vectors) at the edges of
their forms: odd and even block heights and widths from 1 to 256 (one to
eight column slots per thread, several block groups per workgroup, and rows
that keep the LDS kernel), many blocks per row, empty leaves: the oracle's
integers bit for bit."""
import numpy as np
import pytest

import h2gen
import oracle

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("case", [
    dict(q=2, ranks=([1, 2, 3], [3, 1, 2]), max_leaf=3), dict(q=2, ranks=([17, 16, 15], [15, 17, 16]), max_leaf=31),
    dict(q=2, ranks=([36, 25, 33], [33, 36, 25]), max_leaf=50), dict(q=1, ranks=([64, 64], [64, 63]), max_leaf=65),
    dict(q=1, ranks=([129, 90], [70, 129]), max_leaf=130), dict(q=1, ranks=([256, 255], [256, 256]), max_leaf=256),
    dict(q=5, max_children=4, ranks=([2] * 6, [3] * 6), max_leaf=2, p_adm=0.03)])
def test_cols_integer_bitwise(case):
    from paper_2109_05451_amd import H2Operator
    case = dict(dict(max_children=3, p_adm=0.2), **case)
    for seed in range(3):
        buf = h2gen.random_rep(300 + seed, integer=True, int_range=1, **case)
        ref = oracle.Oracle(buf)
        g = H2Operator(buf)
        for nv in (1, 2, 3, 4):
            X = np.random.default_rng(nv).integers(-2, 3, size=(g.n, nv)).astype(np.float64)
            assert ref.gemv(X, op="T", absval=True).max(initial=0.0) < 2.0 ** 53
            Y = g.gemv(torch.from_numpy(np.asfortranarray(X)).cuda(), op="T")
            torch.cuda.synchronize()
            assert np.array_equal(Y.cpu().numpy(), ref.gemv(X, op="T")), (seed, nv)
        g.close()
        ref.close()
