"""Code paths that small operators do not take, each with an assertion that
the operator of the test takes it:

* FP64 schedules, graph replay and the no-allocation product with a composed
  downsweep stage (60 000 points): only there does schedule 3 fork the third
  stream, in op 'N' products of one vector and of many;
* op 'T' on the matrix cores under graph capture;
* op 'T' launches of enough block columns to run one wave per row, their
  number not a multiple of the rows of a workgroup;
* rows of more columns than one source-row table (1024): dense rows and
  composed sweep rows split over four waves (4096 columns and more), coupling
  rows on the wave-row kernels.

Built operators: 1e-12 * B, B the oracle's product in absolute values (the
FP64 bar of the parity tests).  Integer representations: every partial sum is
an integer below 2^53, so the products are the oracle's bit for bit."""
import ctypes

import numpy as np
import pytest

import h2gen
import oracle
from h2gen import fmt

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def dev(X):
    return torch.from_numpy(np.asfortranarray(X)).cuda()


def run(g, X, op="N", **kw):
    Y = g.gemv(dev(X), op=op, **kw)
    torch.cuda.synchronize()
    return Y.cpu().numpy()


def close(ref, X, got, op="N", alpha=1.0, beta=0.0, Y0=None):
    want = ref.gemv(X, op=op, alpha=alpha, beta=beta, Y=Y0)
    B = ref.gemv(X, op=op, alpha=alpha, beta=beta, Y=Y0, absval=True)
    return np.all(np.abs(got - want) <= 1e-12 * B)


@pytest.fixture(scope="module")
def staged():
    """An operator with a composed downsweep stage of its own."""
    from paper_2109_05451_amd import H2Operator
    buf = np.array(h2gen.build(h2gen.points(60000, 2, 5), leaf=50, p=5, eta=0.7, kernel="exp").array, copy=True)
    g, ref = H2Operator(buf), oracle.Oracle(buf)
    lines = g.plan_info().splitlines()
    assert any(s.startswith("down rows=") for s in lines) and any(s.startswith("couple_deep rows=") for s in lines)
    assert not any(s.startswith("input ") for s in lines)
    yield g, ref
    g.close()
    ref.close()


@pytest.mark.parametrize("nv", [1, 3, 16, 64])
def test_schedules_with_a_downsweep_stage(staged, nv):
    g, ref = staged
    X = h2gen.vectors(g.n, nv, 70 + nv)
    got = []
    for sc in (0, 1, 2, 3, 3):
        g.set_schedule("fp64", sc)
        got.append(run(g, X))
    assert close(ref, X, got[0])
    assert all(np.array_equal(y, got[0]) for y in got[1:])


@pytest.mark.parametrize("op,nv,schedule", [("N", 1, 3), ("N", 20, 0), ("N", 20, 3), ("T", 1, 0), ("T", 24, 0)])
def test_graph_replay_with_a_downsweep_stage(staged, op, nv, schedule):
    g, ref = staged
    g.set_schedule("fp64", schedule)
    stream = torch.cuda.Stream()
    rng = np.random.default_rng(nv)
    inputs = [rng.standard_normal((g.n, nv)) for _ in range(2)]
    Y0 = rng.standard_normal((g.n, nv))
    X, Y = dev(inputs[0]), dev(Y0)

    def product(Xh):
        X.copy_(torch.from_numpy(Xh))
        Y.copy_(torch.from_numpy(Y0))
        torch.cuda.synchronize()
        g.gemv_raw(op, 1.5, X.data_ptr(), g.n, nv, -0.5, Y.data_ptr(), g.n, stream.cuda_stream)
        stream.synchronize()
        return Y.cpu().numpy()

    eager = [product(Xh) for Xh in inputs]
    assert close(ref, inputs[0], eager[0], op, 1.5, -0.5, Y0)
    g.graph(True)
    for rep in range(5):  # the first captures
        assert np.array_equal(product(inputs[rep % 2]), eager[rep % 2]), rep
        torch.randn(300, 300, device="cuda").sum()
        torch.cuda.synchronize()
    g.graph(False)


def test_growing_workspace_drops_the_graphs():
    """One vector captured, then 20 on the same handle, then the first call again."""
    from paper_2109_05451_amd import H2Operator
    buf = np.array(h2gen.build_config("c1_2d_4096").array, copy=True)
    g, ref = H2Operator(buf), oracle.Oracle(buf)
    stream = torch.cuda.Stream()
    X1, X20 = h2gen.vectors(g.n, 1, 1), h2gen.vectors(g.n, 20, 2)
    bufs = [(X, dev(X), dev(np.zeros_like(X))) for X in (X1, X20)]
    torch.cuda.synchronize()
    g.graph(True)
    for Xh, X, Y in (bufs[0], bufs[1], bufs[0], bufs[1]):
        g.gemv_raw("N", 1.0, X.data_ptr(), g.n, Xh.shape[1], 0.0, Y.data_ptr(), g.n, stream.cuda_stream)
        stream.synchronize()
        assert close(ref, Xh, Y.cpu().numpy())
        Y.zero_()
        torch.cuda.synchronize()
    g.close()
    ref.close()


@pytest.mark.parametrize("schedule", [0, 3])
def test_noalloc_with_a_downsweep_stage(staged, schedule):
    from paper_2109_05451_amd import load_library
    g, ref = staged
    g.set_schedule("fp64", schedule)
    X = h2gen.vectors(g.n, 3, 9)
    Xd, Y = dev(X), dev(np.zeros_like(X))
    rc = load_library().h2_gemv_noalloc(g._h, b"N", 1.0, Xd.data_ptr(), g.n, 3, 0.0, Y.data_ptr(), g.n,
                                        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    torch.cuda.synchronize()
    assert rc == 0 and np.array_equal(Y.cpu().numpy(), run(g, X))


# points, leaf, Chebyshev order: 32 768 leaves of 4 points (rank 4), 16 384 of 20 (rank 9)
@pytest.mark.parametrize("n,leaf,p", [(131073, 8, 2), (330001, 24, 3)])
def test_transposed_products_one_wave_per_row(n, leaf, p):
    from paper_2109_05451_amd import H2Operator
    buf = np.array(h2gen.build(h2gen.points(n, 2, 5), leaf=leaf, p=p, eta=0.7, kernel="exp").array, copy=True)
    g, ref = H2Operator(buf), oracle.Oracle(buf)
    st = g.stats()
    # launches of 8192 waves and more: the coupling rows (one per node) and each half of the dense rows
    assert st["nleaves"] // 2 >= 8192 and st["nnodes"] % 4 != 0 and st["nnodes"] % 2 != 0
    X = h2gen.vectors(g.n, 64, 64)
    want, B = ref.gemv(X, op="T"), ref.gemv(X, op="T", absval=True)
    for nv in (16, 24, 40, 64):
        assert np.all(np.abs(run(g, X[:, :nv], "T") - want[:, :nv]) <= 1e-12 * B[:, :nv]), nv
    g.close()
    ref.close()


def width(buf, dense):
    """Columns of the longest dense or coupling row."""
    r = fmt.parse(buf)
    if not dense:
        return max(int(np.diff(rp).max()) * int(k) for rp, k in zip(r["s_rowptr"], r["kcol"]))
    lp, q = r["level_ptr"], r["q"]
    m = r["hi"][lp[q]:] - r["lo"][lp[q]:]
    return max(int(m[r["d_col"][a:b]].sum()) for a, b in zip(r["d_rowptr"][:-1], r["d_rowptr"][1:]))


@pytest.mark.parametrize("p_adm", [0.0, 1.0])
def test_split_rows_of_several_tables(p_adm):
    """All dense: rows of n columns, over 1024 for each of the four waves.  One
    coupling block at the root: composed rows of n columns on the way up."""
    from paper_2109_05451_amd import H2Operator
    buf = h2gen.random_rep(4, q=1, max_children=200, max_leaf=64, ranks=([20] * 2, [36] * 2), p_adm=p_adm,
                           integer=True, int_range=1)
    g, ref = H2Operator(buf), oracle.Oracle(buf)
    assert g.n > 4 * 1024 and g.stats()["nleaves"] < 8192 and g.stats()["max_leaf"] <= 64
    if p_adm == 0.0:
        assert (width(buf, True) + 3) // 4 > 1024
    else:  # one stage from the points to the root and back, in three launches
        assert g.stats()["ncoupling"] == 1 and g.stats()["ndense"] == 0
        up = [s for s in g.plan_info().splitlines() if s.startswith("up rows=")]
        assert len(up) == 1 and int(up[0].split("rows=")[1].split()[0]) == g.stats()["nnodes"]
    for nv in (3, 16, 20, 40, 64):
        X = np.random.default_rng(nv).integers(-1, 2, size=(g.n, nv)).astype(np.float64)
        for op in "NT":
            assert np.array_equal(run(g, X, op, alpha=2.0), ref.gemv(X, op=op, alpha=2.0)), (nv, op)
    g.close()
    ref.close()


def test_coupling_rows_of_several_tables():
    from paper_2109_05451_amd import H2Operator
    buf = h2gen.random_rep(3, q=1, max_children=40, max_leaf=20, ranks=([64] * 2, [64] * 2), p_adm=0.6, integer=True,
                           int_range=1)
    assert width(buf, False) > 1024
    g, ref = H2Operator(buf), oracle.Oracle(buf)
    for nv in (16, 32, 40, 64):
        X = np.random.default_rng(nv).integers(-1, 2, size=(g.n, nv)).astype(np.float64)
        want = ref.gemv(X, alpha=2.0)
        assert np.array_equal(run(g, X, alpha=2.0), want), nv  # untuned
        for fl in (False, True):
            g.set_fragment_order("fp64", fl)
            for code in (9, 10, 11, 12):
                g.tune_set("fp64", code)
                if not fl:
                    g.set_fragment_order("fp64", False)  # tune_set lets launches read the copies
                assert np.array_equal(run(g, X, alpha=2.0), want), (nv, fl, code)
    g.close()
    ref.close()
