"""Wide leaf levels and input products of LSTMs and bidirectional recurrences with packed input rows against the oracle: every instance (columns up to 128, 256,
384, 512, 768, 1 024), steps that do not divide evenly, rows that do not fill a block, groups that straddle an XCD, inputs that
are not to be split, the call that allocates nothing.

Tolerance: 1e-6 over the 2-norm, as in test_split_contraction."""
import numpy as np
import pytest

import oracle
from workloads import generators as gen

pytestmark = pytest.mark.gpu

NT = oracle.default_threads()


def rel(got, want):
    want = want.astype(np.float64)
    return float(np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want))


@pytest.fixture(scope="module")
def ctx():
    import paper_2305_10611_amd as A
    c = A.Context(0)
    yield c
    c.close()


def takes_it(ctx, run, kind):
    """The level's launch record says 16-row blocks."""
    import paper_2305_10611_amd as A
    ctx.acrobat_set_profiling(True)
    try:
        out = run()
        r = [x for x in ctx.acrobat_last_profile() if x[0] == getattr(A.binding, kind)]
    finally:
        ctx.acrobat_set_profiling(False)
    assert r and r[0][4] == 16 and r[0][5] == -1
    return out


@pytest.mark.parametrize("H,D,n", [(512, 96, 3391), (512, 256, 1270), (320, 352, 1500), (512, 512, 637), (256, 672, 1000),
                                   (480, 1024, 340), (288, 544, 1073)])
def test_leaf_levels(ctx, H, D, n):
    from tests import parity as P
    w = gen.treelstm_workload(n, 1, 2, H, 50, "uniform", seed=H + D, bias_scale=0.2, D=D)
    h, c = takes_it(ctx, lambda: P.run_treelstm(ctx, w), "K_TREE_LEAF")
    oh, oc = oracle.treelstm(w, nthreads=NT)
    assert rel(h, oh) < 1e-6 and rel(c, oc) < 1e-6


@pytest.mark.parametrize("H,D,n", [(256, 128, 1911), (512, 224, 620), (352, 384, 477), (512, 512, 245), (320, 736, 285),
                                   (256, 992, 263), (1024, 32, 1921)])
def test_lstm_input_products(ctx, H, D, n):
    from tests import parity as P
    w = gen.lstm_workload(n, 2, 2, H, D, seed=H + D, bias_scale=0.2)
    h, c = takes_it(ctx, lambda: P.run_lstm(ctx, w), "K_LSTM_INPUT")
    oh, oc = oracle.varlen_lstm(w, nthreads=NT)
    assert rel(h, oh) < 1e-6 and rel(c, oc) < 1e-6


@pytest.mark.parametrize("H,D,n", [(256, 256, 2865), (512, 288, 1273), (320, 352, 1669), (256, 512, 1433), (512, 736, 499),
                                   (384, 992, 497)])
def test_birnn_input_products(ctx, H, D, n):
    """Both directions in one launch; a feature of 1e9 with weights of 1e-9 and a NaN are what fp32 makes of them."""
    from tests import parity as P
    w = gen.birnn_workload(n, 2, 2, H, D, 5, seed=H + D)
    got = takes_it(ctx, lambda: P.run_birnn(ctx, w), "K_RNN_INPUT")
    for a, b in zip(got, oracle.birnn(w, nthreads=NT)):
        assert rel(a, b) < 1e-6
    w["x"][:, 3] *= 1e9
    w["fWx"][:, 3] *= 1e-9
    w["bWx"][:, 3] *= 1e-9
    want = oracle.birnn(w, nthreads=NT)
    w["x"][9, 7] = np.nan  # of the fifth sequence
    rest = np.r_[0:8, 10:2 * n]
    got = P.run_birnn(ctx, w)
    for a, b in zip(got, want):
        assert rel(a[rest], b[rest]) < 1e-6
    assert np.isnan(got[0][9]).all() and np.isnan(got[1][9]).all()


def test_rows_that_are_not_to_be_split(ctx):
    """A feature of 1e9 with a weight of 1e-9 beside ordinary ones, infinities and NaNs: what fp32 says."""
    from tests import parity as P
    w = gen.treelstm_workload(1200, 1, 2, 320, 64, "uniform", seed=5, bias_scale=0.2, D=352)
    w["emb"][:, 3] *= 1e9
    w["W_leaf"][:, 3] *= 1e-9
    h, c = takes_it(ctx, lambda: P.run_treelstm(ctx, w), "K_TREE_LEAF")
    oh, oc = oracle.treelstm(w, nthreads=NT)
    assert rel(h, oh) < 1e-6 and rel(c, oc) < 1e-6
    w["emb"][5, 7], w["emb"][6, 9] = np.inf, np.nan
    h, c = P.run_treelstm(ctx, w)
    roots_of = np.repeat(np.arange(1200), np.diff(w["tree_off"]))
    odd = np.unique(roots_of[np.isin(w["token"], (5, 6)) & (w["left"] < 0)])
    rest = ~np.isin(roots_of, odd)
    assert np.isfinite(h[rest]).all()
    assert rel(h[rest], oh[rest]) < 1e-6
    assert np.isnan(h[np.flatnonzero((w["token"] == 6) & (w["left"] < 0))]).all()


@pytest.mark.parametrize("kind,H,D,n", [("tree", 512, 512, 1270), ("tree", 256, 992, 1000), ("lstm", 512, 224, 620),
                                        ("lstm", 320, 736, 285), ("birnn", 512, 288, 1273), ("birnn", 320, 992, 597)])
def test_some_rows_that_are_not_to_be_split(ctx, kind, H, D, n):
    """A feature of 1e9 with a weight of 1e-9 in every third row, not in the others: what fp32 says for all of them."""
    from tests import parity as P
    if kind == "tree":
        w = gen.treelstm_workload(n, 1, 2, H, 50, "uniform", seed=H + D, bias_scale=0.2, D=D)
        x, weights, run, want = "emb", ["W_leaf"], P.run_treelstm, oracle.treelstm
    elif kind == "lstm":
        w = gen.lstm_workload(n, 2, 2, H, D, seed=H + D, bias_scale=0.2)
        x, weights, run, want = "x", ["Wx"], P.run_lstm, oracle.varlen_lstm
    else:
        w = gen.birnn_workload(n, 2, 2, H, D, 5, seed=H + D)
        x, weights, run, want = "x", ["fWx", "bWx"], P.run_birnn, oracle.birnn
    w[x][::3, 3] *= 1e9
    for k in weights:
        w[k][:, 3] *= 1e-9
    got = takes_it(ctx, lambda: run(ctx, w), {"tree": "K_TREE_LEAF", "lstm": "K_LSTM_INPUT", "birnn": "K_RNN_INPUT"}[kind])
    for a, b in zip(got, want(w, nthreads=NT)):
        assert rel(a, b) < 1e-6


@pytest.mark.parametrize("kind,H,D,n", [("birnn", 256, 512, 1433), ("birnn", 512, 736, 499), ("birnn", 512, 32, 200),
                                        ("lstm", 320, 736, 285), ("lstm", 256, 992, 263), ("lstm", 256, 32, 200)])
def test_no_less_exact_than_fp32(ctx, kind, H, D, n):
    """Input products and (D = 32) steps that were fp32 before they were split: no further from 64 bits than the fp32 tiles
    (measured: 0.50 to 1.0 of their error)."""
    from tests import parity as P
    if kind == "lstm":
        w, run, want = gen.lstm_workload(n, 2, 9, H, D, seed=H + D, bias_scale=0.2), P.run_lstm, oracle.varlen_lstm
    else:
        w, run, want = gen.birnn_workload(n, 2, 9, H, D, 5, seed=H + D), P.run_birnn, oracle.birnn
    got = run(ctx, w)
    ctx.check(ctx.acrobat_set_tuning(64, 1, 0))
    try:
        plain = run(ctx, w)
    finally:
        ctx.check(ctx.acrobat_set_tuning(0, 0, 0))
    for a, b, r in zip(got, plain, want(w, nthreads=NT)):
        assert rel(a, r) <= 1.02 * rel(b, r)


@pytest.mark.parametrize("kind", ["tree", "lstm", "birnn"])
def test_unscaled_features_cost_a_few_times_the_product(ctx, kind):
    """Features of 1e5: no row is to be split, and all products run on the fp32 matrix cores.  A scalar product per element made
    the launches 44 to 59 times as long as with features of order one (2.6, 3.5 and 1.7 ms); now it is 4 to 5 (0.25, 0.29, 0.16)."""
    from tests import parity as P
    import paper_2305_10611_amd as A
    H, n = 512, 1500
    ms = []
    for scale in (1.0, 1e5):
        if kind == "tree":
            w = gen.treelstm_workload(n, 4, 4, H, 500, "uniform", seed=1, D=H)
            w["emb"] *= scale
            run, record = P.run_treelstm, A.binding.K_TREE_LEAF
        elif kind == "lstm":
            w = gen.lstm_workload(n, 4, 4, H, H, seed=1)
            w["x"] *= scale
            run, record = P.run_lstm, A.binding.K_LSTM_INPUT
        else:
            w = gen.birnn_workload(n, 4, 4, H, H, 5, seed=1)
            w["x"] *= scale
            run, record = P.run_birnn, A.binding.K_RNN_INPUT
        run(ctx, w)
        ctx.acrobat_set_profiling(True)
        try:
            times = []
            for _ in range(5):
                run(ctx, w)
                times += [r[3] for r in ctx.acrobat_last_profile() if r[0] == record]
        finally:
            ctx.acrobat_set_profiling(False)
        ms.append(min(times))
    assert ms[1] < 15 * ms[0]


def test_without_allocations(ctx):
    import paper_2305_10611_amd as A
    from tests import parity as P
    w = gen.treelstm_workload(1300, 1, 2, 320, 64, "uniform", seed=8, bias_scale=0.2, D=352)
    h, c = P.run_treelstm(ctx, w)
    d = {k: P.dev(w[k]) for k in ("emb", "W_leaf", "b_leaf", "U", "b")}
    h1, c1 = P.nan_filled(*h.shape), P.nan_filled(*c.shape)
    rc = ctx.acrobat_treelstm_forward_noalloc(w, 320, 352, 64, d["emb"], d["W_leaf"], d["b_leaf"], d["U"], d["b"], h1, c1,
                                              P.stream_handle())
    assert rc == A.OK
    assert np.array_equal(h1.cpu().numpy(), h) and np.array_equal(c1.cpu().numpy(), c)
