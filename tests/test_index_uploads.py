"""Index lists of more than 16 KB are read out of the staging buffer by a kernel: sizes around the line, lists that are not a
multiple of four long, two calls in a row on one context with other lists (the second rewrites the staging buffer)."""
import numpy as np
import pytest

import oracle
from workloads import generators as gen

pytestmark = pytest.mark.gpu

NT = oracle.default_threads()


@pytest.fixture(scope="module")
def ctx():
    import paper_2305_10611_amd as A
    c = A.Context(0)
    yield c
    c.close()


@pytest.mark.parametrize("rows", [2047, 2048, 2049, 2051, 9001])
def test_lists_around_the_line(ctx, rows):
    """Two lists of int32 per row.  Tolerance: 1e-6 over the 2-norm, fp32 sums of 64 products and two steps."""
    from tests import parity as P
    for seed in (1, 2):
        w = gen.lstm_workload(rows // 2, 2, 2, 32, 32, seed=seed)
        w["len"][seed] += rows % 2
        rng = np.random.default_rng(seed)
        w["len"] = rng.permutation(w["len"]).astype(np.int32)
        w["seq_off"] = np.concatenate([[0], np.cumsum(w["len"])]).astype(np.int64)
        w["x"] = rng.standard_normal((rows, 32), dtype=np.float32)
        got = P.run_lstm(ctx, w)
        for a, b in zip(got, oracle.varlen_lstm(w, nthreads=NT)):
            assert np.linalg.norm(a - b) < 1e-6 * np.linalg.norm(b)


@pytest.mark.parametrize("noalloc", [False, True])
def test_tree_lists(ctx, noalloc):
    import paper_2305_10611_amd as A
    from tests import parity as P
    for n in (273, 274, 701):  # trees of three leaves, three lists per node
        w = gen.treelstm_workload(n, 3, 3, 64, 50, "uniform", seed=n, bias_scale=0.2)
        want = oracle.treelstm(w, nthreads=NT)
        if noalloc:
            d = {k: P.dev(w[k]) for k in ("emb", "W_leaf", "b_leaf", "U", "b")}
            h, c = P.nan_filled(5 * n, 64), P.nan_filled(5 * n, 64)
            assert ctx.acrobat_treelstm_forward_noalloc(w, 64, 64, 50, d["emb"], d["W_leaf"], d["b_leaf"], d["U"], d["b"], h, c,
                                                        P.stream_handle()) == A.OK
            got = h.cpu().numpy(), c.cpu().numpy()
        else:
            got = P.run_treelstm(ctx, w)
        for a, b in zip(got, want):
            assert np.linalg.norm(a - b) < 1e-6 * np.linalg.norm(b)
