"""One-launch trees and recurrences whose operands travel packed: the host's places on the CPU, the kernels against the
oracle at the sizes where a rule changes sides or a block is not full.

Tolerance as in test_split_contraction: 1e-6 over the 2-norm of all states (sqrt(K) 2^-24 per pre-activation, about 1e-6 at
K = 512, which the gates halve at least)."""
import os

import numpy as np
import pytest

from tests.test_sanitizers import CSRC, ROOT, build_and_run


def test_places_are_where_the_reader_looks(tmp_path):
    src = [os.path.join(ROOT, "tests", "sanitize", "places_driver.cpp"), os.path.join(CSRC, "scheduler.cpp")]
    build_and_run(tmp_path, "g++", "-std=c++17", src, "places_driver", [])


def rel(got, want):
    want = want.astype(np.float64)
    return float(np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want))


@pytest.fixture(scope="module")
def ctx():
    import paper_2305_10611_amd as A
    c = A.Context(0)
    yield c
    c.close()


# shares of a level of 1, 15 .. 17, 31 .. 33 rows and more: complete trees of 2^k leaves in 8 or 16 groups; four wavefronts and
# one row block a round (H <= 256) or eight and two (above)
@pytest.mark.gpu
@pytest.mark.parametrize("H,n,leaves", [(96, 16, 16), (256, 8, 34), (256, 33, 32), (288, 8, 32), (288, 8, 34), (512, 8, 66),
                                        (512, 9, 130), (512, 31, 8)])
def test_tree_shares_around_whole_blocks(ctx, H, n, leaves):
    import oracle
    from tests import parity as P
    from workloads import generators as gen
    w = gen.treelstm_workload(n, leaves, leaves, H, 60, "uniform", seed=H + leaves, bias_scale=0.2, D=64)
    h, c = P.run_treelstm(ctx, w)
    oh, oc = oracle.treelstm(w, nthreads=oracle.default_threads())
    assert rel(h, oh) < 1e-6 and rel(c, oc) < 1e-6


# one row block a group and 16 units a workgroup up to 128 (LSTM, H = 512), 256 (H = 192, 256) and 192 (BiRNN, H = 320), 96
# (H = 512, more units from there on) sequences
@pytest.mark.gpu
@pytest.mark.parametrize("kind,H,n", [("lstm", 512, 128), ("lstm", 512, 129), ("lstm", 192, 257), ("lstm", 256, 17),
                                      ("lstm", 288, 300), ("lstm", 128, 260), ("birnn", 512, 65), ("birnn", 512, 129),
                                      ("birnn", 512, 300), ("birnn", 320, 97), ("birnn", 320, 500), ("birnn", 224, 700),
                                      ("birnn", 160, 33), ("birnn", 128, 1100)])
def test_recurrences_around_the_rules(ctx, kind, H, n):
    import oracle
    from tests import parity as P
    from workloads import generators as gen
    if kind == "lstm":
        w = gen.lstm_workload(n, 1, 9, H, 32, seed=H + n, bias_scale=0.2)
        h, c = P.run_lstm(ctx, w)
        oh, oc = oracle.varlen_lstm(w, nthreads=oracle.default_threads())
        assert rel(h, oh) < 1e-6 and rel(c, oc) < 1e-6
    else:
        w = gen.birnn_workload(n, 1, 9, H, 32, 5, seed=H + n)
        hf, hb, y = P.run_birnn(ctx, w)
        of, ob, oy = oracle.birnn(w, nthreads=oracle.default_threads())
        assert rel(hf, of) < 1e-6 and rel(hb, ob) < 1e-6 and rel(y, oy) < 2e-6


@pytest.mark.gpu
def test_weights_that_are_not_to_be_split(ctx):
    """Recurrent weights of 1e5 and 1e-5 in one row: such sums are plain fp32 dot products of the arena's rows."""
    import oracle
    from tests import parity as P
    from workloads import generators as gen
    w = gen.lstm_workload(40, 1, 7, 320, 32, seed=3, bias_scale=0.2)
    w["Wh"][5::64, 7] = 1e5
    h, c = P.run_lstm(ctx, w)
    oh, oc = oracle.varlen_lstm(w, nthreads=oracle.default_threads())
    # (a state next to zero times 1e5 is 2^-24 times that off: gates are compared where the large term does not decide)
    assert np.isfinite(h).all() and rel(h, oh) < 2e-3 and rel(c, oc) < 2e-3
