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


def on_packed_operands(run):
    """What run() returns; one launch of the kernel whose operands arrive packed does the levels or steps."""
    from tests import parity as P
    out = []
    names = P.kernels_of(lambda: out.append(run()))
    assert any("cell_packed_kernel" in k for k in names), names
    assert not any("kernel<5" in k for k in names if "cell_packed" not in k), names  # (five gates: internal tree levels)
    return out[-1]


# Chains of twelve leaves: m trees a group are a share of m rows at every level - one row, a whole block of 16, one row more or
# less, two blocks.  16 groups, four wavefronts and one row block a round (H = 256), 8 groups, eight and two (288, 512).
@pytest.mark.gpu
@pytest.mark.parametrize("H,groups", [(256, 16), (288, 8), (512, 8)])
@pytest.mark.parametrize("m", [1, 15, 16, 17, 31, 32, 33])
def test_tree_shares_around_whole_blocks(ctx, H, groups, m):
    import oracle
    from tests import parity as P
    from workloads import generators as gen
    leaves, n = 12, groups * m
    rng = gen.make_rng(H + m)
    w = gen.treelstm_workload(n, 2, 2, H, 60, "uniform", seed=H + m, bias_scale=0.2, D=64)
    chain, leaf = np.r_[0, leaves:2 * leaves - 2], np.arange(1, leaves)
    sides = rng.integers(0, 2, (n, leaves - 1)).astype(bool)
    none = np.full((n, leaves), -1)
    w.update(tree_off=np.arange(n + 1, dtype=np.int32) * (2 * leaves - 1),
             left=np.hstack([none, np.where(sides, leaf, chain)]).astype(np.int32).ravel(),
             right=np.hstack([none, np.where(sides, chain, leaf)]).astype(np.int32).ravel())
    w["token"] = np.where(w["left"] < 0, rng.integers(0, 60, w["left"].size), -1).astype(np.int32)
    h, c = on_packed_operands(lambda: P.run_treelstm(ctx, w))
    level_off, _ = ctx.acrobat_last_schedule()
    assert set(np.diff(level_off)[1:]) == {n}
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
        h, c = on_packed_operands(lambda: P.run_lstm(ctx, w))
        oh, oc = oracle.varlen_lstm(w, nthreads=oracle.default_threads())
        assert rel(h, oh) < 1e-6 and rel(c, oc) < 1e-6
    else:
        w = gen.birnn_workload(n, 1, 9, H, 32, 5, seed=H + n)
        hf, hb, y = on_packed_operands(lambda: P.run_birnn(ctx, w))
        of, ob, oy = oracle.birnn(w, nthreads=oracle.default_threads())
        assert rel(hf, of) < 1e-6 and rel(hb, ob) < 1e-6 and rel(y, oy) < 2e-6


@pytest.mark.gpu
@pytest.mark.parametrize("kind,H,n", [("lstm", 320, 40), ("lstm", 512, 140), ("birnn", 512, 70), ("birnn", 320, 40),
                                      ("birnn", 512, 300), ("tree", 256, 40), ("tree", 512, 60)])
def test_sums_that_are_not_to_be_split(ctx, kind, H, n):
    """A unit of next to nothing that is read with weights of 1e5 to 1e8, beside ordinary ones: all terms count alike, and fp32
    dot products of the arena's rows keep them.  Split sums would be off by 2e-04 (LSTM, H = 320, the split's arithmetic in 64
    bits).  Tolerance: as everywhere here; the small state itself has 21 2^-24 = 1e-6 from its gate's argument, and is one term."""
    import oracle
    from tests import parity as P
    from workloads import generators as gen
    if kind == "lstm":  # unit 7: its output gate is next to closed
        w = gen.lstm_workload(n, 1, 7, H, 32, seed=3, bias_scale=0.2)
        w["b"][2 * H + 7] -= np.float32(21.0)
        w["Wh"][:, 7] *= np.float32(1e9)
        w["Wh"][2 * H + 7, 7] *= np.float32(1e-9)
        run, want = P.run_lstm, oracle.varlen_lstm
    elif kind == "birnn":
        w = gen.birnn_workload(n, 1, 7, H, 32, 5, seed=3)
        for d in "fb":
            w[d + "b"][7] -= np.float32(21.0)
            w[d + "init"][7] *= np.float32(1e-9)
            w[d + "Wh"][:, 7] *= np.float32(1e9)
        run, want = P.run_birnn, oracle.birnn
    else:  # unit 0: its output gate is next to closed
        w = gen.treelstm_workload(n, 10, 33, H, 100, "uniform", seed=17, bias_scale=0.2, D=64)
        w["b_leaf"][3 * H], w["b"][3 * H] = -15, -15
        w["U"][:, 0], w["U"][:, H] = 1e6 * np.sign(w["U"][:, 0]), 1e6 * np.sign(w["U"][:, H])
        run, want = P.run_treelstm, oracle.treelstm
    got = on_packed_operands(lambda: run(ctx, w))
    for a, b in zip(got, want(w, nthreads=oracle.default_threads())):
        assert rel(a, b) < 1e-6
