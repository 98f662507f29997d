"""Which kernel takes a call, where neither its results nor its launch records tell, and calls at the limits of the room that
packed operands and packed rows have: against the oracle at 1e-6 over the 2-norm (as in test_split_contraction)."""
import numpy as np
import pytest

import oracle
from workloads import generators as gen

pytestmark = pytest.mark.gpu

NT = oracle.default_threads()


def rel(got, want):
    want = want.astype(np.float64)
    return float(np.linalg.norm(got.astype(np.float64) - want) / np.linalg.norm(want))


@pytest.fixture()
def ctx():
    """A context of its own for every test: what calls before it have made room for counts."""
    import paper_2305_10611_amd as A
    c = A.Context(0)
    yield c
    c.close()


def test_captured_leaves_without_room_for_packed_rows(ctx):
    """The call before the capture has leaves too narrow for the packed product: the captured one takes the kernel that
    needs no room, not the level kernels."""
    import torch
    import paper_2305_10611_amd as A
    from tests import parity as P
    make = lambda D: gen.treelstm_workload(340, 3, 3, 512, 60, "uniform", seed=5, bias_scale=0.2, D=D)
    P.run_treelstm(ctx, make(32))
    w = make(512)
    t = {k: P.dev(w[k]) for k in ("emb", "W_leaf", "b_leaf", "U", "b")}
    h, c = P.nan_filled(5 * 340, 512), P.nan_filled(5 * 340, 512)
    st, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=st, capture_error_mode="relaxed"):
        rc = ctx.acrobat_treelstm_forward(w, 512, 512, 60, t["emb"], t["W_leaf"], t["b_leaf"], t["U"], t["b"], h, c, st.cuda_stream)
    assert rc == A.OK, ctx.acrobat_last_error()
    want = oracle.treelstm(w, nthreads=NT)
    for _ in range(2):
        h.fill_(float("nan")); c.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        assert rel(h.cpu().numpy(), want[0]) < 1e-6 and rel(c.cpu().numpy(), want[1]) < 1e-6
    # the profiler does not see a replay's kernels, but a leaf's bits do not depend on the rest of the batch: 90 leaves
    few = dict(w, n_trees=30, tree_off=w["tree_off"][:31])
    few.update({k: w[k][:150] for k in ("left", "right", "token")})
    got = h.cpu().numpy()[:150]
    del g
    names = P.kernels_of(lambda: few.update(h=P.run_treelstm(ctx, few)[0]))
    assert any("cell_stationary_kernel<3," in k for k in names), names
    assert np.array_equal(got, few["h"])


@pytest.mark.parametrize("n,leaves,H,D,mixed", [(700, 6, 512, 512, False), (2330, 6, 512, 512, False), (90, 46, 256, 1024, False),
                                                (2, 2100, 512, 256, False), (700, 6, 512, 512, True)])
def test_leaves_without_allocations_have_the_ordinary_bits(ctx, n, leaves, H, D, mixed):
    """4 200 leaves, whose packed rows take 8.6 MB of the fixed array, 13 980, which run in two pieces, 17 MB of rows at D = 1 024,
    and two trees whose wide levels run on split weights beside them.  mixed: a third of the rows are not to be split, and the
    calls list the leaves in different orders."""
    import paper_2305_10611_amd as A
    from tests import parity as P
    w = gen.treelstm_workload(n, leaves, leaves, H, 500, "uniform", seed=n, bias_scale=0.2, D=D)
    if mixed:
        w["emb"][::3, 3] *= 1e9
        w["W_leaf"][:, 3] *= 1e-9
    h, c = P.run_treelstm(ctx, w)
    d = {k: P.dev(w[k]) for k in ("emb", "W_leaf", "b_leaf", "U", "b")}
    out = [P.nan_filled(*h.shape) for _ in range(2)]
    names = P.kernels_of(lambda: ctx.check(ctx.acrobat_treelstm_forward_noalloc(
        w, H, D, 500, d["emb"], d["W_leaf"], d["b_leaf"], d["U"], d["b"], *out, P.stream_handle())))
    assert ctx.acrobat_device_status() == A.OK
    assert any("cell_dense_kernel<3," in k for k in names), names
    assert np.array_equal(out[0].cpu().numpy(), h) and np.array_equal(out[1].cpu().numpy(), c)
    few = slice(0, (2 * leaves - 1) * min(n, 60))
    part = dict(w, n_trees=min(n, 60), tree_off=w["tree_off"][:min(n, 60) + 1], **{k: w[k][few] for k in ("left", "right", "token")})
    oh, oc = oracle.treelstm(part, nthreads=NT)
    assert rel(h[few], oh) < 1e-6 and rel(c[few], oc) < 1e-6


@pytest.mark.parametrize("n,H,seed,levels", [(64, 256, 6, 16), (40, 512, 7, None), (110, 256, 1, None)])
def test_sentences_without_allocations_run_on_packed_levels(ctx, n, H, seed, levels):
    """Also where they are deep, or their leaves' packed rows (110) or 128 KiB a block (H = 512) leave less room for the levels."""
    import paper_2305_10611_amd as A
    from tests import parity as P
    w = gen.treelstm_workload(n, 10, 50, H, 500, "uniform", seed=seed, bias_scale=0.2)
    h, c = P.run_treelstm(ctx, w)
    if levels:
        assert len(ctx.acrobat_last_schedule()[0]) - 1 == levels
    d = {k: P.dev(w[k]) for k in ("emb", "W_leaf", "b_leaf", "U", "b")}
    out = [P.nan_filled(*h.shape) for _ in range(2)]
    names = P.kernels_of(lambda: ctx.check(ctx.acrobat_treelstm_forward_noalloc(
        w, H, H, 500, d["emb"], d["W_leaf"], d["b_leaf"], d["U"], d["b"], *out, P.stream_handle())))
    assert ctx.acrobat_device_status() == A.OK
    assert any("cell_packed_kernel<5," in k for k in names), names
    assert np.array_equal(out[0].cpu().numpy(), h) and np.array_equal(out[1].cpu().numpy(), c)
    want = oracle.treelstm(w, nthreads=NT)
    assert rel(h, want[0]) < 1e-6 and rel(c, want[1]) < 1e-6


@pytest.mark.parametrize("kind,H,lens", [("lstm", 512, [1000] + [1] * 1999), ("lstm", 320, [9000] * 4 + [1] * 252),
                                         ("lstm", 512, [9000] * 4 + [1] * 252), ("birnn", 512, [4500] * 4 + [2, 1] * 126)])
def test_few_long_sequences_among_many_short_ones(ctx, kind, H, lens):
    """One launch, and no more workspace than a batch of that width needs: a step's packed states last until the next step has
    read them.  Against a launch per step (2e-6, as in test_split_contraction), which needs none."""
    import torch
    import paper_2305_10611_amd as A
    from tests import parity as P
    lens = gen.make_rng(H).permutation(np.asarray(lens, np.int32))
    w = gen.lstm_workload(4, 1, 2, H, 32, seed=H, bias_scale=0.2) if kind == "lstm" else gen.birnn_workload(4, 1, 2, H, 32, 5, seed=H)
    R = int(lens.sum())
    w.update(len=lens, n_seq=len(lens), x=gen.make_rng(H + 1).standard_normal((R, 32), dtype=np.float32))
    run = P.run_lstm if kind == "lstm" else P.run_birnn
    ctx.acrobat_set_persistent(False)
    steps = run(ctx, w)  # (input products, lists and partial tiles have their room now)
    ctx.acrobat_set_persistent(True)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    got = []
    names = P.kernels_of(lambda: got.extend(run(ctx, w)))
    assert ctx.acrobat_device_status() == A.OK
    taken = free - torch.cuda.mem_get_info()[0]
    assert sum("cell_packed_kernel" in k for k in names) == 1 and not any("cell_direct" in k or "cell_tiny" in k for k in names), names
    assert taken < 64 << 20, taken
    for a, b in zip(got, steps):
        assert rel(a, b) < 2e-6


@pytest.mark.parametrize("deep,few,kernel", [(3000, 255, "cell_stationary_kernel<5,"), (120, 15, "cell_packed_kernel<5,")])
def test_one_deep_tree_among_small_ones(ctx, deep, few, kernel):
    """A chain of 3 000 levels beside 255 trees of two leaves: packed operands would take 4 GB for states of 28 MB, so rows are
    gathered.  Of 120 beside 15: they take over 100 times the states as well, but fit the caches."""
    import torch
    import paper_2305_10611_amd as A
    from tests import parity as P
    H = 512
    w = gen.treelstm_workload(few + 1, 2, 2, H, 60, "uniform", seed=4, bias_scale=0.2, D=64)
    rng = gen.make_rng(6)
    chain = np.arange(deep, dtype=np.int32)  # node deep + 1 + i has node deep + i (node 0: a leaf) and leaf i + 1 as children
    left = np.concatenate([np.full(deep + 1, -1, np.int32), [0], deep + 1 + chain[:-1]]).astype(np.int32)
    right = np.concatenate([np.full(deep + 1, -1, np.int32), 1 + chain]).astype(np.int32)
    token = np.where(left < 0, rng.integers(0, 60, 2 * deep + 1), -1).astype(np.int32)
    w = dict(w, tree_off=np.concatenate([w["tree_off"][:-1], [3 * few + 2 * deep + 1]]).astype(np.int32),
             **{k: np.concatenate([w[k][:3 * few], v]) for k, v in (("left", left), ("right", right), ("token", token))})
    ctx.acrobat_set_persistent(False)
    P.run_treelstm(ctx, w)  # (lists and partial tiles have their room now)
    ctx.acrobat_set_persistent(True)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    got = []
    names = P.kernels_of(lambda: got.extend(P.run_treelstm(ctx, w)))
    assert ctx.acrobat_device_status() == A.OK
    assert free - torch.cuda.mem_get_info()[0] < 384 << 20
    assert any(kernel in k for k in names) and any("cell_packed" in k for k in names) == ("packed" in kernel), names
    want = oracle.treelstm(w, nthreads=NT)
    assert rel(got[0], want[0]) < 1e-6 and rel(got[1], want[1]) < 1e-6


@pytest.mark.parametrize("kind,H,n,kernel", [("birnn", 512, 70, "cell_packed_kernel"), ("birnn", 512, 256, "cell_packed_kernel"),
                                             ("birnn", 512, 64, "rnn_persistent_kernel"), ("lstm", 256, 40, "cell_packed_kernel"),
                                             ("lstm", 128, 40, "lstm_persistent_kernel")])
def test_captured_recurrences_of_one_launch(ctx, kind, H, n, kernel):
    """The eager call's kernel and its bits, replay after replay, with other work of the program in between."""
    import torch
    import paper_2305_10611_amd as A
    from tests import parity as P
    w = (gen.lstm_workload(n, 1, 9, H, 32, seed=3, bias_scale=0.2) if kind == "lstm" else gen.birnn_workload(n, 1, 9, H, 32, 5, seed=3))
    ref = []
    names = P.kernels_of(lambda: ref.append((P.run_lstm if kind == "lstm" else P.run_birnn)(ctx, w)))
    assert any(kernel in k for k in names), names
    g, out, keep = captured(ctx, w, kind)
    other = torch.zeros(1 << 20, device="cuda")
    for _ in range(3):
        for o in out:
            o.fill_(float("nan"))
        other.add_(1.0)
        g.replay()
        torch.cuda.synchronize()
        for o, r in zip(out, ref[-1]):
            assert np.array_equal(o.cpu().numpy(), r)
    assert ctx.acrobat_device_status() == A.OK


def test_captured_lstm_with_room_for_two_steps_states_only(ctx):
    """The call before the capture is wider and keeps two sets of packed states; this one would keep all steps': same bits."""
    import torch
    import paper_2305_10611_amd as A
    from tests import parity as P
    w = gen.lstm_workload(40, 30, 40, 512, 32, seed=3, bias_scale=0.2)
    other = A.Context(0)
    want = P.run_lstm(other, w)
    other.close()
    P.run_lstm(ctx, gen.lstm_workload(256, 60, 100, 512, 32, seed=4, bias_scale=0.2))
    g, out, keep = captured(ctx, w, "lstm")
    for _ in range(3):
        for o in out:
            o.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        for o, r in zip(out, want):
            assert np.array_equal(o.cpu().numpy(), r), np.flatnonzero((o.cpu().numpy() != r).any(axis=1))
    assert ctx.acrobat_device_status() == A.OK


def test_captured_lstm_without_room_for_packed_states(ctx):
    """H = 256: the older kernel, which needs none, takes the call in one launch (recorded once more without polls, it gives up
    and says so)."""
    import torch
    import paper_2305_10611_amd as A
    from tests import parity as P
    w = gen.lstm_workload(40, 1, 9, 256, 32, seed=3, bias_scale=0.2)
    ctx.acrobat_set_persistent(False)
    P.run_lstm(ctx, w)  # (a launch per step)
    want = oracle.varlen_lstm(w, nthreads=NT)
    ctx.acrobat_set_persistent(True)
    g, out, keep = captured(ctx, w, "lstm")
    for _ in range(3):
        for o in out:
            o.fill_(float("nan"))
        g.replay()
        torch.cuda.synchronize()
        for o, r in zip(out, want):
            assert rel(o.cpu().numpy(), r) < 1e-6
    assert ctx.acrobat_device_status() == A.OK
    ctx.acrobat_set_persistent(True, 0)
    g, out, keep = captured(ctx, w, "lstm")
    g.replay()
    torch.cuda.synchronize()
    assert ctx.acrobat_device_status() == A.ETIMEOUT


def captured(ctx, w, kind):
    """A call recorded into a graph -> the graph, its outputs, what it reads."""
    import torch
    import paper_2305_10611_amd as A
    from tests import parity as P
    R, H, D = int(np.sum(w["len"])), int(w["H"]), int(w["D"])
    st, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    names = ("x", "Wx", "Wh", "b") if kind == "lstm" else ("x", "fWx", "fWh", "fb", "finit", "bWx", "bWh", "bb", "binit", "C", "cb")
    t = {k: P.dev(np.asarray(w[k], np.float32)) for k in names}
    out = [P.nan_filled(R, H), P.nan_filled(R, H)] + ([] if kind == "lstm" else [P.nan_filled(R, int(w["n_out"]))])
    torch.cuda.synchronize()
    with torch.cuda.graph(g, stream=st, capture_error_mode="relaxed"):
        if kind == "lstm":
            rc = ctx.acrobat_varlen_lstm_forward(w["len"], H, D, t["x"], t["Wx"], t["Wh"], t["b"], *out, st.cuda_stream)
        else:
            rc = ctx.acrobat_birnn_forward(w["len"], H, D, int(w["n_out"]), t["x"], tuple(t["f" + k] for k in ("Wx", "Wh", "b", "init")),
                                           tuple(t["b" + k] for k in ("Wx", "Wh", "b", "init")), t["C"], t["cb"], *out, st.cuda_stream)
    assert rc == A.OK, ctx.acrobat_last_error()
    return g, out, t
