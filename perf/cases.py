"""What a user of this framework has it do, as cases that can be timed and checked.

A case is one mini-batch through one public entry point of the package: TreeLSTM (the specialised call, its
variant that allocates nothing, and the same model as a program of the generic dataflow-graph runtime), MV-RNN,
variable-length LSTM, bidirectional RNN and tree generation with a doubly recurrent network.  `prepare` makes what
a program holds before the call (structure arrays on the host; weights, tables, inputs and output arenas on the
GPU), `run` is one forward pass: host scheduling, index upload and every kernel launch.

Everything is fp32, as the framework is.  The sizes of a batch (leaf counts, sequence lengths) belong to the case,
so that its work does not depend on the seed; tree shapes, token ids, inputs and weights are drawn from the seed.
"""
from __future__ import annotations

import random

import numpy as np
import torch

import paper_2305_10611_amd as A
from paper_2305_10611_amd import binding as B

_CONTEXT = None


def _context():
    """One context per process, as a serving program keeps it: it owns the staging buffers and workspaces."""
    global _CONTEXT
    if _CONTEXT is None:
        _CONTEXT = A.Context(0)
    return _CONTEXT


# ---- the cases -------------------------------------------------------------------------------------------------
def _tree(name, api, n, lo, hi, H, D, V, zipf=True, bias=False):
    return {"name": name, "kind": "treelstm", "api": api, "n": n, "lo": lo, "hi": hi, "H": H, "D": D, "V": V,
            "zipf": zipf, "bias": bias}


def listed():
    return [
        # the smallest call: 8 short sentences, hidden size 256 - latency and launches count
        _tree("treelstm_h256_8x20", "forward", 8, 20, 20, 256, 256, 1000, zipf=False),
        # an ordinary mini-batch of sentences at the small hidden size, served without allocations
        _tree("treelstm_h256_64", "noalloc", 64, 10, 50, 256, 256, 20000, bias=True),
        # the workload of bench.py: 256 sentences at the large hidden size
        _tree("treelstm_h512_256", "forward", 256, 10, 60, 512, 512, 20000),
        # the largest: throughput inference over 1 024 sentences
        _tree("treelstm_h512_1024", "forward", 1024, 10, 60, 512, 512, 20000, bias=True),
        # odd sizes through the generic runtime: the unbatched program is built and bucketed for every mini-batch
        _tree("dfg_treelstm_h288_d160_77", "dfg", 77, 3, 45, 288, 160, 5000, bias=True),
        # matrix-vector networks, small and large model (a wide batch for the large one)
        {"name": "mvrnn_d64_64", "kind": "mvrnn", "n": 64, "lo": 10, "hi": 40, "d": 64, "copy": False},
        {"name": "mvrnn_d128_256", "kind": "mvrnn", "n": 256, "lo": 5, "hi": 35, "d": 128, "copy": False},
        # recurrent encoder over sequences of 1 to 100 steps
        {"name": "lstm_h512_256", "kind": "lstm", "n": 256, "lo": 1, "hi": 100, "H": 512, "D": 512, "bias": True},
        # the same with sizes for which there is no single-launch recurrence: one launch per step
        {"name": "lstm_h320_d96_75", "kind": "lstm", "n": 75, "lo": 1, "hi": 60, "H": 320, "D": 96, "bias": True},
        # bidirectional tagger, the large model at the batch size that it is usually run with
        {"name": "birnn_h512_64", "kind": "birnn", "n": 64, "lo": 5, "hi": 35, "H": 512, "D": 512, "n_out": 16},
        # the small model over a wide batch (more sequences than the single-launch recurrence takes)
        {"name": "birnn_h256_600", "kind": "birnn", "n": 600, "lo": 5, "hi": 35, "H": 256, "D": 256, "n_out": 50},
        # tree generation: control flow that waits for values, many short dependent evaluations
        {"name": "drnn_h512_64", "kind": "drnn", "n": 64, "H": 512, "n_out": 32, "decisions": 20230510},
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def _log_32(rng, lo, hi):  # a multiple of 32, which is what the framework takes
    return max(lo, min(hi, 32 * int(round(_log_int(rng, lo, hi) / 32))))


def draw(rng):
    kind = rng.choice(("treelstm", "treelstm", "mvrnn", "lstm", "birnn", "drnn"))
    most = 2.2e11  # flops; somewhat less than the largest listed case
    while True:
        lo = rng.randint(1, 20)
        hi = lo + rng.randint(0, 50)
        if kind == "treelstm":
            H, D = _log_32(rng, 64, 1024), _log_32(rng, 64, 1024)
            case = _tree("", rng.choice(("forward", "forward", "noalloc", "dfg")), _log_int(rng, 1, 1024), lo, hi, H, D,
                         _log_int(rng, 100, 20000), rng.random() < 0.7, rng.random() < 0.5)
        elif kind == "mvrnn":
            case = {"kind": kind, "n": _log_int(rng, 1, 512), "lo": lo, "hi": hi, "d": rng.choice((64, 128)),
                    "copy": rng.random() < 0.3}
            if case["n"] * (lo + hi) * case["d"] ** 2 > 512 * 40 * 64 ** 2 * 4:
                continue
        elif kind == "lstm":
            case = {"kind": kind, "n": _log_int(rng, 1, 512), "lo": rng.randint(0, 5), "hi": rng.randint(6, 100),
                    "H": rng.choice((128, 256, 512, _log_32(rng, 64, 768))), "D": _log_32(rng, 64, 768),
                    "bias": rng.random() < 0.5}
        elif kind == "birnn":
            case = {"kind": kind, "n": _log_int(rng, 1, 1024), "lo": rng.randint(0, 5), "hi": rng.randint(6, 60),
                    "H": rng.choice((128, 256, 512, _log_32(rng, 64, 768))), "D": _log_32(rng, 64, 768),
                    "n_out": _log_int(rng, 1, 200)}
        else:
            case = {"kind": kind, "n": _log_int(rng, 4, 128), "H": _log_32(rng, 64, 512), "n_out": rng.choice((32, 64)),
                    "decisions": rng.randint(1, 10 ** 9)}
            if case["n"] * case["H"] > 64 * 512:
                continue
        case.pop("name", None)
        if kind == "treelstm" and case["api"] == "noalloc" and case["n"] * (lo + hi) > 60000:
            continue
        if kind in ("treelstm", "lstm", "birnn") and case["n"] * (case["lo"] + case["hi"]) > 72000:
            continue
        if work(case)["flops"] <= most:
            return case


def _counts(case):
    """Leaf counts / sequence lengths of the batch: the case's own, whatever the seed."""
    key = random.Random(1000003 * case["n"] + 1009 * case["lo"] + case["hi"])
    c = [key.randint(case["lo"], case["hi"]) for _ in range(case["n"])]
    if max(c) == 0:
        c[0] = 1
    return np.asarray(c, np.int32)


def work(case):
    k = case["kind"]
    if k == "drnn":
        H, n_out = case["H"], case["n_out"]
        n = len(_forest(case)["inst"])
        return {"bytes": 4.0 * (case["n"] * H + _LABELS * H + 6 * H * H + n_out * H + n * (3 * H + n_out)),
                "flops": 2.0 * n * (6 * H * H + H * n_out)}
    c = _counts(case).astype(np.int64)
    leaves, internal, rows = int(c.sum()), int((c - 1).sum()), int(c.sum())
    if k == "treelstm":
        H, D = case["H"], case["D"]
        return {"bytes": 4.0 * (min(leaves, case["V"]) * D + 3 * H * D + 10 * H * H + 2 * H * (leaves + internal)),
                "flops": 6.0 * leaves * D * H + 20.0 * internal * H * H}
    if k == "mvrnn":
        d = case["d"]
        copied = 2 * leaves if case["copy"] else leaves
        return {"bytes": 4.0 * ((copied + internal) * (d * d + d) + 4 * d * d),
                "flops": internal * (4.0 * d ** 3 + 8.0 * d * d)}
    H, D = case["H"], case["D"]
    if k == "lstm":
        return {"bytes": 4.0 * (rows * D + 4 * H * (D + H) + 2 * rows * H), "flops": 8.0 * rows * H * (D + H)}
    n_out = case["n_out"]
    return {"bytes": 4.0 * (rows * D + 2 * H * (D + H) + 2 * n_out * H + 2 * rows * H + rows * n_out),
            "flops": 4.0 * rows * H * (D + H) + 4.0 * rows * H * n_out}


# ---- inputs ----------------------------------------------------------------------------------------------------
def _tree_shapes(counts, rng):
    """Random binary trees: a span of n leaves is cut at a uniform place; leaves first, internal nodes in
    post-order behind them (children before parents).  -> tree_off, left, right (tree-local ids)"""
    off, left, right = [0], [], []
    for n in counts.tolist():
        lt, rt = [-1] * (2 * n - 1), [-1] * (2 * n - 1)
        nxt = n
        done = []          # ids of finished subtrees
        todo = [(0, n)]
        while todo:
            lo, hi = todo.pop()
            if lo < 0:     # both children of this node are finished
                rt[nxt] = done.pop()
                lt[nxt] = done.pop()
                done.append(nxt)
                nxt += 1
            elif hi - lo == 1:
                done.append(lo)
            else:
                k = lo + 1 + int(rng.random() * (hi - lo - 1))
                todo += [(-1, 0), (k, hi), (lo, k)]
        left += lt
        right += rt
        off.append(len(left))
    return tuple(np.asarray(v, np.int32) for v in (off, left, right))


def _trees(case, rng):
    counts = _counts(case)
    off, left, right = _tree_shapes(counts, rng)
    token = np.full(len(left), -1, np.int32)
    leaf = left < 0
    n_leaf = int(leaf.sum())
    if case["kind"] == "mvrnn":  # every leaf has a matrix of its own
        token[leaf] = np.arange(n_leaf, dtype=np.int32)
    else:
        g = np.random.default_rng(rng.getrandbits(63))
        if case["zipf"]:         # word frequencies
            cdf = np.cumsum(np.arange(1, case["V"] + 1, dtype=np.float64) ** -1.1)
            token[leaf] = np.minimum(np.searchsorted(cdf / cdf[-1], g.random(n_leaf), side="right"), case["V"] - 1)
        else:
            token[leaf] = g.integers(0, case["V"], n_leaf)
    return {"n_trees": case["n"], "tree_off": off, "left": left, "right": right, "token": token}


class _Draw:
    def __init__(self, seed, device):
        self.device = device
        self.g = torch.Generator(device=device)
        self.g.manual_seed(seed)

    def normal(self, *shape):
        return torch.randn(*shape, generator=self.g, device=self.device)

    def uniform(self, bound, *shape):
        return (torch.rand(*shape, generator=self.g, device=self.device) * 2 - 1) * bound


_LABELS = 30


def _inputs(case, seed):
    """Structure (numpy) and tensors of a case; `exact` works from the same ones."""
    rng = random.Random(seed)
    d = _Draw(seed, "cuda")
    k = case["kind"]
    if k == "treelstm":
        H, D = case["H"], case["D"]
        b = H ** -0.5
        t = {"emb": d.normal(case["V"], D), "W_leaf": d.uniform(b, 5 * H, D), "U": d.uniform(b, 5 * H, 2 * H),
             "b_leaf": d.uniform(0.1, 5 * H) if case["bias"] else None, "b": d.uniform(0.1, 5 * H) if case["bias"] else None}
        return _trees(case, rng), t
    if k == "mvrnn":
        n = case["d"]
        s = _trees(case, rng)
        V = int((s["left"] < 0).sum())
        eye = torch.eye(n, device="cuda")
        return s, {"vec": d.normal(V, n), "mat": eye + 0.01 * d.normal(V, n, n), "W": d.uniform(n ** -0.5, n, 2 * n),
                   "WM": d.uniform(n ** -0.5, n, 2 * n)}
    if k == "drnn":
        H, n_out = case["H"], case["n_out"]
        t = {"x0": d.uniform(0.5, case["n"], H) + 0.5, "emb": d.normal(_LABELS, H)}
        for p in "afp":
            t["W" + p], t["b" + p] = d.uniform((2 * H) ** -0.5, H, 2 * H), d.uniform(0.1, H)
        t["Wo"], t["bo"] = d.uniform(H ** -0.5, n_out, H), d.uniform(0.1, n_out)
        return None, t
    H, D = case["H"], case["D"]
    lens = _counts(case).copy()
    lens = lens[np.random.default_rng(seed).permutation(len(lens))]
    R = int(lens.sum())
    if k == "lstm":
        return lens, {"x": d.normal(R, D), "Wx": d.uniform(H ** -0.5, 4 * H, D), "Wh": d.uniform(H ** -0.5, 4 * H, H),
                      "b": d.uniform(0.1, 4 * H) if case["bias"] else None}
    t = {"x": d.normal(R, D)}
    for p in "fb":
        t[p] = (d.uniform(H ** -0.5, H, D), d.uniform(H ** -0.5, H, H), d.uniform(0.1, H), d.uniform(0.5, H) + 0.5)
    t["C"], t["cb"] = d.uniform((2 * H) ** -0.5, case["n_out"], 2 * H), d.uniform(0.1, case["n_out"])
    return lens, t


def prepare(case, seed):
    ctx = _context()
    s, t = _inputs(case, seed)
    st = {"case": case, "ctx": ctx, "s": s, "t": t}
    new = lambda *shape: torch.zeros(*shape, device="cuda")
    k = case["kind"]
    if k == "treelstm":
        N, H, D = len(s["left"]), case["H"], case["D"]
        st["out"] = (new(N, H), new(N, H))
        if case["api"] == "dfg":
            h, c = st["out"]
            g = st["graph"] = A.Dfg(ctx)
            rc, st["leaf"] = g.acrobat_dfg_register_op(
                B.EPI_TREE_LEAF, H, nseg=1, kseg=D, src0=t["emb"], ld0=D, W=t["W_leaf"], ldw=D, bias=t["b_leaf"], h=h, c=c,
                src0_rows=case["V"], out_rows=N)
            ctx.check(rc)
            rc, st["internal"] = g.acrobat_dfg_register_op(
                B.EPI_TREE_INTERNAL, H, nseg=2, kseg=H, src0=h, ld0=H, src1=h, ld1=H, W=t["U"], ldw=2 * H, bias=t["b"],
                h=h, c=c, cprev_src=c, src0_rows=N, src1_rows=N, out_rows=N)
            ctx.check(rc)
    elif k == "mvrnn":
        N, d = len(s["left"]), case["d"]
        st["out"] = (new(N, d), new(N, d, d))  # leaf rows stay as they are unless they are asked for
    elif k == "drnn":
        # a user cannot know how many nodes will be generated: the outputs hold what this batch may reach
        cap = len(_forest(case)["inst"]) + 4096
        st["w"] = {"n_inst": case["n"], "H": case["H"], "n_labels": _LABELS, "n_out": case["n_out"],
                   "seed_decisions": case["decisions"], "cap": cap, **_GROW}
        st["out"] = (new(cap, case["H"]), new(cap, case["H"]), new(cap, case["H"]), new(cap, case["n_out"]))
    else:
        R, H = int(s.sum()), case["H"]
        st["out"] = (new(R, H), new(R, H)) + ((new(R, case["n_out"]),) if k == "birnn" else ())
    return st


def run(st):
    case, ctx, s, t, out = st["case"], st["ctx"], st["s"], st["t"], st["out"]
    k = case["kind"]
    stream = torch.cuda.current_stream().cuda_stream
    if k == "treelstm":
        H, D, V = case["H"], case["D"], case["V"]
        if case["api"] == "dfg":
            g = st["graph"]
            ctx.check(g.acrobat_dfg_clear())
            ctx.check(g.acrobat_dfg_build_treelstm(s, V, st["leaf"], st["internal"]))
            ctx.check(g.acrobat_dfg_run(stream))
        else:
            f = ctx.acrobat_treelstm_forward_noalloc if case["api"] == "noalloc" else ctx.acrobat_treelstm_forward
            ctx.check(f(s, H, D, V, t["emb"], t["W_leaf"], t["b_leaf"], t["U"], t["b"], out[0], out[1], stream))
        return {"h": out[0], "c": out[1]}
    if k == "mvrnn":
        ctx.check(ctx.acrobat_mvrnn_forward(s, case["d"], len(t["vec"]), t["vec"], t["mat"], t["W"], t["WM"], out[0], out[1],
                                            int(case["copy"]), stream))
        return {"vec": out[0], "mat": out[1]}
    if k == "lstm":
        ctx.check(ctx.acrobat_varlen_lstm_forward(s, case["H"], case["D"], t["x"], t["Wx"], t["Wh"], t["b"], out[0], out[1],
                                                  stream))
        return {"h": out[0], "c": out[1]}
    if k == "birnn":
        ctx.check(ctx.acrobat_birnn_forward(s, case["H"], case["D"], case["n_out"], t["x"], t["f"], t["b"], t["C"], t["cb"],
                                            out[0], out[1], out[2], stream))
        return {"hf": out[0], "hb": out[1], "y": out[2]}
    rc, trees, stats = ctx.acrobat_drnn_forward(st["w"], t["x0"], t, *out, stream=stream)
    ctx.check(rc)
    n = stats["n_nodes"]  # the rows behind the generated nodes hold nothing
    return {"a": out[0][:n], "f": out[1][:n], "g": out[2][:n], "y": out[3][:n], "trees": trees}


# ---- what the results should be --------------------------------------------------------------------------------
# Relative errors (2-norm) of the fp32 path against 64 bits as measured over the listed and some drawn cases, times
# four: treelstm 4.6e-7, mvrnn 2.6e-7, lstm 3.6e-7, birnn 3.2e-7, drnn 1.6e-7.  The states are sums of K terms in 32
# bits behind saturating gates; a recurrence does not let errors grow.
_TOLERANCE = {"treelstm": 1.8e-6, "mvrnn": 1.1e-6, "lstm": 1.5e-6, "birnn": 1.3e-6, "drnn": 7e-7}


def tolerance(case):
    return {"rel": _TOLERANCE[case["kind"]]}


def _lstm_gates(z, c):  # gates (i, f, o, u)
    i, f, o, u = z.chunk(4, 1)
    c = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(u)
    return torch.sigmoid(o) * torch.tanh(c), c


def _depths(s):
    """Depth of every node (leaves 0), and the children's global ids."""
    base = np.repeat(s["tree_off"][:-1], np.diff(s["tree_off"]))
    l, r = s["left"] + base, s["right"] + base
    depth = np.zeros(len(base), np.int64)
    for g in np.flatnonzero(s["left"] >= 0):  # children come before their parents
        depth[g] = 1 + max(depth[l[g]], depth[r[g]])
    return depth, l, r


def exact(case, seed):
    s, t32 = _inputs(case, seed)
    f64 = lambda v: tuple(f64(u) for u in v) if isinstance(v, tuple) else (None if v is None else v.double())
    t = {k: f64(v) for k, v in t32.items()}
    dev = lambda a: torch.as_tensor(np.ascontiguousarray(a), device="cuda").long()
    k = case["kind"]
    if k in ("treelstm", "mvrnn"):
        depth, l, r = _depths(s)
        N = len(depth)
        order = np.argsort(depth, kind="stable")
        levels = np.split(order, np.cumsum(np.bincount(depth))[:-1])
        tok = dev(s["token"][levels[0]])
    if k == "treelstm":
        H = case["H"]
        h, c = (torch.zeros(N, H, dtype=torch.float64, device="cuda") for _ in range(2))
        zero = torch.zeros(5 * H, dtype=torch.float64, device="cuda")
        for lv, ids in enumerate(levels):
            at, li, ri = dev(ids), dev(l[ids]), dev(r[ids])
            if lv == 0:
                z = t["emb"][tok] @ t["W_leaf"].T + (zero if t["b_leaf"] is None else t["b_leaf"])
            else:
                z = torch.cat([h[li], h[ri]], 1) @ t["U"].T + (zero if t["b"] is None else t["b"])
            i, fl, fr, o, u = z.chunk(5, 1)
            cc = torch.sigmoid(i) * torch.tanh(u)
            if lv:
                cc = cc + torch.sigmoid(fl) * c[li] + torch.sigmoid(fr) * c[ri]
            c[at], h[at] = cc, torch.sigmoid(o) * torch.tanh(cc)
        return {"h": h, "c": c}
    if k == "mvrnn":
        d = case["d"]
        vec, mat = (torch.zeros(N, *x, dtype=torch.float64, device="cuda") for x in ((d,), (d, d)))
        leaf = dev(levels[0])
        vec[leaf], mat[leaf] = t["vec"][tok], t["mat"][tok]
        for ids in levels[1:]:
            at, li, ri = dev(ids), dev(l[ids]), dev(r[ids])
            mv = lambda m, v: (m * v[:, None, :]).sum(2)
            x = torch.cat([mv(mat[ri], vec[li]), mv(mat[li], vec[ri])], 1)
            vec[at] = torch.tanh(x @ t["W"].T)
            # W_M [A ; B] as plain products: the left half acts on A, the right half on B
            flat = lambda m: m.transpose(0, 1).reshape(d, -1)
            p = t["WM"][:, :d] @ flat(mat[li]) + t["WM"][:, d:] @ flat(mat[ri])
            mat[at] = p.reshape(d, len(ids), d).transpose(0, 1)
        if not case["copy"]:
            vec[leaf], mat[leaf] = 0, 0
        return {"vec": vec, "mat": mat}
    if k == "drnn":
        F = _forest(case)
        n, H = len(F["inst"]), case["H"]
        a, f, g = (torch.zeros(n, H, dtype=torch.float64, device="cuda") for _ in range(3))
        level = np.zeros(n, np.int64)
        for i in range(n):
            level[i] = 1 + max(level[F[q][i]] if F[q][i] >= 0 else -1 for q in ("parent", "prev"))
        label = np.asarray(F["label"])
        for lv in range(int(level.max()) + 1):
            ids = np.flatnonzero(level == lv)
            par, prev = np.asarray(F["parent"])[ids], np.asarray(F["prev"])[ids]
            pick = lambda m, at: dev(np.where(m >= 0, at, 0))
            ap = torch.where(dev(par)[:, None] >= 0, a[pick(par, par)], t["x0"][dev(np.asarray(F["inst"])[ids])])
            fp = torch.where(dev(prev)[:, None] >= 0, f[pick(prev, prev)], torch.zeros_like(ap))
            la, lf = pick(par, label[par]), pick(prev, label[prev])
            an = torch.sigmoid(torch.cat([ap, t["emb"][la]], 1) @ t["Wa"].T + t["ba"])
            fn = torch.sigmoid(torch.cat([fp, t["emb"][lf]], 1) @ t["Wf"].T + t["bf"])
            at = dev(ids)
            a[at], f[at] = an, fn
            g[at] = torch.sigmoid(torch.cat([an, fn], 1) @ t["Wp"].T + t["bp"])
        return {"a": a, "f": f, "g": g, "y": g @ t["Wo"].T + t["bo"],
                "trees": {q: np.asarray(F[q], np.int32) for q in B.DRNN_TREE_FIELDS}}
    H, lens = case["H"], s
    off = np.concatenate([[0], np.cumsum(lens)])[:-1]
    R = int(lens.sum())
    zeros = lambda: torch.zeros(R, H, dtype=torch.float64, device="cuda")
    if k == "lstm":
        xp = t["x"] @ t["Wx"].T + (0 if t["b"] is None else t["b"])
        h, c = zeros(), zeros()
        for step in range(int(lens.max())):
            live = np.flatnonzero(lens > step)
            at = dev(off[live] + step)
            z = xp[at]
            cp = torch.zeros(len(live), H, dtype=torch.float64, device="cuda")
            if step:
                z, cp = z + h[at - 1] @ t["Wh"].T, c[at - 1]
            h[at], c[at] = _lstm_gates(z, cp)
        return {"h": h, "c": c}
    hs = []
    for p in "fb":
        Wx, Wh, b, init = t[p]
        xp, h = t["x"] @ Wx.T + b, zeros()
        for step in range(int(lens.max())):
            live = np.flatnonzero(lens > step)
            row = off[live] + (step if p == "f" else lens[live] - 1 - step)
            at = dev(row)
            prev = h[at + (-1 if p == "f" else 1)] if step else init.expand(len(live), H)
            h[at] = torch.sigmoid(xp[at] + prev @ Wh.T)
        hs.append(h)
    return {"hf": hs[0], "hb": hs[1], "y": torch.relu(torch.cat(hs, 1) @ t["C"].T + t["cb"])}


# ---- the trees that a generation call grows ---------------------------------------------------------------------
_GROW = {"max_depth": 6, "max_children": 4, "p_child": 0.7, "p_sibling": 0.6}
_M64 = (1 << 64) - 1


def _mix(z):  # splitmix64
    z = (z + 0x9E3779B97F4A7C15) & _M64
    z = ((z ^ (z >> 30)) * 0xBF58476D1CE4E5B9) & _M64
    z = ((z ^ (z >> 27)) * 0x94D049BB133111EB) & _M64
    return z ^ (z >> 31)


_FORESTS = {}


def _forest(case):
    """Structure of the generated trees in the order in which the nodes are created: the decisions are emulated from
    a node's position, instances and subtrees run as cooperative threads, first come first served, each of which
    waits after every node for the next evaluation."""
    key = (case["n"], case["decisions"])
    if key in _FORESTS:
        return _FORESTS[key]
    F = {q: [] for q in B.DRNN_TREE_FIELDS}
    p_child, p_sibling = float(np.float32(_GROW["p_child"])), float(np.float32(_GROW["p_sibling"]))
    unit = lambda bits: (bits >> 11) / 9007199254740992.0
    ready, evaluation = [], [0]

    def node(inst, parent, prev, k, depth, key):
        i = len(F["inst"])
        for q, v in zip(B.DRNN_TREE_FIELDS, (inst, parent, prev, k, depth, _mix(key ^ 3) % _LABELS, evaluation[0])):
            F[q].append(v)
        child = depth + 1 < _GROW["max_depth"] and unit(_mix(key ^ 1)) < p_child
        more = parent >= 0 and k + 1 < _GROW["max_children"] and unit(_mix(key ^ 2)) < p_sibling
        return i, child, more

    def children(inst, parent, pkey, pdepth):
        while True:
            prev, last, k = -1, None, 0
            while True:
                key = _mix((pkey + k + 1) & _M64)
                i, child, more = node(inst, parent, prev, k, pdepth + 1, key)
                yield
                if child and more:
                    ready.append(children(inst, i, key, pdepth + 1))
                elif child:
                    last = (i, key)
                if not more:
                    break
                prev, k = i, k + 1
            if last is None:
                return
            (parent, pkey), pdepth = last, pdepth + 1

    def instance(inst):
        key = _mix(case["decisions"] ^ _mix(inst))
        i, child, _ = node(inst, -1, -1, 0, 0, key)
        yield
        if child:
            yield from children(inst, i, key, 0)

    ready = [instance(s) for s in range(case["n"])]
    while ready:
        blocked = []
        while ready:
            f = ready.pop(0)
            try:
                next(f)
                blocked.append(f)
            except StopIteration:
                pass
        ready += blocked
        evaluation[0] += 1
    if len(_FORESTS) > 64:
        _FORESTS.clear()
    _FORESTS[key] = F
    return F
