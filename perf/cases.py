"""Performance cases of the library: what a program does with it, through its
public entry points, over the range of sizes it is used at.

A case is a dict of plain values; ``kind`` names the path:

  lstm       recurrence stack, forward and backward through time, for a given
             gradient of its output (janus_lstm_seq_fwd / _bwd)
  lstm_eval  recurrence stack, forward only (evaluation, feature extraction)
  lm         whole language-model training step: embedding, recurrence stack,
             softmax cross-entropy head, all gradients (LSTMStep)
  treelstm, treernn, childsum
             whole training step over a batch of trees, 5-class softmax at
             the roots, all gradients (TreeStep, TreeRNNStep, ChildSumStep)
  mse        per-row projection with mean squared error, all gradients
             (janus_linear_mse)
  sgd        parameter update with global-norm clipping
             (janus_sgd_clip_update)

Inputs are seeded draws with the distributions of the library's workloads:
data N(0, 1), weights U(-a, a), Zipf(1.1) word ids, random trees.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1812_01329_amd import janus as J
from paper_1812_01329_amd import train_step as ts
from paper_1812_01329_amd import workloads as wl

DEV = "cuda"


def listed():
    return [
        # the smallest training call: a toy LSTM, where launches and latency count
        dict(name="lstm_tiny_f32", kind="lstm", dtype="f32", L=1, I=32, H=64, B=4, T=16, ragged=False, dx=True),
        # an ordinary float32 LSTM over sentences of differing lengths
        dict(name="lstm_f32", kind="lstm", dtype="f32", L=2, I=300, H=256, B=32, T=50, ragged=True, dx=True),
        # the data-dependent loop: one wide bf16 layer, lengths 1..200
        dict(name="lstm_varlen", kind="lstm", dtype="bf16", L=1, I=512, H=1024, B=128, T=200, ragged=True, dx=True),
        # the largest training call: two layers of 2048 units over data (no dx)
        dict(name="lstm_2048", kind="lstm", dtype="bf16", L=2, I=2048, H=2048, B=256, T=256, ragged=False, dx=False),
        # evaluation of a few sequences with sizes that are no multiple of a tile
        dict(name="lstm_eval_odd", kind="lstm_eval", dtype="bf16", L=2, I=250, H=500, B=33, T=64, ragged=True),
        # language-model training step, vocabulary 10000, batch 20, 35 steps
        dict(name="lm_650", kind="lm", dtype="bf16", L=2, H=650, B=20, T=35, V=10000),
        # sentiment trees, one batch of 25 sentences, for each tree model
        dict(name="treelstm", kind="treelstm", trees=25, leaves=50, E=300, H=150, V=20000),
        dict(name="treernn", kind="treernn", trees=25, leaves=50, E=300, H=300, V=20000),
        dict(name="childsum", kind="childsum", trees=25, leaves=50, E=300, H=150, V=20000),
        # a wider tree model over a larger batch of sentences
        dict(name="treelstm_wide", kind="treelstm", trees=100, leaves=50, E=300, H=300, V=20000),
        # the regression head over every step of a long batch
        dict(name="head_mse", kind="mse", dtype="bf16", rows=65536, H=2048, P=2048),
        # the update of a two-layer model's parameters (71 million)
        dict(name="sgd", kind="sgd", dtype="bf16", L=2, I=2048, H=2048, P=2048),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the ranges above."""
    kind = rng.choice(["lstm_f32", "lstm_bf16", "lstm_bf16", "lstm_eval", "lm", "treelstm", "treernn", "childsum",
                       "mse", "sgd"])
    if kind == "lstm_f32":
        return dict(kind="lstm", dtype="f32", L=rng.choice([1, 2]), I=_log(rng, 16, 512), H=_log(rng, 16, 512),
                    B=_log(rng, 1, 64), T=_log(rng, 8, 100), ragged=rng.random() < 0.5, dx=rng.random() < 0.5)
    if kind == "lstm_bf16":
        return dict(kind="lstm", dtype="bf16", L=rng.choice([1, 2]), I=_log(rng, 64, 2048), H=_log(rng, 64, 2048),
                    B=_log(rng, 8, 256), T=_log(rng, 16, 200), ragged=rng.random() < 0.5, dx=rng.random() < 0.5)
    if kind == "lstm_eval":
        return dict(kind="lstm_eval", dtype=rng.choice(["bf16", "bf16", "f32"]), L=rng.choice([1, 2]),
                    I=_log(rng, 32, 512), H=_log(rng, 32, 512), B=_log(rng, 1, 64), T=_log(rng, 8, 100),
                    ragged=rng.random() < 0.5)
    if kind == "lm":
        return dict(kind="lm", dtype="bf16", L=rng.choice([1, 2]), H=_log(rng, 128, 1024), B=_log(rng, 8, 128),
                    T=_log(rng, 10, 70), V=_log(rng, 1000, 20000))
    if kind == "treelstm":
        return dict(kind=kind, trees=_log(rng, 5, 128), leaves=_log(rng, 10, 60), E=_log(rng, 32, 320),
                    H=_log(rng, 24, 320), V=_log(rng, 2000, 20000))
    if kind == "treernn":
        h = _log(rng, 24, 400)
        return dict(kind=kind, trees=_log(rng, 5, 128), leaves=_log(rng, 10, 60), E=h, H=h, V=_log(rng, 2000, 20000))
    if kind == "childsum":
        return dict(kind=kind, trees=_log(rng, 5, 128), leaves=_log(rng, 10, 60), E=_log(rng, 32, 320),
                    H=_log(rng, 24, 320), V=_log(rng, 2000, 20000))
    if kind == "mse":
        return dict(kind="mse", dtype=rng.choice(["bf16", "bf16", "f32"]), rows=_log(rng, 256, 16384),
                    H=_log(rng, 64, 1024), P=_log(rng, 32, 1024))
    return dict(kind="sgd", dtype=rng.choice(["bf16", "f32"]), L=rng.choice([1, 2]), I=_log(rng, 32, 2048),
                H=_log(rng, 32, 1500), P=_log(rng, 32, 2048))


# ------------------------------------------------------------------ inputs
def _tdt(case):
    return torch.bfloat16 if case.get("dtype") == "bf16" else torch.float32


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _uniform(g, a, shape, dt):
    return (torch.rand(shape, generator=g, device=DEV) * (2 * a) - a).to(dt)


def _normal(g, s, shape, dt):
    return (torch.randn(shape, generator=g, device=DEV) * s).to(dt)


def _lengths(case, seed):
    """Host lengths U{1..T} (the longest always T), or None for all T."""
    if not case["ragged"]:
        return None
    n = np.random.default_rng(seed).integers(1, case["T"] + 1, size=case["B"]).astype(np.int32)
    n[int(n.argmax())] = case["T"]
    return n


def _lstm_inputs(case, seed):
    L, I, H, B, T = (case[k] for k in "LIHBT")
    dt, g = _tdt(case), _gen(seed)
    a = 1.0 / math.sqrt(H)
    n = dict(x=_normal(g, 1.0, (T, B, I), dt), lengths=_lengths(case, seed), Wx=[], Wh=[], b=[],
             h0=_normal(g, 0.3, (L, B, H), torch.float32), c0=_normal(g, 0.3, (L, B, H), torch.float32))
    for l in range(L):
        n["Wx"].append(_uniform(g, a, (4 * H, I if l == 0 else H), dt))
        n["Wh"].append(_uniform(g, a, (4 * H, H), dt))
        n["b"].append(_uniform(g, a, (4 * H,), dt))
    if case["kind"] == "lstm":
        n["dy"] = _normal(g, 1.0, (T, B, H), dt)
        n["dhT"] = _normal(g, 1.0, (L, B, H), torch.float32)
    return n


def _lm_workload(case, seed):
    return wl.ptb_lstm(T=case["T"], B=case["B"], H=case["H"], V=case["V"], L=case["L"], seed=seed)


def _tree_workload(case, seed):
    if case["kind"] == "treelstm":
        return wl.sst_treelstm(n_trees=case["trees"], E=case["E"], H=case["H"], V=case["V"],
                               max_leaves=case["leaves"], seed=seed)
    if case["kind"] == "treernn":
        return wl.sst_treernn(n_trees=case["trees"], H=case["H"], V=case["V"], max_leaves=case["leaves"], seed=seed)
    return wl.sst_childsum(n_trees=case["trees"], E=case["E"], H=case["H"], V=case["V"], max_nodes=case["leaves"],
                           seed=seed)


def _mse_inputs(case, seed):
    dt, g = _tdt(case), _gen(seed)
    R, H, P = case["rows"], case["H"], case["P"]
    a = 1.0 / math.sqrt(H)
    return dict(h=_normal(g, 0.3, (R, H), dt), W=_uniform(g, a, (P, H), dt), b=_uniform(g, a, (P,), dt),
                tgt=_normal(g, 1.0, (R, P), dt))


def _sgd_inputs(case, seed):
    g = _gen(seed)
    I, H, P = case["I"], case["H"], case["P"]
    shapes = []
    for l in range(case["L"]):
        shapes += [(4 * H, I if l == 0 else H), (4 * H, H), (4 * H,)]
    shapes += [(P, H), (P,)]
    return dict(p=[_uniform(g, 0.02, s, _tdt(case)) for s in shapes],
                g=[_normal(g, 1.0, s, torch.float32) for s in shapes])


SGD_LR, SGD_MAX_NORM = 0.1, 5.0


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("lstm", "lstm_eval"):
        L, I, H, B, T = (case[k] for k in "LIHBT")
        dt = _tdt(case)
        s = _lstm_inputs(case, seed)
        cdt = J.BF16 if case["dtype"] == "bf16" else J.F32
        s.update(kind=kind, desc=J.LstmDesc(L, I, H, B, T, cdt),
                 ws=torch.empty(J.janus_lstm_workspace_bytes(L, I, H, B, T, cdt), dtype=torch.uint8, device=DEV),
                 y=torch.empty(T, B, H, dtype=dt, device=DEV), hT=torch.empty(L, B, H, device=DEV),
                 cT=torch.empty(L, B, H, device=DEV))
        if kind == "lstm":
            s.update(dx=torch.empty(T, B, I, dtype=dt, device=DEV) if case["dx"] else None,
                     dh0=torch.empty(L, B, H, device=DEV), dc0=torch.empty(L, B, H, device=DEV))
            for k in ("Wx", "Wh", "b"):
                s["d" + k] = [torch.empty(t.shape, device=DEV) for t in s[k]]
        return s
    if kind == "lm":
        return dict(kind=kind, step=ts.make_step(_lm_workload(case, seed), DEV))
    if kind in ("treelstm", "treernn", "childsum"):
        return dict(kind=kind, step=ts.make_step(_tree_workload(case, seed), DEV))
    if kind == "mse":
        R, H, P = case["rows"], case["H"], case["P"]
        cdt = J.BF16 if case["dtype"] == "bf16" else J.F32
        s = _mse_inputs(case, seed)
        s.update(kind=kind, desc=J.MseDesc(R, H, P, cdt), dh=torch.empty_like(s["h"]),
                 dW=torch.empty(P, H, device=DEV), db=torch.empty(P, device=DEV), loss=torch.empty(1, device=DEV),
                 ws=torch.empty(J.janus_mse_workspace_bytes(R, H, P, cdt), dtype=torch.uint8, device=DEV))
        return s
    s = _sgd_inputs(case, seed)
    return dict(kind=kind, up=ts.SgdUpdate(s["p"], s["g"], SGD_LR, SGD_MAX_NORM), p=s["p"])


def run(s):
    kind = s["kind"]
    if kind in ("lstm", "lstm_eval"):
        J.janus_lstm_seq_fwd(s["desc"], s["x"], s["lengths"], s["Wx"], s["Wh"], s["b"], s["h0"], s["c0"], s["y"],
                             s["hT"], s["cT"], s["ws"])
        out = dict(y=s["y"], hT=s["hT"], cT=s["cT"])
        if kind == "lstm":
            J.janus_lstm_seq_bwd(s["desc"], s["x"], s["lengths"], s["Wx"], s["Wh"], s["ws"], s["dy"], s["dhT"], None,
                                 s["dx"], s["dh0"], s["dc0"], s["dWx"], s["dWh"], s["db"])
            out.update({k: s[k] for k in ("dx", "dh0", "dc0", "dWx", "dWh", "db")})
        return out
    if kind == "lm":
        st = s["step"]
        st.run()
        return dict(loss=st.loss, y=st.y, dWx=st.dWx, dWh=st.dWh, db=st.db, dWout=st.dWout, dbout=st.dbout, dE=st.dE)
    if kind in ("treelstm", "treernn", "childsum"):
        st = s["step"]
        st.run()
        out = dict(loss=st.loss, h_root=st.h_root, demb=st.demb, dW=st.dW, db=st.db, dWs=st.dWs, dbs=st.dbs)
        if kind != "treernn":
            out["dU"] = st.dU
        return out
    if kind == "mse":
        J.janus_linear_mse(s["desc"], s["h"], s["W"], s["b"], s["tgt"], s["dh"], s["dW"], s["db"], s["loss"], s["ws"])
        return dict(loss=s["loss"], dh=s["dh"], dW=s["dW"], db=s["db"])
    s["up"].apply()
    return dict(p=s["p"], stats=s["up"].stats)


# -------------------------------------------------------- work and tolerance
def work(case):
    """Products of the method (2 M N K each) and every input and output once."""
    kind = case["kind"]
    es = 2.0 if case.get("dtype") == "bf16" else 4.0
    if kind in ("lstm", "lstm_eval", "lm"):
        L, H, B, T = (case[k] for k in "LHBT")
        I = case.get("I", H)
        rows = B * ((T + 1) / 2.0 if case.get("ragged") else T)
        fl = by = 0.0
        for l in range(L):
            Il = I if l == 0 else H
            passes_x = 1 if kind == "lstm_eval" else 3 if (l > 0 or case.get("dx", True)) else 2
            passes_h = 1 if kind == "lstm_eval" else 3
            fl += 2.0 * rows * 4 * H * (passes_x * Il + passes_h * H)
            by += 4.0 * H * (Il + H + 1) * (es if kind == "lstm_eval" else es + 4.0)
        if kind == "lm":
            V = case["V"]
            fl += 3 * 2.0 * rows * V * H
            by += V * H * (es + 4.0) * 2
        elif kind == "lstm":
            by += rows * es * ((2 if case["dx"] else 1) * I + 2 * H)
        else:
            by += rows * es * (I + H)
        return dict(bytes=by, flops=fl)
    if kind in ("treelstm", "treernn", "childsum"):
        E, H, V = case["E"], case["H"], case["V"]
        n = case["trees"] * (5 + case["leaves"]) / 2.0    # leaves (nodes of a childsum batch)
        if kind == "treelstm":      # leaves take W (i, o, u blocks), internal nodes U
            fl = 3 * 2.0 * (n * 3 * H * E + n * 5 * H * 2 * H)
            w = 5.0 * H * (E + 2 * H + 1)
        elif kind == "treernn":
            fl = 3 * 2.0 * n * H * 2 * H
            w = H * (2.0 * H + 1)
        else:
            fl = 3 * 2.0 * n * 4 * H * (E + H)
            w = 4.0 * H * (E + H + 1)
        return dict(bytes=8.0 * w + 4.0 * V * E + 4.0 * n * E, flops=fl)
    if kind == "mse":
        R, H, P = case["rows"], case["H"], case["P"]
        return dict(bytes=es * (2.0 * R * H + R * P + P * H) + 4.0 * P * H, flops=3 * 2.0 * R * H * P)
    I, H, P = case["I"], case["H"], case["P"]
    n = sum(4.0 * H * ((I if l == 0 else H) + H + 1) for l in range(case["L"])) + P * (H + 1.0)
    return dict(bytes=n * (4.0 + 2 * es), flops=4.0 * n)


def tolerance(case):
    """About four times the largest 2-norm error against 64 bits seen over the
    ranges: bf16 paths 4.5e-3 (stored h, gates and gradients rounded to bf16),
    float32 paths 9e-7, bf16 parameters after the update 1.8e-3 (their own
    rounding)."""
    if case["kind"] == "sgd":
        return dict(rel=5e-3) if case["dtype"] == "bf16" else dict(rel=2e-7)
    if case.get("dtype") == "bf16":
        return dict(rel=2e-2)
    return dict(rel=5e-6)


# ------------------------------------------------------- the same in 64 bits
def _lstm64(x, lengths, Wx, Wh, b, h0, c0):
    """Masked LSTM stack in float64; returns y, hT, cT (graph kept)."""
    T, B, _ = x.shape
    L = len(Wx)
    H = Wh[0].shape[1]
    mask = None
    if lengths is not None:
        n = torch.from_numpy(lengths.astype(np.int64)).to(x.device)
        mask = (torch.arange(T, device=x.device)[:, None] < n[None, :])[..., None]
    inp, hs, cs = x, [], []
    for l in range(L):
        xg = inp @ Wx[l].T + b[l]
        h, c, ys = h0[l], c0[l], []
        for t in range(T):
            i, f, g, o = (xg[t] + h @ Wh[l].T).split(H, dim=1)
            cn = torch.sigmoid(f) * c + torch.sigmoid(i) * torch.tanh(g)
            hn = torch.sigmoid(o) * torch.tanh(cn)
            if mask is None:
                h, c = hn, cn
                ys.append(h)
            else:
                ys.append(torch.where(mask[t], hn, 0.0))
                h, c = torch.where(mask[t], hn, h), torch.where(mask[t], cn, c)
        inp = torch.stack(ys)
        hs.append(h)
        cs.append(c)
    return inp, torch.stack(hs), torch.stack(cs)


def _d(t, grad=False):
    t = (torch.from_numpy(np.ascontiguousarray(t)).to(DEV) if isinstance(t, np.ndarray) else t).double()
    return t.requires_grad_() if grad else t


def _binary_levels(t):
    """Per level: node ids (level 0 = leaves), children before parents."""
    lev = np.zeros(t.num_nodes, np.int64)
    for n in range(t.num_nodes):        # post-order: children come first
        if t.left[n] >= 0:
            lev[n] = 1 + max(lev[t.left[n]], lev[t.right[n]])
    return [np.flatnonzero(lev == k) for k in range(lev.max() + 1)]


def _nary_levels(t):
    lev = np.zeros(t.num_nodes, np.int64)
    for n in range(t.num_nodes - 1, -1, -1):   # numbered from the root: children come later
        ch = t.children[t.child_offsets[n]:t.child_offsets[n + 1]]
        if len(ch):
            lev[n] = 1 + lev[ch].max()
    return [np.flatnonzero(lev == k) for k in range(lev.max() + 1)]


def _tree64(case, seed):
    kind, w = case["kind"], _tree_workload(case, seed)
    t, H = w.trees, w.H
    names = ["emb", "W", "b", "Ws", "bs"] + ([] if kind == "treernn" else ["U"])
    P = {k: _d(getattr(w, k), True) for k in names}
    idx = lambda a: torch.from_numpy(np.asarray(a, np.int64)).to(DEV)  # noqa: E731
    levels = _nary_levels(t) if kind == "childsum" else _binary_levels(t)
    pos = np.empty(t.num_nodes, np.int64)
    pos[np.concatenate(levels)] = np.arange(t.num_nodes)
    hall = call = None
    for k, nodes in enumerate(levels):
        if kind == "treernn":
            if k == 0:
                h = P["emb"][idx(t.word[nodes])]
            else:
                ch = torch.cat([hall[idx(pos[t.left[nodes]])], hall[idx(pos[t.right[nodes]])]], 1)
                h = torch.tanh(ch @ P["W"].T + P["b"])
            c = h
        elif kind == "treelstm":
            if k == 0:
                a = P["emb"][idx(t.word[nodes])] @ P["W"].T + P["b"]
            else:
                l, r = idx(pos[t.left[nodes]]), idx(pos[t.right[nodes]])
                a = torch.cat([hall[l], hall[r]], 1) @ P["U"].T + P["b"]
            i, fl, fr, o, u = a.split(H, dim=1)
            c = torch.sigmoid(i) * torch.tanh(u)
            if k > 0:
                c = c + torch.sigmoid(fl) * call[l] + torch.sigmoid(fr) * call[r]
            h = torch.sigmoid(o) * torch.tanh(c)
        else:
            x = P["emb"][idx(t.word[nodes])] @ P["W"].T + P["b"]
            xi, xf = x[:, :3 * H], x[:, 3 * H:]
            if k > 0:
                cnt = t.child_offsets[nodes + 1] - t.child_offsets[nodes]
                kids = idx(pos[np.concatenate([t.children[t.child_offsets[n]:t.child_offsets[n + 1]] for n in nodes])])
                par = idx(np.repeat(np.arange(len(nodes)), cnt))
                hk, ck = hall[kids], call[kids]
                hsum = torch.zeros(len(nodes), H, dtype=torch.float64, device=DEV).index_add(0, par, hk)
                xi = xi + hsum @ P["U"][:3 * H].T
                f = torch.sigmoid(xf[par] + hk @ P["U"][3 * H:].T)
                csum = torch.zeros_like(hsum).index_add(0, par, f * ck)
            i, o, u = xi.split(H, dim=1)
            c = torch.sigmoid(i) * torch.tanh(u)
            if k > 0:
                c = c + csum
            h = torch.sigmoid(o) * torch.tanh(c)
        hall = h if hall is None else torch.cat([hall, h])
        call = c if call is None else torch.cat([call, c])
    h_root = hall[idx(pos[t.root])]
    loss = torch.nn.functional.cross_entropy(h_root @ P["Ws"].T + P["bs"], idx(w.labels))
    g = dict(zip(names, torch.autograd.grad(loss, [P[k] for k in names], allow_unused=True)))
    g = {k: torch.zeros_like(P[k]) if v is None else v for k, v in g.items()}
    out = dict(loss=loss.reshape(1), h_root=h_root, demb=g["emb"], dW=g["W"], db=g["b"], dWs=g["Ws"], dbs=g["bs"])
    if kind != "treernn":
        out["dU"] = g["U"]
    return out


def exact(case, seed):
    kind = case["kind"]
    if kind in ("lstm", "lstm_eval"):
        n = _lstm_inputs(case, seed)
        train = kind == "lstm"
        x = _d(n["x"], train and case["dx"])
        Wx, Wh, b = ([_d(t, train) for t in n[k]] for k in ("Wx", "Wh", "b"))
        h0, c0 = _d(n["h0"], train), _d(n["c0"], train)
        with torch.set_grad_enabled(train):
            y, hT, cT = _lstm64(x, n["lengths"], Wx, Wh, b, h0, c0)
        out = dict(y=y, hT=hT, cT=cT)
        if train:
            L = case["L"]
            obj = (y * _d(n["dy"])).sum() + (hT * _d(n["dhT"])).sum()
            g = torch.autograd.grad(obj, Wx + Wh + b + [h0, c0] + ([x] if case["dx"] else []))
            out.update(dWx=list(g[:L]), dWh=list(g[L:2 * L]), db=list(g[2 * L:3 * L]), dh0=g[3 * L], dc0=g[3 * L + 1],
                       dx=g[3 * L + 2] if case["dx"] else None)
        return out
    if kind == "lm":
        w = _lm_workload(case, seed)
        L, B, T, H = case["L"], case["B"], case["T"], case["H"]
        Wx, Wh, b = ([_d(a, True) for a in v] for v in (w.Wx, w.Wh, w.b))
        E, Wout, bout = _d(w.E, True), _d(w.Wout, True), _d(w.bout, True)
        ids = torch.from_numpy(w.input_ids.astype(np.int64)).to(DEV)
        tgt = torch.from_numpy(w.target_ids.astype(np.int64).reshape(-1)).to(DEV)
        z = torch.zeros(L, B, H, dtype=torch.float64, device=DEV)
        y, _, _ = _lstm64(E[ids], None, Wx, Wh, b, z, z)
        loss = torch.nn.functional.cross_entropy(y.reshape(T * B, H) @ Wout.T + bout, tgt)
        g = torch.autograd.grad(loss, Wx + Wh + b + [Wout, bout, E])
        return dict(loss=loss.reshape(1), y=y, dWx=list(g[:L]), dWh=list(g[L:2 * L]), db=list(g[2 * L:3 * L]),
                    dWout=g[3 * L], dbout=g[3 * L + 1], dE=g[3 * L + 2])
    if kind in ("treelstm", "treernn", "childsum"):
        return _tree64(case, seed)
    if kind == "mse":
        n = _mse_inputs(case, seed)
        h, W, b, tgt = (_d(n[k]) for k in ("h", "W", "b", "tgt"))
        d = h @ W.T + b - tgt
        dy = d * (2.0 / d.numel())
        return dict(loss=(d * d).mean().reshape(1), dh=dy @ W, dW=dy.T @ h, db=dy.sum(0))
    n = _sgd_inputs(case, seed)
    norm = math.sqrt(sum(float(g.double().square().sum()) for g in n["g"]))
    s = min(1.0, SGD_MAX_NORM / (norm + 1e-6))
    return dict(p=[p.double() - SGD_LR * s * g.double() for p, g in zip(n["p"], n["g"])],
                stats=torch.tensor([norm, s], dtype=torch.float64))
