"""Tree level programs whose groups of trees each live on one XCD, against the
float64 oracle: the widths at which the row tiles of a workgroup change, odd
sizes, one tree, more trees than groups, batches of several launches, and the
placement in which a group's workgroups share no L2 (JANUS_XCD_REMOTE=1)."""
import numpy as np
import pytest

from oracle import steps as oracle_steps
from paper_1812_01329_amd import workloads as wl
from tests.parity import TOL, check
from tests.test_gpu_parity import _run

pytestmark = pytest.mark.gpu


def _launches(recs, model):
    """Launches of the forward's and the backward's level program."""
    n = {r["label"]: r["launches"] for r in recs}
    assert f"{model}_bwd_tail" in n, n
    return n[f"{model}_fwd_persistent"], n[f"{model}_bwd_persistent"]


def _treelstm(w, parts=1):
    from paper_1812_01329_amd import janus as J
    J.janus_trace_begin()
    step, g = _run(w)
    assert _launches(J.janus_trace_end(), "treelstm") == (parts, parts)
    assert J.janus_treelstm_device_report(step.desc, w.trees, step.ws) == 0
    r = oracle_steps.tree_step(w)
    t = TOL["f32"]
    check("h_root", g["h_root"], r["h_root"], t["out"])
    for k in ("dh_root", "dWs", "dbs", "dW", "dU", "db", "demb"):
        check(k, g[k], r[k], t["grad"])
    return g


@pytest.mark.parametrize("H,E,n_trees", [(1, 1, 3), (3, 5, 1), (48, 37, 70), (96, 64, 9), (97, 33, 9), (192, 40, 20),
                                         (193, 16, 20), (256, 8, 5), (257, 300, 5), (288, 12, 9), (289, 512, 9),
                                         (384, 20, 6)])
def test_treelstm_widths(H, E, n_trees):
    print(f"[tree-xcd] H={H} E={E} trees={n_trees}", flush=True)
    _treelstm(wl.sst_treelstm(n_trees=n_trees, E=E, H=H, V=60, seed=H + E))


def test_treelstm_several_launches():
    """A group's cells keep dh and dc of every node in LDS, so a large batch
    runs in parts."""
    print("[tree-xcd] parts", flush=True)
    _treelstm(wl.sst_treelstm(n_trees=300, E=16, H=260, V=100, min_leaves=25, max_leaves=31, seed=14), parts=3)


@pytest.mark.parametrize("H", [29, 200])
def test_treelstm_without_shared_l2(H, monkeypatch):
    w = wl.sst_treelstm(n_trees=30, E=24, H=H, V=50, seed=5)
    g0 = _treelstm(w)
    monkeypatch.setenv("JANUS_XCD_REMOTE", "1")
    print(f"[tree-xcd-remote] H={H}", flush=True)
    g1 = _treelstm(w)
    for k in ("h_root", "dW", "dU", "db", "demb"):
        assert np.array_equal(g0[k], g1[k]), k


def _treernn(w, parts=1):
    from paper_1812_01329_amd import janus as J
    J.janus_trace_begin()
    step, g = _run(w)
    assert _launches(J.janus_trace_end(), "treernn") == (parts, parts)
    assert J.janus_treernn_device_report(step.desc, w.trees, step.ws) == 0
    r = oracle_steps.treernn_step(w)
    t = TOL["f32"]
    check("h_root", g["h_root"], r["h_root"], t["out"])
    for k in ("dh_root", "dWs", "dbs", "dW", "db", "demb"):
        check(k, g[k], r[k], t["grad"])
    return g


@pytest.mark.parametrize("H,n_trees", [(1, 3), (5, 1), (16, 70), (17, 9), (255, 9), (256, 20), (257, 20), (512, 6)])
def test_treernn_widths(H, n_trees):
    print(f"[rnn-xcd] H={H} trees={n_trees}", flush=True)
    _treernn(wl.sst_treernn(n_trees=n_trees, H=H, V=60, seed=H))


def test_treernn_several_launches():
    print("[rnn-xcd] parts", flush=True)
    _treernn(wl.sst_treernn(n_trees=500, H=300, V=100, min_leaves=35, max_leaves=41, seed=14), parts=3)


def test_treernn_without_shared_l2(monkeypatch):
    w = wl.sst_treernn(n_trees=30, H=100, V=50, seed=5)
    g0 = _treernn(w)
    monkeypatch.setenv("JANUS_XCD_REMOTE", "1")
    print("[rnn-xcd-remote]", flush=True)
    g1 = _treernn(w)
    for k in ("h_root", "dW", "db", "demb"):
        assert np.array_equal(g0[k], g1[k]), k


def _childsum(w, persistent=True, parts=1):
    from paper_1812_01329_amd import janus as J
    from paper_1812_01329_amd.train_step import make_step
    step = make_step(w)
    J.janus_trace_begin()
    step.run()
    g = step.results()
    recs = J.janus_trace_end()
    if persistent:
        assert _launches(recs, "childsum") == (parts, parts)
    else:
        assert not any(r["label"].endswith("_persistent") for r in recs), recs
    assert J.janus_childsum_device_report(step.desc, w.trees, step.ws) == 0
    r = oracle_steps.childsum_step(w)
    t = TOL["f32"]
    check("h_root", g["h_root"], r["h_root"], t["out"])
    for k in ("dh_root", "dWs", "dbs", "dW", "dU", "db", "demb"):
        check(k, g[k], r[k], t["grad"])
    return g


@pytest.mark.parametrize("H,E,n_trees", [(1, 1, 3), (3, 5, 1), (64, 37, 70), (128, 64, 9), (129, 33, 20), (256, 8, 5),
                                         (257, 300, 9), (319, 512, 6)])
def test_childsum_widths(H, E, n_trees):
    print(f"[childsum-xcd] H={H} E={E} trees={n_trees}", flush=True)
    _childsum(wl.sst_childsum(n_trees=n_trees, E=E, H=H, V=60, seed=H + E))


def test_childsum_several_launches():
    print("[childsum-xcd] parts", flush=True)
    _childsum(wl.sst_childsum(n_trees=300, E=16, H=300, V=100, min_nodes=35, max_nodes=45, seed=14), parts=5)


def test_childsum_past_the_groups_width_runs_levels():
    print("[childsum-xcd] H 320", flush=True)
    _childsum(wl.sst_childsum(n_trees=2, E=16, H=320, V=100, sizes=[90, 20], seed=15), persistent=False)


# One tree that the other XCDs would wait for, and trees of more nodes than a
# group's LDS holds, run in pieces: launches of the pieces, then of what is above.
@pytest.mark.parametrize("H,E,sizes,parts", [(29, 24, [300], 2), (150, 16, [700, 5, 1], 2), (150, 300, [2600], 2),
                                             (200, 40, [400, 300], 2), (300, 20, [500], 2), (384, 8, [900, 30], 2)])
def test_treelstm_pieces(H, E, sizes, parts):
    print(f"[tree-xcd-pieces] H={H} sizes={sizes}", flush=True)
    _treelstm(wl.sst_treelstm(n_trees=len(sizes), E=E, H=H, V=60, sizes=sizes, seed=H), parts=parts)


@pytest.mark.parametrize("H,sizes,parts", [(29, [400], 2), (150, [2600, 1], 2), (300, [700, 600], 2), (512, [900], 2)])
def test_treernn_pieces(H, sizes, parts):
    print(f"[rnn-xcd-pieces] H={H} sizes={sizes}", flush=True)
    _treernn(wl.sst_treernn(n_trees=len(sizes), H=H, V=60, sizes=sizes, seed=H), parts=parts)


@pytest.mark.parametrize("H,E,sizes,parts", [(29, 24, [500], 2), (128, 16, [900, 5], 2), (150, 300, [2400], 2),
                                             (260, 16, [900, 20], 2), (319, 8, [600, 300], 2)])
def test_childsum_pieces(H, E, sizes, parts):
    print(f"[childsum-xcd-pieces] H={H} sizes={sizes}", flush=True)
    _childsum(wl.sst_childsum(n_trees=len(sizes), E=E, H=H, V=60, sizes=sizes, seed=H), parts=parts)


@pytest.mark.parametrize("shape", ["chain", "star"])
def test_childsum_extreme_shapes_in_pieces(shape):
    """A chain longer than a group's LDS holds (371 nodes; pieces one above the
    other: 900 = 56 + 371 + 371 + 102), and a node of more children than that."""
    w = wl.sst_childsum(n_trees=1, E=16, H=300, V=60, sizes=[900], chain=shape == "chain", seed=8)
    if shape == "star":
        t = w.trees
        n = len(t.word)
        t.children[:] = [i for i in range(n) if i != t.root[0]]
        t.child_offsets[:] = [0 if i <= t.root[0] else n - 1 for i in range(n + 1)]
    print(f"[childsum-xcd-pieces] {shape}", flush=True)
    _childsum(w, parts=4 if shape == "chain" else 2)


@pytest.mark.parametrize("model", ["treelstm", "treernn", "childsum"])
def test_pieces_without_shared_l2(model, monkeypatch):
    make, run = {"treelstm": (lambda: wl.sst_treelstm(n_trees=2, E=24, H=120, V=50, sizes=[400, 40], seed=5), _treelstm),
                 "treernn": (lambda: wl.sst_treernn(n_trees=2, H=120, V=50, sizes=[400, 40], seed=5), _treernn),
                 "childsum": (lambda: wl.sst_childsum(n_trees=2, E=24, H=120, V=50, sizes=[800, 40], seed=5), _childsum),
                 }[model]
    g0 = run(make(), parts=2)
    monkeypatch.setenv("JANUS_XCD_REMOTE", "1")
    print(f"[tree-xcd-pieces-remote] {model}", flush=True)
    g1 = run(make(), parts=2)
    for k in ("h_root", "dW", "db", "demb"):
        assert np.array_equal(g0[k], g1[k]), k


@pytest.mark.parametrize("H", [29, 200])
def test_childsum_without_shared_l2(H, monkeypatch):
    w = wl.sst_childsum(n_trees=30, E=24, H=H, V=50, seed=5)
    g0 = _childsum(w)
    monkeypatch.setenv("JANUS_XCD_REMOTE", "1")
    print(f"[childsum-xcd-remote] H={H}", flush=True)
    g1 = _childsum(w)
    for k in ("h_root", "dW", "dU", "db", "demb"):
        assert np.array_equal(g0[k], g1[k]), k


@pytest.mark.parametrize("model", ["treelstm", "treernn", "childsum"])
def test_groups_without_trees(model):
    """Nine trees of which no two fit one group, eight groups a launch: two
    launches, seven groups of them without a tree."""
    print(f"[tree-xcd-empty] {model}", flush=True)
    if model == "treelstm":
        _treelstm(wl.sst_treelstm(n_trees=9, E=16, H=300, V=50, sizes=[300] * 9, seed=6), parts=2)
    elif model == "treernn":
        _treernn(wl.sst_treernn(n_trees=9, H=300, V=50, sizes=[600] * 9, seed=6), parts=2)
    else:
        _childsum(wl.sst_childsum(n_trees=9, E=16, H=300, V=50, sizes=[200] * 9, seed=6), parts=2)


@pytest.mark.parametrize("model", ["treelstm", "treernn", "childsum"])
def test_nan_word_vectors_do_not_stall(model):
    """A word vector holding a NaN of the bit pattern that marks a row not yet
    stored: its tree's root is NaN, the other trees keep their bits."""
    from paper_1812_01329_amd import janus as J
    make = {"treelstm": lambda: wl.sst_treelstm(n_trees=9, E=20, H=72, V=40, seed=3),
            "treernn": lambda: wl.sst_treernn(n_trees=9, H=72, V=40, seed=3),
            "childsum": lambda: wl.sst_childsum(n_trees=9, E=20, H=72, V=40, seed=3)}[model]
    report = {"treelstm": J.janus_treelstm_device_report, "treernn": J.janus_treernn_device_report,
              "childsum": J.janus_childsum_device_report}[model]
    w = make()
    word = w.trees.word
    word[word == 39] = 0
    n = int(w.trees.root[2])
    if model == "childsum":
        while w.trees.child_offsets[n] < w.trees.child_offsets[n + 1]:
            n = int(w.trees.children[w.trees.child_offsets[n]])
    else:
        while w.trees.left[n] >= 0:
            n = int(w.trees.left[n])
    word[n] = 39
    _, clean = _run(w)
    w.emb.view(np.uint32)[39, 5] = 0xffffffff
    print(f"[tree-xcd-nan] {model}", flush=True)
    step, g = _run(w)
    assert report(step.desc, w.trees, step.ws) == 0
    assert np.isnan(g["h_root"][2]).all()
    rest = [k for k in range(9) if k != 2]
    assert np.array_equal(g["h_root"][rest], clean["h_root"][rest])
