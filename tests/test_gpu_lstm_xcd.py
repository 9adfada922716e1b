"""The recurrence in row groups that each live on one XCD, against the
float64 oracle.

Sizes sit at the edges of its plan: one unit block, the last and first H of
each weight size (256 | 257, 512 | 513, 768, 1024), an H that is no multiple
of 4 (float32), one row, one row tile and a row more, two row tiles per group,
more rows than one launch takes.  JANUS_XCD_REMOTE=1 takes the placement in
which a group's workgroups share no L2."""
import numpy as np
import pytest

from oracle import steps as oracle_steps
from paper_1812_01329_amd import workloads as wl
from tests.parity import compare_lstm
from tests.test_gpu_parity import _lstm, _run

pytestmark = pytest.mark.gpu


def _ragged(B, T, seed):
    n = np.random.default_rng(seed).integers(0, T + 1, B)
    n[0] = T
    if B > 1:
        n[-1] = 0
    return [int(v) for v in n]


def _report(step):
    from paper_1812_01329_amd import janus as J
    return J.janus_lstm_device_report(step.desc, step.ws)


@pytest.mark.parametrize("ragged", [False, True])
@pytest.mark.parametrize("dtype,H,B", [
    ("f32", 8, 1030), ("f32", 130, 1), ("f32", 256, 16), ("f32", 257, 17), ("f32", 509, 33), ("f32", 512, 150),
    ("bf16", 16, 5), ("bf16", 64, 256), ("bf16", 256, 17), ("bf16", 272, 300), ("bf16", 512, 129), ("bf16", 520, 16),
    ("bf16", 768, 40), ("bf16", 784, 130), ("bf16", 1024, 33)])
def test_row_groups(dtype, H, B, ragged):
    T = 9
    w = _lstm("mse", dtype, L=2, I=24, H=H, B=B, T=T, lengths=_ragged(B, T, H + B) if ragged else None, seed=H, h0=True,
              P=16, scale=1.0 / np.sqrt(H))
    print(f"[xcd] {dtype} H={H} B={B} ragged={ragged}", flush=True)
    step, g = _run(w)
    rep = _report(step)
    print(f"[xcd] report {rep}", flush=True)
    assert rep["timed_out"] == 0 and rep["bwd_groups"] > 0
    compare_lstm(g, oracle_steps.lstm_step(w), dtype)


@pytest.mark.parametrize("dtype,H,B", [("f32", 157, 50), ("bf16", 704, 100)])
def test_row_groups_without_shared_l2(dtype, H, B, monkeypatch):
    """The same bits as with each group on one XCD, and none counted as local."""
    T = 12
    w = _lstm("mse", dtype, L=1, I=24, H=H, B=B, T=T, lengths=_ragged(B, T, 3), seed=4, h0=True, P=16,
              scale=1.0 / np.sqrt(H))
    _, g0 = _run(w)
    monkeypatch.setenv("JANUS_XCD_REMOTE", "1")
    print(f"[xcd-remote] {dtype} H={H} B={B}", flush=True)
    step, g1 = _run(w)
    rep = _report(step)
    assert rep["timed_out"] == 0 and rep["bwd_groups"] > 0 and rep["bwd_local_groups"] == 0
    for k in ("y", "hT", "cT", "dh0", "dc0"):
        assert np.array_equal(g0[k], g1[k]), k
    for k in ("dWx", "dWh", "db"):
        assert np.array_equal(g0[k][0], g1[k][0]), k


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_nan_rows_do_not_stall(dtype):
    """A NaN in the state, of the bit pattern that marks an operand not yet
    stored too, travels through its own row and leaves the others alone."""
    T, B, H = 6, 20, 144
    w = _lstm("mse", dtype, L=1, I=24, H=H, B=B, T=T, seed=9, h0=True, P=16)
    _, clean = _run(w)
    w.h0 = w.h0.copy()
    w.h0.view(np.uint32)[0, 3, 5] = 0xffffffff
    print(f"[xcd-nan] {dtype}", flush=True)
    step, g = _run(w)
    assert _report(step)["timed_out"] == 0
    assert np.isnan(g["hT"][0, 3]).all()
    rest = [b for b in range(B) if b != 3]
    assert np.array_equal(g["y"][:, rest], clean["y"][:, rest])


@pytest.mark.parametrize("H,B,groups", [(16, 16, False), (64, 1, False), (65, 1, True), (16, 17, True), (1, 2048, False),
                                        (3, 700, True), (64, 40, True)])
@pytest.mark.parametrize("ragged", [False, True])
def test_small_float32_on_both_sides_of_the_rule(H, B, groups, ragged):
    """float32 problems of up to 4096 products per step run in one workgroup,
    larger ones that would fit one too in row groups."""
    from paper_1812_01329_amd import janus as J
    w = _lstm("mse", "f32", L=2, I=24, H=H, B=B, T=7, lengths=_ragged(B, 7, H + B) if ragged else None, seed=H, h0=True,
              P=16)
    print(f"[xcd-small] H={H} B={B} ragged={ragged}", flush=True)
    J.janus_trace_begin()
    step, g = _run(w)
    labels = {r["label"] for r in J.janus_trace_end()}
    assert ("lstm_fwd_small" in labels, "lstm_bwd_small" in labels) == (not groups, not groups), labels
    rep = _report(step)
    assert rep["timed_out"] == 0 and (rep["bwd_groups"] > 0) == groups
    compare_lstm(g, oracle_steps.lstm_step(w), "f32")


def test_two_threads_on_two_streams():
    """Kernels whose workgroups wait for each other take turns across
    streams: two host threads, each on its own stream, give the bits of the
    same steps run one after another."""
    import threading

    import torch
    from paper_1812_01329_amd.train_step import make_step
    ws = [_lstm("mse", "f32", L=1, I=24, H=400, B=40, T=12, seed=21, P=16),
          _lstm("mse", "bf16", L=2, I=24, H=1024, B=64, T=12, seed=22, P=16),
          wl.sst_treelstm(n_trees=9, E=64, H=96, V=200, seed=23)]
    steps = [make_step(w) for w in ws]
    keys = ["y", "y", "h_root"]
    for s in steps:
        s.run()
    want = [s.results()[k] for s, k in zip(steps, keys)]
    torch.cuda.synchronize()
    print("[xcd-threads]", flush=True)

    def work(step):
        st = torch.cuda.Stream()
        with torch.cuda.stream(st):
            for _ in range(20):
                step.run()
        st.synchronize()

    th = [threading.Thread(target=work, args=(s,)) for s in steps]
    for t in th:
        t.start()
    for t in th:
        t.join()
    for s, k, a in zip(steps, keys, want):
        assert np.array_equal(s.results()[k], a), k
    for s in steps[:2]:
        assert _report(s)["timed_out"] == 0
