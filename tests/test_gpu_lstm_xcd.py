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
from tests.parity import TOL, compare_lstm
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
    assert rep["bwd_local_groups"] > 0   # groups that exchanged through their XCD's L2
    compare_lstm(g, oracle_steps.lstm_step(w), dtype)


@pytest.mark.parametrize("H,B,groups", [(512, 513, 2 * 8 + 1), (256, 520, 2 * 8 + 1), (1024, 255, 8), (1024, 256, 0)])
def test_backward_rule_looks_at_the_rows_of_a_launch(H, B, groups):
    """Row groups in the backward, unless the 256 rows that a launch takes have
    2 MB of dG a step (H 1024); the sliced kernels report other groups."""
    w = _lstm("mse", "bf16", L=1, I=24, H=H, B=B, T=3, seed=H, P=16, scale=1.0 / np.sqrt(H))
    print(f"[xcd-rule] H={H} B={B}", flush=True)
    step, g = _run(w)
    rep = _report(step)
    assert rep["timed_out"] == 0 and (rep["bwd_groups"] == groups) == (groups > 0), rep
    compare_lstm(g, oracle_steps.lstm_step(w), "bf16")


@pytest.mark.parametrize("dtype,H,B", [("f32", 157, 50), ("bf16", 704, 100)])
def test_row_groups_without_shared_l2(dtype, H, B, monkeypatch):
    """The same bits as with each group on one XCD, and none counted as local."""
    T = 12
    w = _lstm("mse", dtype, L=1, I=24, H=H, B=B, T=T, lengths=_ragged(B, T, 3), seed=4, h0=True, P=16,
              scale=1.0 / np.sqrt(H))
    step, g0 = _run(w)
    assert _report(step)["bwd_local_groups"] > 0
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


@pytest.mark.parametrize("dtype,B", [("f32", (1 << 19) + 17), ("bf16", (1 << 20) + 17)])
def test_step_of_more_than_4_gib_of_gate_rows(dtype, B):
    """One step of a batch whose gate rows (B x 4H) pass 4 GiB, every row
    against the same step in float64."""
    import torch

    from paper_1812_01329_amd import janus as J
    H, I = 512, 8
    dt, cdt = (torch.float32, J.F32) if dtype == "f32" else (torch.bfloat16, J.BF16)
    g = torch.Generator(device="cuda").manual_seed(7)
    rnd = lambda *s, k=1.0: (torch.randn(*s, generator=g, device="cuda") * k).to(dt)
    x, dy = rnd(1, B, I), rnd(1, B, H)
    Wx, Wh, b = rnd(4 * H, I, k=0.3), rnd(4 * H, H, k=0.04), rnd(4 * H, k=0.1)
    h0 = rnd(1, B, H, k=0.5).float()
    y, dx = torch.zeros_like(dy), torch.zeros_like(x)
    dh0 = torch.zeros_like(h0)
    dWx, dWh, db = (torch.zeros(t.shape, device="cuda") for t in (Wx, Wh, b))
    d = J.LstmDesc(1, I, H, B, 1, cdt)
    ws = torch.empty(J.janus_lstm_workspace_bytes(1, I, H, B, 1, cdt), dtype=torch.uint8, device="cuda")
    print(f"[xcd-4gib] {dtype} B={B} ws={ws.numel() >> 20} MiB", flush=True)
    J.janus_lstm_seq_fwd(d, x, None, [Wx], [Wh], [b], h0, None, y, None, None, ws)
    J.janus_lstm_seq_bwd(d, x, None, [Wx], [Wh], ws, dy, None, None, dx, dh0, None, [dWx], [dWh], [db])
    assert J.janus_lstm_device_report(d, ws)["timed_out"] == 0
    t = TOL[dtype]

    def near(name, a, ref, tol):
        e = float((a.double() - ref).abs().max() / ref.abs().max())
        assert e <= tol, f"{name}: relative error {e:.3e} > {tol:.1e}"

    X, H0, U, V = x.double()[0], h0[0], Wx.double(), Wh.double()
    sWx, sWh, sb = torch.zeros_like(U), torch.zeros_like(V), torch.zeros(4 * H, dtype=torch.float64, device="cuda")
    for r in range(0, B, 1 << 16):
        q = slice(r, min(r + (1 << 16), B))
        hp = H0[q].double()
        i, f, gg, o = (X[q] @ U.T + hp @ V.T + b.double()).chunk(4, 1)
        i, gg, o = i.sigmoid(), gg.tanh(), o.sigmoid()
        c = i * gg
        tau = c.tanh()
        near(f"y[{r}]", y[0, q], o * tau, t["out"])
        dh = dy[0, q].double()
        dc = dh * o * (1 - tau * tau)
        da = torch.cat([dc * gg * i * (1 - i), torch.zeros_like(dc), dc * i * (1 - gg * gg), dh * tau * o * (1 - o)], 1)
        near(f"dx[{r}]", dx[0, q], da @ U, t["grad"])
        near(f"dh0[{r}]", dh0[0, q], da @ V, t["grad"])
        sWx += da.T @ X[q]
        sWh += da.T @ hp
        sb += da.sum(0)
    for k, a, ref in (("dWx", dWx, sWx), ("dWh", dWh, sWh), ("db", db, sb)):
        near(k, a, ref, t["grad"])


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


def test_many_streams_come_and_go():
    """Streams that are destroyed right after a step, and more of them than
    the library keeps in mind: small steps that fit the chip together, and
    some that need it whole, all with the bits of the first run."""
    import ctypes

    import torch
    from paper_1812_01329_amd.train_step import make_step
    hip = ctypes.CDLL("libamdhip64.so")
    ws = [_lstm("mse", "f32", L=1, I=24, H=72, B=9, T=5, seed=31, P=16),
          _lstm("mse", "bf16", L=1, I=24, H=1024, B=128, T=5, seed=32, P=16),
          wl.sst_treernn(n_trees=20, H=64, V=50, seed=33)]
    steps = [make_step(w) for w in ws]
    keys = ["y", "y", "h_root"]
    for s in steps:
        s.run()
    want = [s.results()[k] for s, k in zip(steps, keys)]
    print("[xcd-streams]", flush=True)
    last = [None] * len(steps)   # a step's runs follow each other
    for i in range(60):
        j = 0 if i % 4 else 1 + i // 4 % 2
        h = ctypes.c_void_p()
        assert hip.hipStreamCreateWithFlags(ctypes.byref(h), 1) == 0
        st = torch.cuda.ExternalStream(h.value)
        if last[j] is not None:
            st.wait_event(last[j])
        with torch.cuda.stream(st):
            steps[j].run()
        last[j] = torch.cuda.Event()
        last[j].record(st)
        assert hip.hipStreamDestroy(h) == 0
    torch.cuda.synchronize()
    for s, k, a in zip(steps, keys, want):
        assert np.array_equal(s.results()[k], a), k
    for s in steps[:2]:
        assert _report(s)["timed_out"] == 0
