"""The contractions behind the heads at the sizes where their plans change:
around one tile, few rows or columns, K shorter than one K block, and a K long
enough to be split over the chip.  Through the public heads, against the
float64 oracle."""
import numpy as np
import pytest

from oracle import steps as oracle_steps
from tests.parity import compare_lstm
from tests.test_gpu_heads import test_linear_mse as _linear_mse
from tests.test_gpu_heads import test_softmax_cross_entropy as _softmax
from tests.test_gpu_parity import _lstm, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,H,P", [(15, 64, 16), (16, 64, 16), (17, 63, 130), (63, 65, 16), (64, 8, 300),
                                      (127, 300, 33), (129, 72, 2100), (3000, 20, 40), (5000, 16, 16)])
def test_thin_bf16(rows, H, P):
    _linear_mse("bf16", rows, H, P)


@pytest.mark.parametrize("V,H,rows", [(15000, 300, 96), (3001, 40, 20), (1000, 130, 1)])
def test_thin_bf16_softmax(V, H, rows, monkeypatch):
    _softmax("bf16", V, H, rows, "1", "random", monkeypatch)


@pytest.mark.parametrize("rows,H,P", [(1, 1, 1), (3, 7, 2), (64, 64, 64), (65, 63, 66), (63, 129, 65), (7, 1000, 5),
                                      (2000, 33, 31), (700, 130, 257)])
def test_float32(rows, H, P):
    _linear_mse("f32", rows, H, P)


@pytest.mark.parametrize("V,H,rows", [(3001, 37, 20), (130, 1, 9)])
def test_float32_softmax(V, H, rows, monkeypatch):
    _softmax("f32", V, H, rows, "1", "random", monkeypatch)


@pytest.mark.parametrize("V,H,rows", [(300, 64, 130), (129, 128, 600), (1000, 192, 129), (260, 256, 257),
                                      (640, 320, 200), (127, 584, 700)])
def test_few_tiles_bf16(V, H, rows, monkeypatch):
    """128 x 128 tiles: partial tiles either way, one to more K blocks than
    there are LDS stages."""
    _softmax("bf16", V, H, rows, "1", "random", monkeypatch)


@pytest.mark.parametrize("I,H,B,T,rows", [(240, 80, 54, 40, 2034), (120, 120, 63, 72, 4334)])
def test_ragged_batches_keep_the_split_contractions(I, H, B, T, rows):
    """Fewer running rows than T B can take more K splits than T B would: the
    workspace has room for them, so no weight gradient walks its K serially."""
    from paper_1812_01329_amd import janus as J
    n = np.full(B, T, np.int64)
    for i in range(B * T - rows):
        n[i % B] -= 1
    w = _lstm("mse", "bf16", L=1, I=I, H=H, B=B, T=T, lengths=[int(v) for v in n], seed=I, P=128)
    print(f"[ragged-splits] I={I} H={H} B={B} T={T} rows={rows}", flush=True)
    J.janus_trace_begin()
    _, g = _run(w)
    labels = {r["label"] for r in J.janus_trace_end()}
    assert "gemm_nt_splitk" in labels and not any(k.startswith(("gemm_tn", "gemm_nn")) for k in labels), labels
    compare_lstm(g, oracle_steps.lstm_step(w), "bf16")
