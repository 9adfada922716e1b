"""The contractions behind the heads at the sizes where their plans change:
around one tile, few rows or columns, K shorter than one K block, and a K long
enough to be split over the chip.  Through the public heads, against the
float64 oracle."""
import pytest

from tests.test_gpu_heads import test_linear_mse as _linear_mse
from tests.test_gpu_heads import test_softmax_cross_entropy as _softmax

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
