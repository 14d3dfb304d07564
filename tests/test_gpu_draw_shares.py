"""Draws from rows whose kept pairs give a thread one pair, up to four, up to eight and more (256 threads): decisions, windows and tokens
bit-exact against the oracle on the same logits, residual draws after rejections among them."""
import pytest

from test_gpu_decide import _drive

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("K", [1, 255, 256, 257, 1024, 1025, 2048, 2049])
def test_draws_of_every_share(oracle, K):
    st = _drive(oracle, "cfg0", 12, 8, 40, 2, K, 0.5, 31, 2.0, 0.3)
    assert st["rej"] > 0
