"""LDS-tile launches that carry workgroups which only touch the next launch's weights: output projection behind QKV, down behind
gate/up, and the next QKV and gate/up behind either.  Against float64, the bound of test_gpu_lds_tiles.py."""
import pytest

from test_gpu_lds_tiles import test_against_float64 as _against_float64

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,heads,kv,ff,ids,window,lens", [
    (1280, 20, 20, 3456, 3001, 16, [(120, 96), (40, 41), (77, 130), (99, 100), (140, 111), (2, 1)]),   # rows of a step / prompts: 192 / 945
    (1280, 20, 20, 3456, 3001, 33, [(98, 96), (120, 99), (2, 1)]),    # 198 / 410
    (640, 10, 10, 2240, 3001, 4, [(112, 112)]),                       # 8 / 222
])
def test_touching_launches(d, heads, kv, ff, ids, window, lens):
    _against_float64(d, heads, kv, ff, ids, window, lens)
