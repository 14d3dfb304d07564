"""LDS-tile launches that carry workgroups which only touch the next launch's weights: output projection behind QKV, down behind
gate/up, and the next QKV and gate/up behind either; tests/test_plan_choice.py holds the cases to such launches, all four of them.
Against float64, the bound of test_gpu_lds_tiles.py."""
import pytest

from test_gpu_lds_tiles import test_against_float64 as _against_float64

pytestmark = pytest.mark.gpu

CASES = [
    (1280, 20, 20, 3456, 3001, 16, [(70, 68)]),                       # rows of a step / prompts: 32 / 136: QKV and gate/up touch
    (768, 12, 12, 2048, 3001, 24, [(400, 380), (199, 183)]),          # 96 / 1158: gate/up and down
    (2048, 16, 16, 5632, 3001, 33, [(370, 368)]),                     # 66 / 736: output
    (640, 10, 10, 2240, 3001, 4, [(112, 112)]),                       # 8 / 222: gate/up
]


@pytest.mark.parametrize("d,heads,kv,ff,ids,window,lens", CASES)
def test_touching_launches(d, heads, kv, ff, ids, window, lens):
    _against_float64(d, heads, kv, ff, ids, window, lens)
