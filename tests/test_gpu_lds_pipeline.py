"""LDS-tile projections of few pipeline stages of 32 k: fewer than, as many as and a few more than the six that are in flight, odd and
even (the operands of consecutive stages alternate between two sets of registers).  Against float64, the bound of
test_gpu_lds_tiles.py."""
import pytest

import plan_choice
from test_gpu_lds_tiles import case_arch, test_against_float64 as _against_float64

# d, heads, kv heads, ff: stages of QKV and gate/up = d / 32, of the down projection = ff / 32; 1500 prompt rows
CASES = [(64, 1, 1, 96), (320, 5, 1, 96), (320, 5, 1, 160), (192, 3, 1, 352), (320, 5, 1, 224), (320, 5, 1, 352), (384, 6, 1, 1056)]
LENS = [(751, 751)]


@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,kv,ff", CASES)
def test_few_stages(d, heads, kv, ff):
    _against_float64(d, heads, kv, ff, 301, 1, LENS)


def test_the_cases_reach_these_stages():
    seen = set()
    for (d, h, kv, ff), p in zip(CASES, plan_choice.choose([(case_arch(*c, 301), 1500, 0, 0) for c in CASES])):
        for name, K in (("qkv", d), ("gate_up", d), ("down", ff)):
            shape, ks = p[name]
            if shape >= 0 and ks == 1:
                seen.add(K // 32)
    assert {2, 3, 5, 6, 7, 10, 11, 12, 33} <= seen, seen


# The 256 x 128 tiles of eight wavefronts, ragged in rows and columns: QKV (a last column tile of two blocks), output and down
# projections of prompts and the QKV of a step; norm gains in the weights and (window 33) in the rows
WIDE_CASES = [
    (4096, 32, 32, 8192, 1, [(1022, 1019)], {"out", "down"}),     # 2039 prompt rows
    (5120, 40, 8, 13824, 33, [(640, 642)], {"out", "down"}),      # 1280
    (4096, 32, 32, 1024, 32, [(8, 7)] * 8, {"qkv"}),              # 512 rows of a step
    (3264, 51, 17, 2560, 1, [(570, 567)], {"qkv"}),               # 1135 prompt rows, 170 column blocks
]


@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,kv,ff,window,lens,reached", WIDE_CASES)
def test_wide_tiles(d, heads, kv, ff, window, lens, reached):
    _against_float64(d, heads, kv, ff, 301, window, lens)


def test_the_wide_cases_reach_the_wide_tiles():
    for d, h, kv, ff, window, lens, reached in WIDE_CASES:
        rows = len(lens) * 2 * window if window == 32 else sum(c + u - 2 for c, u in lens)
        p = plan_choice.choose([(case_arch(d, h, kv, ff, 301), rows, 0, 0)])[0]
        assert {n for n in ("qkv", "out", "down") if p[n] == (6, 1)} == reached, (d, rows, p)
