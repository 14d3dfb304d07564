"""Row counts of a forward that are no multiple of any tile: windows and batches whose rows end inside a 64-row group (or
inside a 32-row tile) of the projection kernels, each step against the oracle.  Tolerance of the small stress models:
8e-2 of a row's largest |logit| (tests/test_gpu_e2e.py says where it comes from)."""
import pytest

import workload
from helpers import make_pair
from test_gpu_e2e import _lockstep

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,n_seqs,window", [
    ("small_fused64", 1, 33),    # 66 rows: one row tile of two rows past the first group
    ("small_fused64", 1, 37),    # 74 rows
    ("small_fused64", 3, 16),    # 96 rows: half a group, the branches of a sequence in one 32-row tile
    ("small_fused64", 5, 7),     # 70 rows, segments that straddle row tiles
    ("small_fused128", 2, 41),   # 164 rows, two query tiles of a segment in different groups
    ("small_fused128", 1, 150),  # 300 rows: from 256 rows on the tile kernels are eligible
    ("small_tile", 5, 27),       # 270 rows, ragged column tiles
])
def test_rows_that_fill_no_tile(oracle, name, n_seqs, window):
    cfg = workload.get_config(name)
    n_img = [70 - 9 * s for s in range(n_seqs)] if window < 100 else [190]
    for flags in ((0,) if window < 100 else (0, 16)):   # 16: tile kernels also for a narrow model
        o, g, cond, uncond, n = make_pair(oracle, cfg, window=window, n_image=n_img, n_seqs=n_seqs, kernel_flags=flags, head_alpha=6.0, std=0.08)
        worst, steps = _lockstep(o, g, n_seqs, 200, tol_rel=8e-2)
        assert [len(g.tokens(s)) for s in range(n_seqs)] == n
        print(name, n_seqs, window, flags, "steps", steps, "worst logits error abs/rel:", worst)
