"""Projections of at most 64 rows whose column groups are split over workgroups of 16 columns: one, two and three 16-row tiles whole and
ragged, K that leaves wavefronts without a step or without a whole round, column groups that are no multiple of 8, gains in the
weights and in the rows (contexts that hold more sequences).  Against float64, the bound of tests/test_gpu_lds_tiles.py."""
import numpy as np
import pytest

import plan_choice
from test_gpu_lds_tiles import _forward64, _weights, case_arch

CASES = [
    # d, heads, kv heads, ff, window, sequences, sequences the context holds
    (128, 2, 1, 160, 1, 1, 1),        # 2 rows; 4 and 5 steps of k for 8 wavefronts
    (192, 3, 1, 352, 8, 1, 1),        # 16 rows, 6 column groups
    (320, 5, 5, 608, 9, 1, 1),        # 18: a row tile of two rows
    (1280, 20, 20, 3456, 16, 1, 1),   # 32
    (1280, 20, 4, 3456, 17, 1, 3),    # 34, gains in the rows
    (768, 12, 12, 2080, 24, 1, 1),    # 48: three tiles of 16 rows or two of 32
    (1024, 16, 16, 2816, 31, 1, 1),   # 62
    (2048, 16, 16, 5632, 32, 1, 1),   # 64, 128-wide heads
    (640, 10, 2, 1760, 5, 3, 7),      # 30 rows of three sequences, gains in the rows
]


@pytest.mark.gpu
@pytest.mark.parametrize("d,heads,kv,ff,window,seqs,room", CASES)
def test_against_float64(d, heads, kv, ff, window, seqs, room):
    import paper_2512_07503_amd as sjd
    arch, n = case_arch(d, heads, kv, ff, 901), 70
    w = _weights(arch, 23)
    rng = np.random.default_rng(8)
    prompts = [[rng.integers(0, arch["vocab"], m).astype(np.int32) for m in (5 + 3 * s, 1 + s)] for s in range(seqs)]
    g = sjd.Decoder(arch, w, "bf16", window, 100, max_seqs=room, top_k=200, seed=5, kernel_flags=sjd.KEEP_LOGITS)
    for again in range(3):   # the second and third time a replay of the first one's graph, over its buffers
        assert g.prefill([p[0] for p in prompts], [p[1] for p in prompts], [n] * seqs) == 0
        windows = [g.window(s)[0] for s in range(seqs)]
        g.step()
        out = g.logits().astype(np.float64)
        for s in range(seqs):
            for b in range(2):
                want = _forward64(arch, w, np.concatenate([prompts[s][b], windows[s][1:]]), window)
                err = np.linalg.norm(out[s, b] - want) / np.linalg.norm(want)
                print(d, window, "sequence", s, "branch", b, "relative error of the logits", err)
                assert err < 1.5e-2
    g.close()


def test_every_row_has_one_workgroup(tmp_path):
    """The rule, on the host: a workgroup per CU at most, all rows covered, 1, 2 or 4 tiles a workgroup, and the same projections with
    SJD_NO_ROW_SPLIT; CASES reach 1 and 2 tiles in every projection."""
    import subprocess
    (tmp_path / "main.cpp").write_text(r"""
#include <cstdio>
#include "plans.h"
int main() {
    for (int cus : {32, 64, 256, 304}) for (int groups = 1; groups <= 500; ++groups) for (int M = 1; M <= 200; ++M) {
        const ProjShape s{1280, 20, 20, 3456, 900, cus, 0}, u{1280, 20, 20, 3456, 900, cus, SJD_NO_ROW_SPLIT};
        const int rt = few_rows(s, M, groups), one = few_rows(u, M, groups);
        if ((rt != 0) != (one != 0) || (rt && (M > 64 || (rt != 1 && rt != 2) || few_wgs(M, groups, rt) > cus || 16 * one < M || (one != 1 && one != 2 && one != 4)))) {
            printf("cus %d groups %d M %d: %d %d\n", cus, groups, M, rt, one);
            return 1;
        }
    }
    int d, h, kv, f, M;
    while (scanf("%d %d %d %d %d", &d, &h, &kv, &f, &M) == 5) {
        const ProjShape s{d, h, kv, f, 900, 256, 0};
        printf("%d%d%d ", few_rows(s, M, s.qkv_groups()), few_rows(s, M, plan_div(d, 32)), few_rows(s, M, s.gate_up_groups()));
    }
}
""")
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", plan_choice.CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")], check=True)
    queries = "\n".join(f"{d} {h} {kv} {ff} {2 * window * seqs}" for d, h, kv, ff, window, seqs, _ in CASES)
    r = subprocess.run([str(tmp_path / "main")], input=queries, capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    got = r.stdout.split()
    assert all({"1", "2"} <= {g[i] for g in got} for i in range(3)), got
