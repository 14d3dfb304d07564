"""The choice of projection kernels (csrc/plans.h), compiled for the host, over widths, MLPs, row counts and kernel flags: the K
splits stay within what a context's workspace is sized for, no split is empty, every projection has a kernel and is expected to take that kernel's time."""
import subprocess

import pytest

import plan_choice

_MAIN = r"""
#include <cstdio>
#include <cstdlib>
#include <math.h>
#include "plans.h"
// the expected time of the kernels that the plan names (whether the weights are touched ahead: row groups, 0.82)
static bool own_time(const ProjShape &s, int M, PlanEpi epi, int blocks, int KB, const ProjPlan &p) {
    const int nbw = epi == PLAN_RESID ? resid_nbw(s.d_model) : 2, groups = plan_div(blocks, nbw);
    const int mt = p.ks > 1 ? (M <= 32 ? 1 : 2) : skinny_mt(s, M, groups);
    const PlanEpi e = p.ks > 1 ? PLAN_PARTIAL : epi;
    const double reduce = p.ks > 1 ? reduce_us(M, s.d_model, p.ks) : 0.0;
    const double us = (p.tile ? tile_us(e, M, blocks, KB, p.ks, s.n_cus) : p.lds >= 0 ? lds_us(p.lds, e, M, blocks, KB, p.ks, s.n_cus)
                                                                                   : skinny_us(e, M, mt, groups, nbw, KB, p.ks, s.n_cus)) + reduce;
    return fabs(p.us - us) < 1e-9 * us || (!p.tile && p.lds < 0 && epi != PLAN_RESID && fabs(p.us - 0.82 * us) < 1e-9 * us);
}
int main(int, char **v) {
    const int d = atoi(v[1]), hd = d % 128 ? 64 : 128, flags[] = {0, SJD_KERNELS_ROWGROUPS, SJD_KERNELS_TILES, SJD_NO_ROW_SPLIT, SJD_NO_L2_WARM};
    for (int ff : {d / 32 * 32 + 32, 2 * d + 96, 7 * d / 2 / 32 * 32}) for (int kv : {1, 4}) for (int fl : flags) for (int cus : {256, 304, 64}) for (int M = 1; M <= 2200; M += cus == 256 ? 1 : 9) {
        if (d / hd % kv) continue;
        const ProjShape s{d, d / hd, d / hd / kv, ff, 16384, cus, fl};
        const ForwardPlan f = forward_plan(s, M, M % 64 == 0);
        if (!own_time(s, M, PLAN_QKV, s.qkv_groups() * 2, d / 16, f.qkv) || !own_time(s, M, PLAN_RESID, plan_div(d, 32), d / 16, f.o) ||
            !own_time(s, M, PLAN_SWIGLU, s.gate_up_groups() * 2, d / 16, f.gate_up) || !own_time(s, M, PLAN_RESID, plan_div(d, 32), ff / 16, f.down)) {
            printf("expected time: d %d ff %d kv %d M %d flags %d\n", d, ff, d / hd / kv, M, fl);
            return 1;
        }
        for (const ProjPlan *p : {&f.qkv, &f.o, &f.gate_up, &f.down}) {
            const int K = p == &f.down ? ff : d, KB = K / 16, unit = p->lds >= 0 ? 2 : 1, per = plan_div(KB, unit * p->ks) * unit;
            if (p->ks < 1 || (p->ks - 1) * per >= KB) { printf("empty split: d %d ff %d M %d flags %d\n", d, ff, M, fl); return 1; }
            if ((p == &f.o || p == &f.down) ? p->ks > max_splits(s, M, K) : p->ks != 1) { printf("splits: d %d ff %d M %d flags %d\n", d, ff, M, fl); return 1; }
            if (!(p->us > 0 && p->us < 1e8) || (p->tile && p->lds >= 0) || (p->tile && M < TILE_M) || (p->lds >= 0 && M <= 64)) { printf("kernel: d %d ff %d M %d flags %d\n", d, ff, M, fl); return 1; }
        }
    }
}
"""


@pytest.fixture(scope="module")
def program(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "main.cpp").write_text(_MAIN)
    subprocess.run(["g++", "-std=c++17", "-O2", "-I", plan_choice.CSRC, str(d / "main.cpp"), "-o", str(d / "main")], check=True)
    return d / "main"


@pytest.mark.parametrize("d", [64, 128, 512, 640, 768, 1280, 2048, 3072, 4096, 5120])
def test_every_choice_fits(program, d):
    r = subprocess.run([str(program), str(d)], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout


def test_which_fp32_projections_have_their_norm_inside(tmp_path):
    """(QKV, gate/up, head) of a step and (QKV, gate/up) of the prompt: few results inside, many apart, and the GPU cases on both sides."""
    import test_gpu_f32_fused as t
    (tmp_path / "main.cpp").write_text("""#include <cstdio>
#include "plans.h"
int main() { int M, n, f, v; while (scanf("%d %d %d %d", &M, &n, &f, &v) == 4)
    printf("%d%d%d\\n", f32_inside(M, n, F32_QKV_INSIDE), f32_inside(M, 2 * f, F32_GATE_UP_INSIDE), f32_inside(M, v, F32_HEAD_INSIDE)); }
""")
    subprocess.run(["g++", "-std=c++17", "-I", plan_choice.CSRC, str(tmp_path / "main.cpp"), "-o", str(tmp_path / "main")], check=True)

    def sides(*queries):
        return subprocess.run([str(tmp_path / "main")], input="\n".join("%d %d %d %d" % q for q in queries), capture_output=True, text=True, check=True).stdout.split()
    # 62 prompt and 32 step rows of 256; 512 prompt rows of 512 and 2048
    assert sides((62, 768, 1024, 1), (32, 768, 1024, 4096), (512, 1536, 1440, 1), (512, 6144, 5632, 1)) == ["111", "111", "001", "001"]
    seen = []
    for a, window, seqs, prompt in t.CASES[-3:]:
        n = (a["n_heads"] + 2 * a["n_kv_heads"]) * a["d_model"] // a["n_heads"]
        step, rows = sides((2 * seqs * window, n, a["d_ff"], a["vocab"]), (min(512, 2 * seqs * (prompt - 1)), n, a["d_ff"], 1))
        seen.append((step, rows[:2]))
    assert seen == [("100", "10"), ("111", "01"), ("000", "11")], seen
