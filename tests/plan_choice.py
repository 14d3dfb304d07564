"""The library's choice of projection kernels (csrc/plans.h, plain C++), compiled for the host: which kernels a test case
reaches, without a GPU."""
import os
import subprocess
import tempfile

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2512_07503_amd", "csrc")
_MAIN = r"""
#include <cstdio>
#include "plans.h"
int main() {
    ProjShape s; int M, win32;
    while (scanf("%d %d %d %d %d %d %d %d", &s.d_model, &s.n_heads, &s.n_kv_heads, &s.d_ff, &s.n_sampled, &s.kernel_flags, &M, &win32) == 8) {
        s.n_cus = 256;
        const ForwardPlan f = forward_plan(s, M, win32 != 0);
        const int nbw = resid_nbw(s.d_model), nd = plan_div(plan_div(s.d_model, 32), nbw) * nbw, tiles_d = plan_div(s.d_model, 64) * 2;
        const int nq = s.qkv_groups() * 2, ng = s.gate_up_groups() * 2, nh = s.head_groups() * 2, KB = s.d_model / 16, KF = s.d_ff / 16;
        const ProjPlan *p[5] = {&f.qkv, &f.o, &f.gate_up, &f.down, &f.head};
        const int blocks[5] = {nq, tiles_d, ng, tiles_d, nh};
        // workgroups that touch the weights of the projection behind: of launches through LDS tiles
        auto touches = [&](const ProjPlan &w, int n_blocks, const ProjPlan &next, int next_blocks, int next_KB, int next_nbw) {
            if (f.tile || w.lds < 0 || w.ks > 1) return 0;
            return touch(s, M, lds_wgs(w.lds, M, n_blocks), w.us, slabs_of(next, next_blocks, next_KB, next_nbw)).wgs;
        };
        const int touched[5] = {touches(f.qkv, nq, f.o, nd, KB, nbw), touches(f.o, plan_div(s.d_model, 32), f.gate_up, ng, KB, 2),
                                touches(f.gate_up, ng, f.down, nd, KF, nbw), touches(f.down, plan_div(s.d_model, 32), f.qkv, nq, KB, 2), 0};
        for (int i = 0; i < 5; ++i)
            printf("%d %d %d %d %d %d  ", p[i]->tile, p[i]->lds, p[i]->ks, p[i]->tile ? tile_rows_for(M, blocks[i], p[i]->ks, s.n_cus) : 0,
                   p[i]->tile && i < 4 && tile_two_heights(M, blocks[i], p[i]->ks, s.n_cus), touched[i]);
        printf("\n");
    }
}
"""
TILES, ROWGROUPS = 16, 4
NAMES = ("qkv", "out", "gate_up", "down", "head")


def choose(queries):
    """queries: (arch dict, rows, window of a step with its head fused (0: prompt rows), kernel flags) -> a dict each.  Per projection, by
    name: (LDS tile shape or -1, K splits).  by_tile: whether it runs through the tile kernels (tile: whether any does), and where it does
    tile_rows (of a workgroup) and two_heights (in one launch).  touches: how many workgroups of its launch, where that is one through
    LDS tiles, touch the next projection's weights."""
    with tempfile.TemporaryDirectory() as tmp:
        src, exe = os.path.join(tmp, "main.cpp"), os.path.join(tmp, "main")
        with open(src, "w") as f:
            f.write(_MAIN)
        subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", exe], check=True)
        lines = []
        for a, rows, window, flags in queries:
            win32 = int(window == 32 and not flags & 2048)
            lines.append(f"{a['d_model']} {a['n_heads']} {a['n_kv_heads']} {a['d_ff']} {a['sample_hi'] - a['sample_lo']} {flags} {rows} {win32}\n")
        out = subprocess.run([exe], input="".join(lines), capture_output=True, text=True, check=True).stdout
    res = []
    for line in out.splitlines():
        v = [int(x) for x in line.split()]
        by = {n: v[6 * i:6 * i + 6] for i, n in enumerate(NAMES)}
        r = {n: (x[1], x[2]) for n, x in by.items()}
        r["by_tile"] = {n: bool(x[0]) for n, x in by.items()}
        r["tile"] = any(r["by_tile"][n] for n in NAMES[:4])
        r["tile_rows"] = {n: x[3] for n, x in by.items() if x[0]}
        r["two_heights"] = {n: bool(x[4]) for n, x in by.items() if x[0]}
        r["touches"] = {n: x[5] for n, x in by.items()}
        res.append(r)
    return res


def evaluate(tmp, expression, queries):
    """The value of an expression of plans.h in int q[8] (the query's numbers) for each query."""
    src, exe = os.path.join(str(tmp), "expression.cpp"), os.path.join(str(tmp), "expression")
    n = len(queries[0])
    with open(src, "w") as f:
        f.write('#include <cstdio>\n#include "plans.h"\nint main() {\n    int q[8] = {0}, n = 0;\n    while (scanf("%d", &q[n]) == 1)\n'
                f'        if (++n == {n}) {{ n = 0; printf("%.9g\\n", (double)({expression})); }}\n}}\n')
    subprocess.run(["g++", "-std=c++17", "-O1", "-I", CSRC, src, "-o", exe], check=True)
    out = subprocess.run([exe], input="\n".join(" ".join(map(str, q)) for q in queries), capture_output=True, text=True, check=True).stdout
    return [float(x) for x in out.split()]
