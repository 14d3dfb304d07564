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
        const int d64 = plan_div(s.d_model, 64) * 2;
        auto mixed = [&](int blocks, int ks) { return (int)tile_two_heights(M, blocks, ks, s.n_cus); };
        auto rows = [&](int blocks, int ks) { return tile_rows_for(M, blocks, ks, s.n_cus); };
        const int ko = tile_splits(s, M, s.q_dim() / 16), kd = tile_splits(s, M, s.d_ff / 16);
        printf("%d %d %d %d %d  ", f.qkv.tile, f.o.tile, f.gate_up.tile, f.down.tile, f.head.tile);
        printf("%d  %d %d  %d %d  %d %d  %d %d  %d %d  %d %d %d %d  %d %d %d %d  %d %d\n", f.tile, f.qkv.lds, f.qkv.ks, f.o.lds, f.o.ks, f.gate_up.lds,
               f.gate_up.ks, f.down.lds, f.down.ks, f.head.lds, f.head.ks, rows(s.qkv_groups() * 2, 1), rows(d64, ko), rows(s.gate_up_groups() * 2, 1),
               rows(d64, kd), mixed(s.qkv_groups() * 2, 1), mixed(d64, ko), mixed(s.gate_up_groups() * 2, 1), mixed(d64, kd), ko, kd);
    }
}
"""
TILES, ROWGROUPS = 16, 4


def choose(queries):
    """queries: (arch dict, rows, window of a step with its head fused (0: prompt rows), kernel flags) -> a dict each: tile (every
    projection through the tile kernels, whose heights, height mixes and K splits come along), by_tile (each projection on its own) and
    per projection (LDS tile shape or -1, K splits)."""
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
        by_tile, v = v[:5], v[5:]
        names = ("qkv", "out", "gate_up", "down")
        r = {n: (v[1 + 2 * i], v[2 + 2 * i]) for i, n in enumerate(names + ("head",))}
        r["tile"] = bool(v[0])
        r["by_tile"] = {n: bool(t) for n, t in zip(names + ("head",), by_tile)}
        r["tile_rows"] = dict(zip(names, v[11:15]))
        r["two_heights"] = {n: bool(m) for n, m in zip(names, v[15:19])}
        r["tile_splits"] = dict(zip(("out", "down"), v[19:21]))
        res.append(r)
    return res
