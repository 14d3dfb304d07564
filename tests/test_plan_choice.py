"""The choice of projection kernels (csrc/plans.h): the GPU tests that are there for certain kernels reach them."""
import plan_choice
import workload

EPILOGUE = dict(qkv="QKV", gate_up="SWIGLU", head="HEAD")


def _pairs(plan, with_head):
    """(epilogue, LDS tile shape or -1) of the launches of a forward that do not run through the tile kernels."""
    out = set()
    for proj in ("qkv", "out", "gate_up", "down") + (("head",) if with_head else ()):
        shape, ks = plan[proj]
        if plan["by_tile"][proj]:
            continue
        out.add((EPILOGUE.get(proj, "RESID" if ks == 1 else "PARTIAL"), shape))
    return out


def test_the_lds_tile_cases_reach_every_shape_and_epilogue():
    import test_gpu_lds_tiles as t
    queries, heads = [], []
    for d, h, kv, ff, ids, window, lens in t.CASES:
        a, rows = t.case_arch(d, h, kv, ff, ids), len(lens) * 2 * window
        queries += [(a, rows, window, 0), (a, rows, window, 2048), (a, sum(c + u - 2 for c, u in lens), 0, 0)]
        heads += [True, True, False]
    reached = set()
    for plan, head in zip(plan_choice.choose(queries), heads):
        reached |= _pairs(plan, head)
    shapes = {(e, s) for e in ("QKV", "SWIGLU", "RESID", "PARTIAL", "HEAD") for s in range(4)} | {("HEAD", 4)}
    assert shapes <= reached, shapes - reached
    # the fused head's shape is compared with two of the others: windows of 32 with and without it
    fused = [(p[0]["head"][0], p[1]["head"][0]) for p in zip(*[iter(plan_choice.choose([q for q in queries if q[2] == 32]))] * 2) if p[0]["head"][0] >= 0]
    assert {f for f, _ in fused} == {4} and len({g for _, g in fused}) >= 3, fused


def test_the_benchmark_shape_cases_reach_the_tile_kernels():
    arch = workload.get_config("cfg4")["arch"]

    def plan(seqs, flags):
        return plan_choice.choose([(arch, seqs * 64, 32, flags)])[0]
    assert not plan(3, 0)["tile"] and not plan(5, 0)["tile"]
    p = plan(5, 16)                           # all through the tile kernels, the down projection with its K split
    assert all(p["by_tile"].values()) and p["two_heights"]["gate_up"] and 128 in p["tile_rows"].values() and p["down"][1] > 1
    p = plan(7, 0)                            # gate/up and head alone, beside LDS tiles and a down projection whose K they split
    assert [n for n, t in p["by_tile"].items() if t] == ["gate_up", "head"] and p["two_heights"]["gate_up"] and p["down"][0] >= 0 and p["down"][1] > 1
    p = plan(8, 0)                            # the benchmark's throughput batch
    assert p["by_tile"]["gate_up"] and p["by_tile"]["down"] and p["down"][1] == 4
    assert not plan(8, 4)["tile"]             # row groups only
    import test_gpu_e2e as e
    marks = [m for m in e.test_benchmark_shapes_bf16.pytestmark if m.name == "parametrize"][0]
    cases = {(c[4], c[5]) for c in marks.args[1] if c[0] == "cfg4"}
    assert {(3, 0), (5, 0), (5, 16), (5, 16 + 64), (5, 16 + 256), (7, 0)} <= cases


def test_few_rows_and_the_row_group_flag_keep_the_row_groups():
    arch = workload.get_config("cfg1")["arch"]
    for rows, flags in ((32, 0), (64, 0), (500, 4)):
        p = plan_choice.choose([(arch, rows, 0, flags)])[0]
        assert not p["tile"] and all(p[n][0] == -1 for n in ("qkv", "out", "gate_up", "down", "head"))


def test_the_big_tile_cases_reach_the_256_x_256_tiles():
    import test_gpu_lds_tiles as t
    queries = [(t.case_arch(d, h, kv, ff, ids), sum(c + u - 2 for c, u in lens), 0, 0) for d, h, kv, ff, ids, _, lens in t.BIG_CASES]
    got = [(n, p["by_tile"]["gate_up" if n == "qkv" else "qkv"]) for p in plan_choice.choose(queries) for n in ("qkv", "gate_up") if p[n][0] == 5]
    assert got == [("gate_up", False), ("qkv", True), ("gate_up", False), ("qkv", False), ("qkv", True)], got


def test_the_whole_k_cases_reach_the_tile_kernels_with_256_rows():
    import test_gpu_lds_tiles as t
    assert {(c[5] == 1, c[7]) for c in t.WHOLE_K_CASES} == {(True, 0), (True, 16), (False, 16)}   # gains in the weights, in the rows
    queries = [(t.case_arch(d, h, kv, ff, ids), sum(c + u - 2 for c, u in lens), 0, flags) for d, h, kv, ff, ids, _, lens, flags in t.WHOLE_K_CASES]
    for p, q in zip(plan_choice.choose(queries), queries):
        for n in ("out", "down"):
            assert p["by_tile"][n] and p[n][1] == 1 and p["tile_rows"][n] == 256 and not p["two_heights"][n], p
        assert p["by_tile"]["gate_up"] and p["tile_rows"]["gate_up"] == 256 and (p["by_tile"]["qkv"] if q[3] else p["qkv"][0] == 5), p


def test_the_tile_before_row_groups_case_is_one():
    import test_gpu_lds_tiles as t
    queries = [(t.case_arch(d, h, kv, ff, ids), sum(c + u - 2 for c, u in lens), 0, 0) for d, h, kv, ff, ids, _, lens in t.TILE_BEFORE_ROW_GROUPS]
    for p in plan_choice.choose(queries):
        assert p["by_tile"]["out"] and p["out"] == (-1, 1) and not p["by_tile"]["gate_up"] and p["gate_up"][0] == -1, p


def test_narrow_models_keep_the_row_groups_at_any_number_of_rows():
    import test_gpu_lds_tiles as t
    queries = [(t.case_arch(d, h, kv, ff, ids), sum(c + u - 2 for c, u in lens), 0, 0) for d, h, kv, ff, ids, _, lens in t.NARROW_CASES]
    for p in plan_choice.choose(queries):
        assert all(p[n] == (-1, 1) and not p["by_tile"][n] for n in ("out", "down")), p
    # more than a workgroup per CU: LDS tiles
    assert all(plan_choice.choose([(t.case_arch(512, 8, 8, 1792, 301), 1434, 0, 0)])[0][n][0] >= 0 for n in ("out", "down"))


def test_row_groups_are_taken_for_what_they_touch_ahead():
    import test_gpu_lds_tiles as t
    for d, h, kv, ff, rows in ((1280, 20, 20, 3456, 70), (1280, 20, 5, 3456, 67), (640, 10, 10, 3200, 86)):
        p = plan_choice.choose([(t.case_arch(d, h, kv, ff, 301), rows, 0, 0)])[0]
        assert p["down"] == (-1, 1) and p["qkv"] == (-1, 1), p
    for rows in (71, 128):
        p = plan_choice.choose([(t.case_arch(1024, 16, 8, 3584, 301), rows, 0, 0)])[0]
        assert p["out"] == (-1, 1) and p["gate_up"] == (-1, 1), p


def test_short_launches_of_narrow_models_stay_out_of_the_tile_kernels():
    import test_gpu_lds_tiles as t
    short = [(1024, 16, 16, 3584, 1257), (2048, 32, 32, 5504, 704), (2560, 20, 20, 6400, 1152), (1280, 20, 10, 4480, 931)]
    longer = [(4096, 32, 32, 11008, 512), (4096, 32, 8, 14336, 2000), (3072, 24, 24, 12288, 1024), (2048, 16, 8, 10240, 1024)]
    plans = plan_choice.choose([(t.case_arch(d, h, kv, ff, 301), rows, 0, 0) for d, h, kv, ff, rows in short + longer])
    assert [p["tile"] for p in plans] == [False] * 4 + [True] * 4


def test_the_touching_cases_touch():
    import test_gpu_lds_tiles as t
    import test_gpu_touched_weights as w
    queries = []
    for d, h, kv, ff, ids, window, lens in w.CASES:
        a = t.case_arch(d, h, kv, ff, ids)
        queries.append([(a, len(lens) * 2 * window, window, 0), (a, sum(c + u - 2 for c, u in lens), 0, 0)])
    seen = [{n for p in plan_choice.choose(q) for n, wgs in p["touches"].items() if wgs} for q in queries]
    assert all(seen) and set.union(*seen) == {"qkv", "out", "gate_up", "down"}, seen


def test_qkv_projections_are_expected_to_take_what_launches_took(tmp_path):
    """Medians of QKV launches of the tile kernels, all heads their own: 256-row tiles, 128-row tiles, both heights.  Within 15 %: 11 is
    what a rate per height leaves, 37 what the rate of the other projections left."""
    measured = [(4096, 32, 1700, 250.5), (4096, 32, 1932, 269.0), (4096, 32, 1964, 268.2), (5120, 40, 1300, 309.9), (5120, 40, 1900, 352.4),
                (4096, 32, 1300, 184.7), (4096, 32, 1500, 196.4), (5120, 40, 1700, 314.4), (3072, 24, 2048, 152.4),
                (3072, 24, 1300, 126.1), (3072, 24, 1600, 137.0)]
    out = plan_choice.evaluate(tmp_path, "tile_us(PLAN_QKV, q[2], q[1] * 12, q[0] / 16, 1, 256)", [m[:3] for m in measured])
    for m, us in zip(measured, out):
        assert abs(us - m[3]) < 0.15 * m[3], (m, us)
    # and so 128 x 128 or 192 x 128 LDS tiles, 226 and 153 us, are taken
    import test_gpu_lds_tiles as t
    for p in plan_choice.choose([(t.case_arch(4096, 32, 32, ff, 301), rows, 0, 0) for ff, rows in ((7136, 1964), (11008, 1964), (6048, 1960), (11008, 1300))]):
        assert not p["by_tile"]["qkv"] and p["qkv"][0] in (2, 3), p


def test_a_wider_mlp_is_not_expected_to_take_less_time(tmp_path):
    """4096 wide, 8 key/value heads, 1940 to 2040 rows, MLPs of 5664 to 8192: a line in K between two kernels of the down projection once put whole
    layers of the narrower ones into kernels that were 2 to 3 % slower."""
    mlps = range(5664, 8193, 32)
    for rows in (1940, 1980, 2000, 2040):
        us = plan_choice.evaluate(tmp_path, "layer_us(forward_plan(ProjShape{4096, 32, q[2], q[0], 16384, 256, 0}, q[1], false))", [(ff, rows, 8) for ff in mlps])
        for ff, a, b in zip(mlps, us, us[1:]):
            assert b > a - 2.0, (rows, ff, a, b)   # 2 us: where kernels take turns, a layer gains 2 % before it changes


def test_no_projection_leaves_out_a_256_x_128_tile_that_is_expected_to_be_faster(tmp_path):
    queries = [(d, g, ff, rows) for d in (4096, 5120) for g in (1, 4) for ff in range(d, 2 * d, 256) for rows in range(1040, 2040, 90)]
    best = "[&] { const ProjShape s{q[0], q[0] / 128, q[0] / 128 / q[1], q[2], 16384, 256, 0}; const ProjPlan p = forward_plan(s, q[3], false).down; return lds_us(6, PLAN_RESID, q[3], q[0] / 32, q[2] / 16, 1, 256) - p.us; }()"
    for q, slack in zip(queries, plan_choice.evaluate(tmp_path, best, queries)):
        assert slack > -1e-9, (q, slack)


def test_no_launch_is_expected_to_slow_down_for_its_size(tmp_path):
    """Gate/up of 28672 x 4096 and 35840 x 5120 in whole tiles of 192 and of 128 rows: one row tile more never costs more than a tile's share and 1 %
    (a step of 4.5 % at 0.42 TFLOP once did), and long launches of 192 x 128 tiles take what was measured within 4 %."""
    for d, blocks in ((4096, 896), (5120, 1120)):
        for shape, rows in ((2, 128), (3, 192)):
            tiles = range(4, 2049 // rows)
            us = plan_choice.evaluate(tmp_path, "lds_us(q[0], PLAN_SWIGLU, q[1], q[2], q[3], 1, 256)", [(shape, rows * n, blocks, d // 16) for n in tiles])
            share = plan_choice.evaluate(tmp_path, "plan_div(plan_div(plan_div(q[0], 4), 8) * q[1], 32)", [(blocks, n) for n in tiles])   # of the busiest CU
            for n, a, b, u, v in zip(tiles, us, us[1:], share, share[1:]):
                if v * n <= u * (n + 1):   # which grows no faster than the rows
                    assert b <= a * (n + 1) / n * 1.01, (d, shape, n, a, b)
    measured = [(4096, 14336, 1500, 337.8), (4096, 14336, 1700, 381.7), (4096, 14336, 1780, 425.0), (4096, 14336, 1800, 418.3), (4096, 14336, 1950, 470.3),
                (4096, 14336, 2048, 470.9), (5120, 13824, 1480, 400.5), (5120, 13824, 1700, 460.3), (5120, 13824, 1900, 514.5), (5120, 13824, 2048, 568.2),
                (5120, 17920, 1140, 406.2), (5120, 17920, 1300, 468.7), (5120, 17920, 1500, 526.5), (5120, 17920, 1900, 659.0), (5120, 17920, 2048, 747.6)]
    for m, us in zip(measured, plan_choice.evaluate(tmp_path, "lds_us(3, PLAN_SWIGLU, q[2], q[1] / 16, q[0] / 16, 1, 256)", [m[:3] for m in measured])):
        assert abs(us - m[3]) < 0.04 * m[3], (m, us)


def test_layers_expected_to_gain_less_than_2_percent_stay_out_of_the_tile_kernels():
    """Prompts, and by how much the tile kernels made them slower where 1.5 % sufficed: 5.8, 4.5, 4.0, 3.7, 3.0, 2.8, 2.5 and 1.3 %."""
    import test_gpu_lds_tiles as t
    slower = [(3072, 24, 6, 6208, 1218), (3072, 24, 24, 10272, 654), (5120, 40, 40, 5248, 1304), (3072, 24, 24, 3808, 1044),
              (3072, 24, 24, 3168, 1286), (3072, 24, 24, 4512, 1542), (2560, 20, 20, 8160, 1522), (5120, 40, 10, 17152, 396)]
    for p in plan_choice.choose([(t.case_arch(d, h, kv, ff, 301), rows, 0, 0) for d, h, kv, ff, rows in slower]):
        assert not p["tile"], p
