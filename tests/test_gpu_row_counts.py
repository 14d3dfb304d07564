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


@pytest.mark.parametrize("name,n_seqs,window,prompt,flags", [
    ("small_fused64", 3, 16, 13, 0),      # 96 rows; a prompt forward of 72
    ("small_fused64", 3, 16, 8, 0),       # ... of 42: row groups of 32 rows within a context of wider steps
    ("small_fused64", 1, 33, 25, 4),      # 66 rows in row groups
    ("small_fused64", 1, 150, 140, 0),    # 300 rows, 278 prompt rows
    ("small_fused64", 1, 150, 140, 16),   # ... through the tile kernels, whole K
    ("small_fused128", 3, 41, 70, 0),     # 246 rows, 414 prompt rows
    ("small_tile", 5, 27, 60, 16),        # 270 rows, ragged column tiles
    ("small_tile", 5, 27, 60, 80),        # ... in tiles of 256 rows
])
def test_norm_gains_cost_no_precision(oracle, name, n_seqs, window, prompt, flags):
    """Norm gains drawn from U(0.5, 1.5), on contexts that once ran the generic GEMMs with the caller's bf16 weights and the
    gains applied in fp32: the error of the first step's logits against double precision (2-norm) is no larger than that
    of the reference kernels, which still do that.  Both sides round at the same number of places (a projection's operand
    once, after the gain), but for the attention probabilities, which the MFMA kernels have always rounded: one of some ten
    roundings a layer, up to 1.05 on the ratio.  Gains rounded into the weights are a second rounding of every product of
    the projections behind a norm, about half of what reaches the logits: sqrt(1.4) = 1.18 (1.15 - 1.22 measured).  The
    bound lies between; three weight sets a case, so that the ratio scatters by a percent or two."""
    import numpy as np
    cfg = workload.get_config(name)
    sq = np.zeros((2, 2))
    for i, f in [(i, f) for i in range(3) for f in (flags, 1)]:
        cfg["seed"] = 100 + i
        o, g, cond, uncond, n = make_pair(oracle, cfg, window=window, n_image=window + 20, n_seqs=n_seqs, prompt_len=prompt,
                                          kernel_flags=f, head_alpha=6.0, std=0.05, random_gains=True)
        want = o.peek_logits().astype(np.float64)
        g.step()
        got = g.logits().astype(np.float64)
        assert np.isfinite(got).all()
        sq[int(f == 1)] += ((got - want) ** 2).sum(), (want ** 2).sum()
        o.close(), g.close()
    err = np.sqrt(sq[:, 0] / sq[:, 1])
    print(name, n_seqs, window, prompt, flags, "relative error, reference kernels, ratio:", err, err[0] / err[1])
    assert err[0] <= 1.08 * err[1]


@pytest.mark.parametrize("n_seqs,flags", [(1, 0), (1, 128), (1, 256), (2, 0), (2, 128), (2, 256), (2, 512), (3, 0)])
def test_fewer_sequences_than_the_context_holds(n_seqs, flags):
    """A context for three 16-token windows (96 rows: norm gains in the rows) with one or two of them in use: 32 and 64 rows,
    whose projections run as 16-row halves, 32- and 64-row groups and, with more than 256 column groups (8 256-wide MLP, 17 000
    ids), as workgroups of two widths; flags 128, 256 and 512 take the other kernels.  Against float64, bound as in
    tests/test_gpu_lds_tiles.py; gains from U(0.5, 1.5)."""
    import numpy as np
    import torch
    import paper_2512_07503_amd as sjd
    from test_gpu_lds_tiles import _forward64, _weights, case_arch
    arch, window, n = case_arch(256, 4, 2, 8256, 17000), 16, 40
    w = _weights(arch, 13)
    for name in ("attn_norm", "mlp_norm"):
        w[name] = [(torch.rand(256, device="cuda") + 0.5).to(torch.bfloat16) for _ in w[name]]
    w["final_norm"] = (torch.rand(256, device="cuda") + 0.5).to(torch.bfloat16)
    rng = np.random.default_rng(4)
    cond = [rng.integers(0, arch["vocab"], c).astype(np.int32) for c in (20, 9, 31)[:n_seqs]]
    uncond = [rng.integers(0, arch["vocab"], c).astype(np.int32) for c in (14, 20, 1)[:n_seqs]]
    g = sjd.Decoder(arch, w, "bf16", window, 80, max_seqs=3, top_k=200, seed=5, kernel_flags=flags | sjd.KEEP_LOGITS)
    for again in range(2):   # the second time over the first one's buffers, replaying its graph
        assert g.prefill(cond, uncond, [n] * n_seqs) == 0
        windows = [g.window(s)[0] for s in range(n_seqs)]
        g.step()
        out = g.logits().astype(np.float64)
        assert np.isfinite(out).all()
        for s in range(n_seqs):
            for b, p in enumerate((cond[s], uncond[s])):
                want = _forward64(arch, w, np.concatenate([p, windows[s][1:]]), window)
                err = np.linalg.norm(out[s, b] - want) / np.linalg.norm(want)
                print(n_seqs, flags, "sequence", s, "branch", b, "relative error of the logits", err)
                assert err < 1.5e-2


@pytest.mark.parametrize("window,ff", [(16, 2560), (32, 2560), (24, 2048), (32, 2048)])
def test_row_splits_change_no_bit(window, ff):
    """A 1280-wide model (its MLP narrow enough that K is whole in every projection), up to 64 rows in workgroups of 16 and 32 against all of them
    in one (flag 128; every workgroup walking K from 0, since with the rotation of k the block's number says where it starts).  MLP 2560: gate/up
    of 64 rows in row groups of 32 and of 64; 2048: in the few-row kernels, four tiles of 16 rows with the flag.  The same
    sums in the same order, and a rotation whose operations the source fixes, so logits, keys and values agree bit for bit.
    (Which of the rotation's products was rounded ahead of the sum was once left to the compiler: one key in some 10^5 moves to
    the next bf16, and the pages hold 24 x 32 x 1280 keys of this step.)"""
    import numpy as np
    import paper_2512_07503_amd as sjd
    from test_gpu_lds_tiles import _weights, case_arch
    arch = dict(case_arch(1280, 20, 20, ff, 3001), n_layers=24)
    w = _weights(arch, 17)
    runs = []
    for flags in (sjd.NO_K_ROTATION, sjd.NO_K_ROTATION | sjd.NO_ROW_SPLIT):
        g = sjd.Decoder(arch, w, "bf16", window, 200, top_k=200, seed=5, kernel_flags=flags | sjd.KEEP_LOGITS)
        one = [np.array([7], dtype=np.int32)]   # a prompt of one token: no forward before the step
        assert g.prefill(one, one, [190]) == 0
        g.step()
        # the cache pages that end a snapshot: one page of 64 tokens a segment holds the whole window
        runs.append((g.logits(), g.snapshot()[-2 * arch["n_layers"] * 2 * 64 * 1280 * 2:]))
        g.close()
    assert runs[0][0].any() and runs[0][1].any()
    assert all(np.array_equal(a, b) for a, b in zip(*runs))
