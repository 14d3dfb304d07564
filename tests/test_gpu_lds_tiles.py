"""Projections through LDS tiles (more than 64 rows): every tile shape and epilogue against a float64 forward of the same
bf16 weights, at row counts that end inside tiles.  Which shape a projection takes depends on the model's width and the
rows; tests/test_plan_choice.py computes it for CASES and holds them to all shapes.

Bound: a projection's operand, the rotated queries and keys, values, probabilities, attention output and hidden activations are
rounded to bf16 (2^-9 / sqrt(3) = 1.1e-3 in the 2-norm each, the gains where they are in the weights once more), some
ten independent ones a layer: sqrt(20) x 1.1e-3 = 5e-3 for two layers of projections that neither shrink nor amplify, up to
twice that where they amplify (0.02 sqrt(d) = 1.28 at 4096); 1.5e-2 leaves half of that again.  Wider models have weights of 1.28 / sqrt(d):
at 16384 with 0.02 a projection amplifies 2.56 times, the attention's scores reach 2.56^2 times a unit normal, whose operands' roundings alone
move a probability by 6.6 sqrt(2) x 1.1e-3 = 1.0e-2 a layer (2.2e-2 measured over two)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _weights(arch, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    d, hd, ff = arch["d_model"], arch["d_model"] // arch["n_heads"], arch["d_ff"]
    q, kv = arch["n_heads"] * hd, arch["n_kv_heads"] * hd

    def rnd(*s):
        return torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) * min(0.02, 1.28 / d ** 0.5)
    shapes = dict(wq=(q, d), wk=(kv, d), wv=(kv, d), wo=(d, q), w_gate=(ff, d), w_up=(ff, d), w_down=(d, ff))
    w = {n: [rnd(*s) for _ in range(arch["n_layers"])] for n, s in shapes.items()}
    for n in ("attn_norm", "mlp_norm"):
        w[n] = [1 + 4 * rnd(d) for _ in range(arch["n_layers"])]
    w.update(tok_emb=rnd(arch["vocab"], d), final_norm=1 + 4 * rnd(d), lm_head=rnd(arch["vocab"], d))
    return w


# d, heads, kv heads, ff, sampled ids, window, (conditional, unconditional) prompt tokens of each sequence: rows of the step
# / packed prompt rows
CASES = [
    (768, 12, 12, 2048, 8003, 32, [(70, 66), (70, 66)]),             # 128, guidance inside the head / 268
    (768, 12, 12, 2048, 8003, 33, [(70, 68)]),                       # 66 / 136
    (1280, 20, 20, 3456, 3001, 48, [(60, 61)]),                      # 96 / 119
    (1280, 20, 20, 3456, 3001, 250, [(117, 3)]),                     # 500 / 118
    (1280, 20, 20, 3456, 3001, 16, [(120, 96), (40, 41), (77, 130), (99, 100), (140, 111), (2, 1)]),   # 192 / 945
    (1280, 20, 20, 3456, 3001, 1, [(700, 702)]),                     # 2 / 1400
    (2048, 16, 16, 5632, 3001, 65, [(120, 141)]),                    # 130 / 259
    (2048, 16, 8, 5632, 3001, 32, [(200, 210), (280, 313)]),         # 128 / 999
    (2048, 16, 8, 5632, 20003, 32, [(200, 210), (280, 313)]),        # 128, guidance inside the head / 999
    (2048, 16, 8, 5632, 20003, 32, [(200, 210), (280, 313), (50, 40)]),   # 192, guidance inside the head / 1087
    (3072, 24, 8, 8192, 3001, 33, [(170, 93)]),                      # 66, 128-wide heads / 261
    (4096, 32, 32, 11008, 3001, 96, [(64, 64)]),                     # 192 / 126
    (4096, 32, 8, 14336, 3001, 35, [(350, 352), (340, 358)]),        # 140 / 1396
]


def case_arch(d, heads, kv, ff, ids):
    return dict(n_layers=2, d_model=d, n_heads=heads, n_kv_heads=kv, d_ff=ff, vocab=ids + 99, sample_lo=50, sample_hi=50 + ids)


def _forward64(arch, w, tokens, last):
    """Logits of the last rows of a causal forward in float64, without any of the library's code."""
    import torch
    f64 = torch.float64
    d, H, Hkv = arch["d_model"], arch["n_heads"], arch["n_kv_heads"]
    hd, T = d // H, len(tokens)
    x = w["tok_emb"][torch.as_tensor(tokens, device="cuda").long()].to(f64)
    freq = torch.tensor(10000.0, dtype=f64, device="cuda") ** (-2.0 * torch.arange(hd // 2, device="cuda", dtype=f64) / hd)
    ang = torch.arange(T, device="cuda", dtype=f64)[:, None] * freq
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    mask = torch.full((T, T), float("-inf"), device="cuda", dtype=f64).triu(1)

    def norm(v, gain):
        return v / torch.sqrt((v * v).mean(-1, keepdim=True) + 1e-5) * gain.to(f64)

    def rope(v):
        a, b = v[..., :hd // 2], v[..., hd // 2:]
        return torch.cat([a * cos - b * sin, b * cos + a * sin], -1)
    for l in range(arch["n_layers"]):
        h = norm(x, w["attn_norm"][l])
        q, k, v = ((h @ w[n][l].to(f64).T).view(T, -1, hd) for n in ("wq", "wk", "wv"))
        q, k, o = rope(q), rope(k), torch.empty(T, H, hd, dtype=f64, device="cuda")
        for i in range(H):
            j = i // (H // Hkv)
            o[:, i] = torch.softmax(q[:, i] @ k[:, j].T.contiguous() / hd ** 0.5 + mask, -1) @ v[:, j]
        x = x + o.reshape(T, d) @ w["wo"][l].to(f64).T
        h = norm(x, w["mlp_norm"][l])
        x = x + (torch.nn.functional.silu(h @ w["w_gate"][l].to(f64).T) * (h @ w["w_up"][l].to(f64).T)) @ w["w_down"][l].to(f64).T
    head = w["lm_head"][arch["sample_lo"]:arch["sample_hi"]].to(f64)
    return (norm(x[-last:], w["final_norm"]) @ head.T).cpu().numpy()


@pytest.mark.parametrize("d,heads,kv,ff,ids,window,lens", CASES)
def test_against_float64(d, heads, kv, ff, ids, window, lens, kernels=0):
    import torch
    import paper_2512_07503_amd as sjd
    arch = case_arch(d, heads, kv, ff, ids)
    w, n, S = _weights(arch, 11), 300, len(lens)
    max_ctx = max(max(p) for p in lens) + n
    rng = np.random.default_rng(2)
    cond = [rng.integers(0, arch["vocab"], c).astype(np.int32) for c, _ in lens]
    uncond = [rng.integers(0, arch["vocab"], u).astype(np.int32) for _, u in lens]
    out = []
    for flags in (0, sjd.NO_HEAD_FUSION):
        g = sjd.Decoder(arch, w, "bf16", window, max_ctx, max_seqs=S, top_k=200, seed=5, kernel_flags=flags | kernels | sjd.KEEP_LOGITS)
        assert g.prefill(cond, uncond, [n] * S) == 0
        windows = [g.window(s)[0] for s in range(S)]
        g.step()
        out.append(g.logits().astype(np.float64))
        g.close()
    assert np.isfinite(out[0]).all()
    for s in sorted({0, S - 1}):
        for b, p in enumerate((cond[s], uncond[s])):
            want = _forward64(arch, w, np.concatenate([p, windows[s][1:]]), window)
            err = np.linalg.norm(out[0][s, b] - want) / np.linalg.norm(want)
            row = np.linalg.norm(out[0][s, b] - want, axis=1) / np.linalg.norm(want, axis=1)
            print(d, window, lens, "sequence", s, "branch", b, "relative error of the logits", err, "of the worst row", row.max())
            # a row's error has few independent directions (its 2 x 10 rounded vectors): three times the mean at most
            assert err < 1.5e-2 and row.max() < 4.5e-2
    # windows of 32: the head that combines the branches against the tile shape that it takes otherwise, the same sums
    assert np.abs(out[0] - out[1]).max() <= (1e-5 if window == 32 else 0.0) * np.abs(out[1]).max()


# 256 x 256 tiles (QKV or gate/up of prompts whose tiles number at most one per CU), ragged in rows and in columns; same bound
BIG_CASES = [
    (2048, 16, 16, 5664, 3001, 33, [(500, 505)]),    # 1003 prompt rows: gate/up, its last column tile two blocks wide
    (2048, 16, 16, 5664, 3001, 1, [(1000, 1005)]),   # 2003, beside tile kernels: QKV
    (1280, 20, 20, 6912, 3001, 1, [(480, 480)]),     # 958, 64-wide heads: gate/up
    (3072, 24, 24, 8224, 3001, 2, [(700, 709)]),     # 1407, beside LDS tiles of other shapes: QKV
    (4096, 32, 8, 5664, 3001, 33, [(1000, 1003)]),   # 2001, gains in the rows, beside tile kernels: QKV
]


@pytest.mark.parametrize("d,heads,kv,ff,ids,window,lens", BIG_CASES)
def test_big_tiles_against_float64(d, heads, kv, ff, ids, window, lens):
    test_against_float64(d, heads, kv, ff, ids, window, lens)


# A whole-K output projection of the tile kernels ahead of a gate/up in row groups that sums the squares for itself (gains in the weights)
TILE_BEFORE_ROW_GROUPS = [
    (16384, 128, 32, 128, 301, 1, [(250, 244)]),     # 492 prompt rows
]


@pytest.mark.parametrize("d,heads,kv,ff,ids,window,lens", TILE_BEFORE_ROW_GROUPS)
def test_tile_kernels_before_row_groups_against_float64(d, heads, kv, ff, ids, window, lens):
    test_against_float64(d, heads, kv, ff, ids, window, lens)


# Narrow models: output and down projections in row groups, a workgroup per CU at most, however many rows
NARROW_CASES = [
    (256, 4, 4, 1280, 301, 33, [(380, 365)]),        # 743 prompt rows
    (512, 8, 2, 1376, 301, 1, [(470, 466)]),         # 934
]


@pytest.mark.parametrize("d,heads,kv,ff,ids,window,lens", NARROW_CASES)
def test_row_groups_of_many_rows_against_float64(d, heads, kv, ff, ids, window, lens):
    test_against_float64(d, heads, kv, ff, ids, window, lens)


# Long prompts whose projections run through the tile kernels with K whole: output and down projections of 256-row tiles that
# leave one partial sum of squares per column tile (64 and 32 of them), read by a 256 x 256 QKV and a 256-row gate/up (by choice, 8192 wide) or by tile kernels (flag 16: all of them); gains in the weights (window 1) and in the rows (33).  Ragged in rows and in the
# MLP's columns; same bound.
WHOLE_K_CASES = [
    (8192, 64, 16, 10912, 3001, 1, [(512, 511)], 0),     # 1021 prompt rows
    (4096, 32, 8, 5664, 3001, 1, [(1022, 1019)], 16),    # 2039
    (4096, 32, 8, 5664, 3001, 33, [(1000, 1003)], 16),   # 2001
]


@pytest.mark.parametrize("d,heads,kv,ff,ids,window,lens,kernels", WHOLE_K_CASES)
def test_whole_k_tiles_against_float64(d, heads, kv, ff, ids, window, lens, kernels):
    test_against_float64(d, heads, kv, ff, ids, window, lens, kernels)
