"""Prompts of unequal lengths, one-token prompts among them, packed into prefill forwards without gaps: the first steps'
logits against the oracle, which runs every prompt on its own.  Tolerance of the small stress models: 8e-2 of a row's
largest |logit| (tests/test_gpu_e2e.py says where it comes from), 1e-4 in fp32."""
import numpy as np
import pytest

import workload
from helpers import gpu_weights, logits_error

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name,lens,flags", [
    ("small_f32", [(1, 1)], 0),                                  # nothing to prefill
    ("small_f32", [(40, 1), (2, 33), (65, 17)], 0),              # segments that start inside a query tile
    ("small_f32", [(300, 290)], 0),                              # two forwards of at most 512 rows
    ("small_bf16", [(200, 31), (97, 300)], 0),                   # generic projections, two forwards
    ("small_fused64", [(33, 1), (1, 70), (32, 34)], 0),
    ("small_fused64", [(1500, 1300)], 0),                        # a branch that starts in one forward and goes on in the next
    ("small_fused64", [(90, 80), (100, 60)], 1),                 # reference kernels
    ("small_fused64", [(90, 80), (100, 60)], 8),                 # chunked attention, window by window, in a row group
    ("small_fused128", [(257, 1), (129, 70), (31, 32)], 8),      # ... 192 rows, segments that end in different windows
    ("small_bf16", [(200, 31)], 8),                              # ... generic projections
    ("small_fused128", [(257, 1), (129, 70), (31, 32)], 0),
    ("small_tile", [(400, 399), (127, 2), (258, 130)], 16),      # tile kernels, ragged last tile
])
def test_packed_prompts(oracle, name, lens, flags):
    import paper_2512_07503_amd as sjd
    cfg = workload.get_config(name)
    arch, n = cfg["arch"], 40
    S, L, max_ctx = len(lens), cfg["window"], max(max(p) for p in lens) + n
    w = workload.make_weights(arch, cfg["seed"], 6.0, cfg["dtype"], std=0.08)
    rng = np.random.default_rng(5)
    cond = [rng.integers(0, arch["vocab"], c).astype(np.int32) for c, _ in lens]
    uncond = [rng.integers(0, arch["vocab"], u).astype(np.int32) for _, u in lens]
    o = oracle.Oracle(arch, w, L, max_ctx, top_k=cfg["top_k"], seed=3, max_seqs=S)
    g = sjd.Decoder(arch, gpu_weights(w, cfg["dtype"]), cfg["dtype"], L, max_ctx, max_seqs=S, top_k=cfg["top_k"], seed=3,
                    kernel_flags=flags | sjd.KEEP_LOGITS)
    assert o.prefill(cond, uncond, [n] * S) == 0
    for again in range(2):   # the second prefill of a context starts over
        assert g.prefill(cond, uncond, [n] * S) == 0
        les = [g.window(s)[2] for s in range(S)]
        g.step()
        if again == 0:
            want = o.peek_logits()
        worst = logits_error(g.logits(), want, les)
        print(name, lens, flags, "logits error abs/rel:", worst)
        assert worst[0] <= 1e-4 if cfg["dtype"] == "f32" else worst[1] <= 8e-2


@pytest.mark.parametrize("flags,forwards", [(0, 1), (8, 5)])
def test_chunked_attention_serves_the_prompts_too(flags, forwards):
    """SJD_ATTENTION_CHUNKED always splits the context over workgroups: with it, 79 prompt rows run as five windows of 16
    (every layer but the last attends), without it as one packed forward."""
    import paper_2512_07503_amd as sjd
    cfg = workload.get_config("small_fused64")
    w = workload.make_weights(cfg["arch"], cfg["seed"], 6.0, cfg["dtype"], std=0.08)
    ids = np.arange(80, dtype=np.int32)
    g = sjd.Decoder(cfg["arch"], gpu_weights(w, cfg["dtype"]), cfg["dtype"], 16, 120, kernel_flags=flags)
    g.trace(True)
    assert g.prefill([ids], [ids], [40]) == 0
    t = g.trace_read()
    assert t["embed"][0] == forwards and t["window_attention"][0] == forwards * (cfg["arch"]["n_layers"] - 1)


def _cache_rows(g, arch, pt, n_prompt):
    """Keys and values of every prompt position from a snapshot taken before the first step: per segment [layers][2][positions]
    [kv heads * hd].  The pages are the snapshot's tail, [layer][keys, values][segment][page of the segment], a page
    [kv heads][pt * hd] in the attention's operand layouts (csrc/common.hip.h, Layout<bf16_t>)."""
    hkv, hd, nl = arch["n_kv_heads"], arch["d_model"] // arch["n_heads"], arch["n_layers"]
    pages = [-(-n // pt) for n in n_prompt]
    raw = g.snapshot()
    blk = hkv * pt * hd
    vals = raw[raw.size - nl * 2 * sum(pages) * blk * 2:].copy().view(np.uint16).astype(np.uint32) << 16
    vals = vals.view(np.float32).reshape(nl, 2, sum(pages), hkv, pt * hd)
    t, j = np.arange(pt)[:, None], np.arange(hd)[None, :]
    k_idx = (((t >> 5) * (hd >> 4) + (j >> 4)) * 64 + (((j >> 3) & 1) << 5) + (t & 31)) * 8 + (j & 7)
    grp, e = ((t >> 2) & 1), ((t >> 3) & 1) * 4 + (t & 3)
    v_idx = ((((t >> 5) * 2 + ((t >> 4) & 1)) * (hd >> 5) + (j >> 5)) * 64 + (grp << 5) + (j & 31)) * 8 + e
    out, p0 = [], 0
    for n, np_ in zip(n_prompt, pages):
        seg = vals[:, :, p0:p0 + np_]
        kv = np.stack([seg[:, 0][..., k_idx], seg[:, 1][..., v_idx]], 1)       # [layers][2][pages][kv heads][pt][hd]
        kv = kv.transpose(0, 1, 2, 4, 3, 5).reshape(nl, 2, np_ * pt, hkv * hd)
        out.append(kv[:, :, :n])
        p0 += np_
    return out


@pytest.mark.parametrize("name,lens,flags", [
    ("small_fused64", [(33, 1), (1, 70), (32, 34)], 0),
    ("small_fused64", [(1500, 1300)], 0),                        # a branch cut between two forwards
    ("small_fused64", [(90, 80), (100, 60)], 8),                 # window by window
    ("small_fused128", [(257, 1), (129, 70), (31, 32)], 0),
    ("small_tile", [(400, 399), (127, 2), (258, 130)], 16),
])
def test_every_cached_position(name, lens, flags):
    """Keys and values of every prompt position, layer by layer, against the reference kernels' (which cut the prompts at 512
    rows).  A position that holds another's row differs by about sqrt(2) of its 2-norm, a missing one by 1.  Roundings of these
    wide-weight models move a logit by up to 6e-2 of its row's maximum, i.e. 0.2 of the rms at a maximum of 3 to 4 sigma: the
    2-norm of a row, a mean over its elements, stays below that."""
    import paper_2512_07503_amd as sjd
    cfg = workload.get_config(name)
    arch, n, pt = cfg["arch"], 40, 64
    S, L, max_ctx = len(lens), cfg["window"], max(max(p) for p in lens) + n
    w = gpu_weights(workload.make_weights(arch, cfg["seed"], 6.0, cfg["dtype"], std=0.08), cfg["dtype"])
    rng = np.random.default_rng(7)
    cond = [rng.integers(0, arch["vocab"], c).astype(np.int32) for c, _ in lens]
    uncond = [rng.integers(0, arch["vocab"], u).astype(np.int32) for _, u in lens]
    got = []
    for f in (flags, 1):
        g = sjd.Decoder(arch, w, cfg["dtype"], L, max_ctx, max_seqs=S, top_k=cfg["top_k"], seed=3, kernel_flags=f, kv_page_tokens=pt)
        assert g.prefill(cond, uncond, [n] * S) == 0
        got.append(_cache_rows(g, arch, pt, [x - 1 for p in lens for x in p]))
        g.close()
    worst = 0.0
    for a, b in zip(*got):
        if a.shape[2]:
            assert np.isfinite(a).all()
            size = np.linalg.norm(b, axis=-1)
            assert (size > 0).all()
            worst = max(worst, float((np.linalg.norm(a - b, axis=-1) / size).max()))
    print(name, lens, flags, "worst relative difference of a position's keys or values", worst)
    assert worst < 0.2


def test_neighbours_do_not_change_a_sequence():
    """Sequence 0 beside prompts of other lengths: fp32 sums keep their order whatever the rows of a forward, so its logits
    and tokens are the same bits; bf16 ones follow the number of rows and agree to rounding (8e-2, as above)."""
    import paper_2512_07503_amd as sjd
    for name in ("small_f32", "small_fused64"):
        cfg = workload.get_config(name)
        arch, L = cfg["arch"], cfg["window"]
        w = gpu_weights(workload.make_weights(arch, cfg["seed"], 6.0, cfg["dtype"], std=0.08), cfg["dtype"])
        rng = np.random.default_rng(9)
        mine = [rng.integers(0, arch["vocab"], 70).astype(np.int32) for _ in range(2)]
        runs = []
        for other in (3, 41, 600):
            mate = [rng.integers(0, arch["vocab"], other).astype(np.int32) for _ in range(2)]
            g = sjd.Decoder(arch, w, cfg["dtype"], L, 700, max_seqs=2, top_k=cfg["top_k"], seed=3, kernel_flags=sjd.KEEP_LOGITS)
            assert g.prefill([mine[0], mate[0]], [mine[1], mate[1]], [30, 30]) == 0
            g.step()
            logits = g.logits()[0]
            g.decode()
            runs.append((logits, g.tokens(0).copy()))
            g.close()
        for logits, tokens in runs[1:]:
            if cfg["dtype"] == "f32":
                assert np.array_equal(logits, runs[0][0]) and np.array_equal(tokens, runs[0][1])
            else:
                assert logits_error(logits[None], runs[0][0][None], [L])[1] <= 8e-2
