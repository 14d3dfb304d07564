"""The decoding work that the performance of this package is measured on.

A pass is what a serving program does for a new request: `Decoder.prefill` on the prompts, then `Decoder.step`, on a
context whose weights were laid out once.  Passes over a real image repeat the step a few hundred to a few thousand times;
here the bf16 passes end after the first step, because that is the last point at which two correct bf16 implementations
can be compared at all: its window (last prompt token + uniform drafts) follows from the seed alone, so its logits agree to
rounding, while every later window depends on draws that a rounding in the last place may move to the next token id.  Cases
that stand for decoding proper therefore have the shortest prompt there is (one start token: prefill runs no forward), cases
with a text prompt weigh the prefill as well.  The fp32 passes run many steps and return the tokens.

Shapes are this repository's benchmark configurations (workload/configs.py); the wide ones at a reduced depth (every layer
costs the same) so that a model is drawn and laid out in a second.  Windows are the paper's: 1 (plain autoregressive
decoding), 16, 32, 96 and 250.
"""
import ctypes
import math

import numpy as np
import torch

import paper_2512_07503_amd as sjd

# name: layers, d_model, heads, kv heads, MLP hidden, vocabulary, first sampled id, sampled ids, dtype
TINY = dict(layers=2, d=256, heads=4, kv_heads=4, ff=1024, vocab=4096, lo=0, sampled=4096, f32=True)
XL = dict(layers=36, d=1280, heads=20, kv_heads=20, ff=3456, vocab=16384, lo=0, sampled=16384, f32=False)
WIDE = dict(layers=8, d=4096, heads=32, kv_heads=32, ff=11008, vocab=65536, lo=0, sampled=65536, f32=False)
GQA = dict(layers=8, d=4096, heads=32, kv_heads=8, ff=14336, vocab=184622, lo=151854, sampled=32768, f32=False)


def _case(shape, window, prompts, steps=1, seqs=1, top_k=2000, tau=0.5, n_image=576, init_mode=0, spread=0):
    """prompts: prompt tokens of the longest sequence; spread: how much shorter the shortest one is."""
    return dict(shape, window=window, prompt=prompts, spread=spread, steps=steps, seqs=seqs, top_k=top_k, tau=tau, n_image=n_image,
                init_mode=init_mode)


def listed():
    return [
        # the tiny fp32 model: launch latency, many small steps; tokens must come out the same
        dict(_case(TINY, 16, 32, steps=12, top_k=256, n_image=256), name="tiny_fp32"),
        # class-conditional generation (one conditioning token) on the 36-layer narrow model: one step of a 16-token window,
        # the smallest bf16 call, and the same model after a text prompt with the window used for it in the paper
        dict(_case(XL, 16, 1, top_k=1000), name="narrow_step_w16"),
        dict(_case(XL, 32, 120, top_k=1000), name="narrow_text_w32"),
        # the paper's longest window (24 x 24 token images), which is 500 rows: not a multiple of any tile
        dict(_case(XL, 250, 60, top_k=1000), name="narrow_text_w250"),
        # several users' prompts of different lengths decoded together with a short window (192 rows)
        dict(_case(XL, 16, 120, seqs=6, spread=80, top_k=1000), name="narrow_batch6_w16"),
        # the autoregressive baseline: window 1, text prompt
        dict(_case(XL, 1, 120, top_k=1000), name="narrow_ar"),
        # the 7B shape: one decoding step; a text prompt with the paper's window of 96
        dict(_case(WIDE, 32, 1, n_image=2352), name="wide_step_w32"),
        dict(_case(WIDE, 96, 64, n_image=2352), name="wide_text_w96"),
        # grouped-query attention, a sampled sub-range of the vocabulary, SJD without reuse
        dict(_case(GQA, 32, 64, top_k=2048, tau=1e30, n_image=4096), name="gqa_text_w32"),
        # an image in the prompt (editing, interleaved models): 2 000 tokens of context, then a step over them
        dict(_case(GQA, 32, 2000, top_k=2048, n_image=4096), name="gqa_long_w32"),
        # throughput: eight prompts of different lengths together, and their autoregressive baseline
        dict(_case(WIDE, 32, 64, seqs=8, spread=45, n_image=2352), name="wide_batch8_w32"),
        dict(_case(WIDE, 1, 24, seqs=8, spread=13, n_image=2352), name="wide_batch8_ar"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: model widths, depths, windows, batches, prompts and sampling options over the range of the listed ones."""
    kind = rng.choice(("f32", "narrow", "narrow", "wide", "wide"))
    if kind == "f32":
        hd = rng.choice((32, 64))
        heads = rng.randint(2, 8)
        sampled = rng.randint(600, 6000)
        shape = dict(layers=rng.randint(1, 3), d=hd * heads, heads=heads, kv_heads=heads, ff=16 * rng.randint(12, 90), vocab=sampled + 100,
                     lo=rng.choice((0, 100)), sampled=sampled, f32=True)
        return _case(shape, rng.randint(1, 24), _log_int(rng, 1, 60), steps=rng.randint(2, 12), seqs=rng.randint(1, 3),
                     top_k=_log_int(rng, 1, 500), tau=rng.choice((0.5, 0.5, 1e30)), n_image=320, init_mode=rng.choice((0, 0, 1, 2)))
    hd = 64 if kind == "narrow" else 128
    kv = rng.choice((2, 4, 5, 8)) if kind == "narrow" else rng.choice((4, 8))
    group = rng.choice((1, 2, 4))
    heads = kv * group
    lo_heads, hi_heads = (8, 24) if kind == "narrow" else (16, 40)
    heads = max(1, min(hi_heads // kv, max(-(-lo_heads // kv), group))) * kv
    kv = heads if rng.random() < 0.5 else max(kv, heads // 4)
    while heads % kv:
        kv += 1
    d = hd * heads
    sampled = rng.randint(8192, 20000) if kind == "narrow" else rng.randint(16384, 65536)
    lo = rng.choice((0, 0, 4000))
    shape = dict(layers=rng.randint(6, 36) if kind == "narrow" else rng.randint(3, 8), d=d, heads=heads, kv_heads=kv,
                 ff=32 * int(d * rng.uniform(2.5, 3.6) / 32), vocab=lo + sampled + rng.randint(0, 2000), lo=lo, sampled=sampled, f32=False)
    window = rng.choice((1, 16, 32, 32, 96, _log_int(rng, 1, 256), _log_int(rng, 1, 256)))
    rows = 1024 if kind == "narrow" else 512
    seqs = rng.choice((1, 1, 1, 2, rng.randint(2, 8)))
    seqs = max(1, min(seqs, rows // (2 * window)))
    prompt = _log_int(rng, 1, max(8, min(2000 if seqs == 1 else 400, 64 * window)))
    return _case(shape, window, prompt, seqs=seqs, spread=rng.randint(0, prompt - 1), top_k=_log_int(rng, 1, 2500),
                 tau=rng.choice((0.5, 0.5, 0.5, 1e30, 0.0)), n_image=rng.randint(600, 1500), init_mode=rng.choice((0, 0, 0, 1, 2, 3, 4)))


def _matrices(c):
    """Elements of the linear layers of one block."""
    hd = c["d"] // c["heads"]
    return c["d"] * (c["heads"] + 2 * c["kv_heads"]) * hd + c["heads"] * hd * c["d"] + 3 * c["d"] * c["ff"]


def _lengths(c):
    """Prompt tokens of every sequence (the same for its two guidance branches)."""
    n = c["seqs"]
    return [c["prompt"] - (c["spread"] * s // (n - 1) if n > 1 else 0) for s in range(n)]


def prepare(case, seed):
    c = case
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dtype = torch.float32 if c["f32"] else torch.bfloat16
    d, ff, hd = c["d"], c["ff"], c["d"] // c["heads"]

    def normal(rows, cols, std=0.02):
        return torch.randn((rows, cols), generator=g, device="cuda", dtype=dtype) * std

    def ones():
        return torch.ones(d, device="cuda", dtype=dtype)

    # random-init weights N(0, 0.02); the head is scaled so that the sampled distribution has an entropy of about 4 nats
    # (0.31 of the closed form for independent Gaussian logits: the guidance weight of 3 spreads them by the rest)
    alpha = 0.31 * math.sqrt(2.0 * max(math.log(c["sampled"]) - 4.0, 0.05)) / (0.02 * math.sqrt(d))
    w = {n: [] for n in ("attn_norm", "wq", "wk", "wv", "wo", "mlp_norm", "w_gate", "w_up", "w_down")}
    w["tok_emb"] = normal(c["vocab"], d)
    w["final_norm"] = ones()
    w["lm_head"] = normal(c["vocab"], d, 0.02 * alpha)
    shapes = dict(wq=(c["heads"] * hd, d), wk=(c["kv_heads"] * hd, d), wv=(c["kv_heads"] * hd, d), wo=(d, c["heads"] * hd), w_gate=(ff, d),
                  w_up=(ff, d), w_down=(d, ff))
    for _ in range(c["layers"]):
        w["attn_norm"].append(ones())
        w["mlp_norm"].append(ones())
        for n, s in shapes.items():
            w[n].append(normal(*s))
    arch = dict(n_layers=c["layers"], d_model=d, n_heads=c["heads"], n_kv_heads=c["kv_heads"], d_ff=ff, vocab=c["vocab"],
                sample_lo=c["lo"], sample_hi=c["lo"] + c["sampled"])
    dec = sjd.Decoder(arch, w, "f32" if c["f32"] else "bf16", c["window"], c["prompt"] + c["n_image"], max_seqs=c["seqs"], top_k=c["top_k"],
                      reuse_tau=c["tau"], seed=seed, kernel_flags=sjd.KEEP_LOGITS, init_mode=c["init_mode"],
                      row_width=24 if c["init_mode"] else 0)
    cond, uncond = [], []
    for n in _lengths(c):
        ids = torch.randint(0, c["vocab"], (2, n), generator=g, device="cuda", dtype=torch.int32).cpu().numpy()
        ids[1, -1] = ids[0, -1]   # both branches end in the start-of-image marker
        cond.append(ids[0].copy())
        uncond.append(ids[1].copy())
    logits = torch.empty((c["seqs"], 2, c["window"], c["sampled"]), dtype=torch.float32, pin_memory=True)
    return dict(case=c, dec=dec, cond=cond, uncond=uncond, logits=logits)


def run(state):
    c, dec, logits = state["case"], state["dec"], state["logits"]
    rc = dec.prefill(state["cond"], state["uncond"], [c["n_image"]] * c["seqs"])
    if rc != sjd.OK:
        raise sjd.SjdError(rc, "prefill")
    for _ in range(c["steps"]):
        dec.step()
    rc = sjd.lib().sjd_debug_copy_logits(dec.ctx, ctypes.cast(logits.data_ptr(), ctypes.POINTER(ctypes.c_float)))
    if rc != sjd.OK:
        raise sjd.SjdError(rc, "logits")
    if not c["f32"]:
        return {"logits": logits}
    image = np.full((c["seqs"], c["n_image"]), -1, dtype=np.int32)   # -1: not decided yet
    for s in range(c["seqs"]):
        tokens = dec.tokens(s)
        image[s, :len(tokens)] = tokens
    return {"logits": logits, "image": image, "window": [dec.window(s)[0] for s in range(c["seqs"])]}


def work(case):
    c = case
    size = 4 if c["f32"] else 2
    hd = c["d"] // c["heads"]
    layer, head = _matrices(c), c["d"] * c["sampled"]
    kv = 2 * 2 * c["kv_heads"] * hd * c["layers"] * size    # keys and values of one position, both branches, all layers
    rows = 2 * c["window"] * c["seqs"]
    lengths = [n - 1 for n in _lengths(c)]                  # prompt positions that the prefill runs
    prefill_rows = 2 * sum(lengths)
    flops = 2.0 * layer * c["layers"] * prefill_rows + c["steps"] * 2.0 * (layer * c["layers"] + head) * rows
    flops += 4.0 * c["heads"] * hd * c["layers"] * 2 * sum(n * n / 2 + c["steps"] * c["window"] * (n + c["window"] / 2) for n in lengths)
    bytes_ = size * (layer * c["layers"] * ((1 if prefill_rows else 0) + c["steps"]) + head * c["steps"])
    bytes_ += kv * sum(n + c["steps"] * (n + c["window"]) for n in lengths)
    bytes_ += (prefill_rows + c["steps"] * rows) * c["d"] * size + rows * c["sampled"] * 4
    return dict(bytes=bytes_, flops=flops)


def tolerance(case):
    # fp32: sums in another order; the tokens are integer-arithmetic functions of the logits.
    # bf16: every operand of a matrix product is rounded to bf16, and a sum in another order flips some of those roundings;
    # the error grows with the square root of the depth.  Measured between this package's own kernel sets on these cases:
    # summation order alone 0.007 (36 narrow layers) to 0.0135 (8 wide layers), fused against reference kernels (which round
    # after the normalisation instead of before it) 0.007 - 0.012 and 0.021 - 0.025; largest difference 0.03 - 0.15 of the
    # root mean square.
    if case["f32"]:
        return dict(rel=1e-5, max=1e-3, differ=0.0)
    return dict(rel=0.03, max=0.6)
