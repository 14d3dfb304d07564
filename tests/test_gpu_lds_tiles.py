"""Projections through LDS tiles (more than 64 rows): every tile shape and epilogue against the reference kernels on the same
device, at row counts that end inside tiles.  Which shape a projection takes depends on the model's width and the rows; the
cases below reach all of them.  Two layers; both sides round GEMM operands to bf16 at different places (the reference kernels
after the normalisation): a difference of 2^-9 a rounding, some ten roundings a layer on independent errors, a factor of three
for the spread -> 3e-2 in the 2-norm of the logits."""
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
        return torch.randn(s, generator=g, device="cuda", dtype=torch.bfloat16) * 0.02
    shapes = dict(wq=(q, d), wk=(kv, d), wv=(kv, d), wo=(d, q), w_gate=(ff, d), w_up=(ff, d), w_down=(d, ff))
    w = {n: [rnd(*s) for _ in range(arch["n_layers"])] for n, s in shapes.items()}
    for n in ("attn_norm", "mlp_norm"):
        w[n] = [1 + 4 * rnd(d) for _ in range(arch["n_layers"])]
    w.update(tok_emb=rnd(arch["vocab"], d), final_norm=1 + 4 * rnd(d), lm_head=rnd(arch["vocab"], d))
    return w


@pytest.mark.parametrize("d,heads,kv,ff,window,lens", [
    (1280, 20, 20, 3456, 48, [(60, 61)]),                      # 96 rows of a step
    (1280, 20, 20, 3456, 250, [(117, 3)]),                     # 500 rows; prompts of 118
    (1280, 20, 20, 3456, 16, [(120, 96), (40, 41), (77, 130), (99, 100), (140, 111), (2, 1)]),   # 192; 945 packed
    (1280, 20, 20, 3456, 1, [(700, 702)]),                     # 1400
    (2048, 16, 16, 5632, 65, [(120, 141)]),                    # 130; 259
    (2048, 16, 8, 5632, 32, [(200, 210), (280, 313)]),         # 128, guidance inside the head; 999
    (3072, 24, 8, 8192, 33, [(170, 93)]),                      # 66 rows, 128-wide heads, 261
    (4096, 32, 32, 11008, 96, [(64, 64)]),                     # 192; 126
    (4096, 32, 8, 14336, 35, [(350, 352), (340, 358)]),        # 140; 1396
])
def test_against_the_reference_kernels(d, heads, kv, ff, window, lens):
    import torch
    import paper_2512_07503_amd as sjd
    arch = dict(n_layers=2, d_model=d, n_heads=heads, n_kv_heads=kv, d_ff=ff, vocab=3100, sample_lo=50, sample_hi=3051)
    w, n, S = _weights(arch, 11), 300, len(lens)
    max_ctx = max(max(p) for p in lens) + n
    rng = np.random.default_rng(2)
    cond = [rng.integers(0, 3100, c).astype(np.int32) for c, _ in lens]
    uncond = [rng.integers(0, 3100, u).astype(np.int32) for _, u in lens]
    out = []
    for flags in (0, 1, 2048):   # default, reference kernels, no guidance inside the head
        g = sjd.Decoder(arch, w, "bf16", window, max_ctx, max_seqs=S, top_k=200, seed=5, kernel_flags=flags | sjd.KEEP_LOGITS)
        assert g.prefill(cond, uncond, [n] * S) == 0
        g.step()
        out.append(g.logits().astype(np.float64))
    err = np.linalg.norm(out[0] - out[1]) / np.linalg.norm(out[1])
    print(d, window, lens, "relative difference of the logits", err, "largest", np.abs(out[0] - out[1]).max())
    assert np.isfinite(out[0]).all() and err < 3e-2
    assert np.abs(out[0] - out[2]).max() <= 1e-5 * np.abs(out[2]).max()   # another tile shape of the head: the same sums
