"""The fp32 projections with norm, rotation, SwiGLU and residual inside (kernels_f32.hip.h) against the separate kernels whose
sums they keep: same logits, same tokens, bit for bit.  tests/test_plan_bounds.py holds the last three cases to the sides of
f32_inside (plans.h) that they are there for."""
import numpy as np
import pytest

import workload
from helpers import gpu_weights

pytestmark = pytest.mark.gpu


CASES = [
    # widths of less than a norm's 256 strided threads, of them exactly, and past them with a remainder; odd pair counts
    (dict(n_layers=1, d_model=6, n_heads=1, n_kv_heads=1, d_ff=5, vocab=40), 2, 1, 4),
    (dict(n_layers=2, d_model=60, n_heads=6, n_kv_heads=3, d_ff=77, vocab=300), 3, 2, 9),
    (dict(n_layers=2, d_model=255 * 2, n_heads=5, n_kv_heads=5, d_ff=333, vocab=1001), 1, 1, 30),
    (dict(n_layers=1, d_model=256, n_heads=4, n_kv_heads=2, d_ff=1024, vocab=4096), 16, 1, 33),
    (dict(n_layers=2, d_model=328, n_heads=4, n_kv_heads=4, d_ff=65, vocab=777), 24, 3, 70),    # four columns a wavefront
    # some of QKV, gate/up and head with their element-wise steps inside, others with them apart
    (dict(n_layers=2, d_model=256, n_heads=4, n_kv_heads=2, d_ff=1600, vocab=3000), 40, 2, 61),
    (dict(n_layers=2, d_model=256, n_heads=4, n_kv_heads=4, d_ff=200, vocab=3000), 1, 1, 240),
    (dict(n_layers=2, d_model=512, n_heads=8, n_kv_heads=8, d_ff=1440, vocab=900), 100, 2, 30),
]


@pytest.mark.parametrize("arch,window,seqs,prompt", CASES)
def test_same_bits_as_the_separate_kernels(arch, window, seqs, prompt):
    import paper_2512_07503_amd as sjd
    arch = dict(arch, sample_lo=1, sample_hi=arch["vocab"])
    w = gpu_weights(workload.make_weights(arch, 3, 6.0, "f32", std=0.08, random_gains=True), "f32")
    cond, uncond = workload.make_prompts(arch, 3, seqs, prompt)
    n_img = [window + 30 + s for s in range(seqs)]
    fused, plain = (sjd.Decoder(arch, w, "f32", window, prompt + max(n_img), max_seqs=seqs, top_k=30, seed=5, kernel_flags=sjd.KEEP_LOGITS | f)
                    for f in (0, sjd.KERNELS_REFERENCE))
    assert fused.prefill(cond, uncond, n_img) == 0 and plain.prefill(cond, uncond, n_img) == 0
    for _ in range(4):
        assert fused.step() == plain.step()
        got, want = fused.logits(), plain.logits()
        assert np.isfinite(want).all() and np.array_equal(got.view(np.uint32), want.view(np.uint32))
    assert all(np.array_equal(fused.tokens(s), plain.tokens(s)) for s in range(seqs))
