"""A context allocates what its path uses: device memory taken by sjd_create against the sum of the weights, the cache and
the buffers of one forward."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,ff,window,seqs", [(2048, 8192, 32, 1), (1024, 4096, 250, 2)])
def test_create_takes_no_more_than_its_path_uses(d, ff, window, seqs):
    import torch
    import paper_2512_07503_amd as sjd
    V, ctx, layers = 2048, 1200, 2
    heads = d // 128
    arch = dict(n_layers=layers, d_model=d, n_heads=heads, n_kv_heads=heads, d_ff=ff, vocab=V, sample_lo=0, sample_hi=V)

    def rnd(*s):
        return torch.randn(s, device="cuda", dtype=torch.bfloat16) * 0.02
    shapes = dict(wq=(d, d), wk=(d, d), wv=(d, d), wo=(d, d), w_gate=(ff, d), w_up=(ff, d), w_down=(d, ff), attn_norm=(d,), mlp_norm=(d,))
    w = {n: [rnd(*s) for _ in range(layers)] for n, s in shapes.items()}
    w.update(tok_emb=rnd(V, d), final_norm=rnd(d), lm_head=rnd(V, d))
    sjd.Decoder(arch, w, "bf16", window, ctx, max_seqs=seqs).close()   # first use: the library's code goes to the device
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    before = torch.cuda.mem_get_info()[0]
    g = sjd.Decoder(arch, w, "bf16", window, ctx, max_seqs=seqs)
    torch.cuda.synchronize()
    used = before - torch.cuda.mem_get_info()[0]
    rows = max(2048, 2 * seqs * window)                     # of a prefill forward or a step
    weights = 2 * V * d * 2 + layers * (4 * d * d + 3 * d * ff) * 2
    cache = 2 * layers * 2 * seqs * (ctx + 64) * d * 2
    forward = rows * (d * 4 + 3 * d * 2 + ff * 2 + 4 * d * 4)   # stream, its copy, queries, attention, MLP, four K splits of partial sums
    slots = 2 * seqs * heads * -(-window // 32) * -(-ctx // 128)   # chunked attention: at most this many partial results
    state = 2 * seqs * window * V * 4 * 2 + 4 * seqs * window * V * 4 + slots * 32 * (128 + 2) * 4   # logits, z, stored rows, ...
    need = weights + cache + forward + state
    g.close()
    print(d, ff, window, seqs, f"used {used / 2**20:.0f} MiB, needed {need / 2**20:.0f} MiB")
    assert used <= 1.05 * need + (24 << 20)   # allocation granularity: some 60 buffers
