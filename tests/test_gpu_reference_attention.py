"""The attention of models whose heads no MFMA kernel takes (five query heads to a key/value head, heads 32 wide) and of fp32 models is one
wavefront per (row, head): at the rows of a prompt it lives from how many wavefronts a CU holds."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd", [64, 128])
def test_half_the_bytes_take_no_longer(hd):
    """bf16 keys and values through the same kernel as fp32 ones: 0.42 of the time while registers leave a CU its wavefronts, 1.7 times with
    the 64 dimensions of a key and 32 tokens' values in flight that once brought it down to two wavefronts a SIMD."""
    import torch
    import paper_2512_07503_amd as sjd
    n, H, ctx, ms = 500, 40, 300, {}
    g = torch.Generator(device="cuda")
    g.manual_seed(hd)
    q, k, v = (torch.randn((r, H, hd), generator=g, device="cuda") for r in (n, ctx + n, ctx + n))
    for dtype in (torch.float32, torch.bfloat16):
        x = [t.to(dtype) for t in (q, k, v)]
        ms[dtype] = min(sjd.op_window_attention(*x, ctx, flags=sjd.KERNELS_REFERENCE, repeat=10)[1] for _ in range(3))
    assert ms[torch.bfloat16] < ms[torch.float32], ms
