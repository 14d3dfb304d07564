"""The fp32 / reference GEMM in its documented order of summation: lane l adds k = l, l + 64, ... with fused multiply-adds, then
lanes 32, 16, ..., 1 apart.  Bit for bit against that order in numpy (the fused multiply-add through float64, whose product
is exact; an emulated sum can differ by a double rounding, hence one unit in the last place of the largest partial sum)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _in_order(A, W):
    M, K = A.shape
    pad = -K % 64
    a = np.pad(A, ((0, 0), (0, pad))).astype(np.float64).reshape(M, 1, -1, 64)
    w = np.pad(W, ((0, 0), (0, pad))).astype(np.float64).reshape(1, W.shape[0], -1, 64)
    s = np.zeros((M, W.shape[0], 64), np.float32)
    for i in range(a.shape[2]):
        s = (a[:, :, i] * w[:, :, i] + s).astype(np.float32)
    off = 32
    while off:
        s = s[..., :off] + s[..., off:2 * off]
        off //= 2
    return s[..., 0]


# one column per wavefront below 6144 columns x row blocks, four from there on; odd K, rows and columns past the last block
@pytest.mark.parametrize("M,N,K", [(1, 1, 1), (7, 5, 63), (9, 767, 70), (32, 1535, 256), (32, 1536, 256), (8, 6143, 65), (8, 6145, 320), (17, 2050, 519)])
def test_order_of_summation(M, N, K):
    import torch
    import paper_2512_07503_amd as sjd
    rng = np.random.default_rng(M + N + K)
    A, W = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((N, K)).astype(np.float32)
    out = sjd.op_gemm(torch.from_numpy(A).cuda(), torch.from_numpy(W).cuda())
    got = (out[0] if isinstance(out, tuple) else out).cpu().numpy()
    want = _in_order(A, W)
    bound = 2.0 ** -23 * np.maximum(1.0, np.abs(A) @ np.abs(W).T)
    assert (np.abs(got - want) <= bound).all() and (got == want).mean() > 0.99
