"""Sampling rows of many ids: the kept ones are looked for among the keys above a sampled bound, where that holds K of them and
few enough, else among all.  Rows on both sides of either condition, against the oracle, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _rows(V, K, rng):
    n = rng.standard_normal((9, V)) * 3
    n[1] = np.sort(n[1])                                    # the sample sees every part of it all the same
    n[2] = 0.25                                             # one value: everything ties, nothing fits
    n[3] = np.round(n[3])                                   # a handful of values
    n[4, rng.permutation(V)[: V - K]] = -1e30               # K values and a floor far below
    n[5, rng.permutation(V)[: max(1, K - 1)]] += 1e4        # K - 1 outliers: the K-th is one of the bulk
    n[6] *= 1e-6                                            # keys of a few bins
    n[7] = np.where(np.arange(V) < 7000, 5.0, n[7])         # more ties at the top than the candidates' room
    n[8] = -np.abs(n[8])                                    # nothing above 0
    return n.astype(np.float32)


@pytest.mark.parametrize("V,K", [(16384, 1), (16384, 1000), (16384, 2600), (4097, 500), (16385, 700), (20000, 3000), (32768, 2048),
                                 (32769, 100), (65535, 6000), (65536, 2000), (65536, 10400),
                                 (17000, 2000), (33000, 2000), (50000, 2500), (20000, 2400)])   # (of up to 16384 ids: never candidates)
def test_rows_on_both_sides_of_the_candidates_conditions(oracle, V, K):
    import torch
    import paper_2512_07503_amd as sjd
    rng = np.random.default_rng(V + K)
    lc, lu = _rows(V, K, rng), _rows(V, K, rng)
    lu[4] = lc[4]
    lu[7] = lc[7]
    e, Z, _, ids, cnt = sjd.op_sampling_rows(torch.from_numpy(lc).cuda(), torch.from_numpy(lu).cuda(), 3.0, 1.0, K, kept=True)
    e, Z, ids, cnt = e.cpu().numpy(), Z.cpu().numpy().view(np.uint64), ids.cpu().numpy(), cnt.cpu().numpy()
    for r in range(len(lc)):
        e_ref, Z_ref = oracle.sampling_row(lc[r], lu[r], 3.0, 1.0, K)
        assert np.array_equal(e[r].view(np.uint32), e_ref.view(np.uint32)), r
        assert int(Z[r]) == Z_ref, r
        kept = ids[r, : cnt[r]]
        assert K <= cnt[r] <= V and (np.diff(kept) > 0).all() and kept[0] >= 0 and kept[-1] < V
        assert np.isin(np.flatnonzero(e_ref), kept).all()
