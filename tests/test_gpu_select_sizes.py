"""The selection at the sizes where it changes (entries per thread 2, 3, 5, 8, then passes over memory; one entry
beside every edge), on hand-made states against the oracle's scoring and selection (Eq. 3, Eq. 6), no tolerance."""
import numpy as np
import pytest
import torch

from oracle.lazyev_oracle import mri_centric_score, select_survivors

pytestmark = pytest.mark.gpu

W, D, HKV = 3, 64, 6
T = W


def _patterns(rng, n):
    t = T
    half = np.arange(n) < n // 2
    return [(np.zeros(n, int), np.zeros(n, int)),                                        # all score 0
            (t - rng.permutation(n) - 1, np.full(n, n)),                                 # all distinct
            (t - rng.integers(0, 20000, n), rng.integers(0, 5000, n)),                   # random
            (t - rng.integers(1, 9, n), rng.integers(2000000, 2000000 + 2 * n, n)),      # distinct, all next to 2
            (np.where(half, t - 50, t - rng.integers(1, 40, n)), np.full(n, 50)),        # a tie group at the cut
            (t - rng.integers(0, 30, n), np.where(rng.random(n) < 0.9, 0, rng.integers(1, 900, n)))]   # mostly 0


@pytest.mark.parametrize("n", [20, 1023, 1024, 1025, 2047, 2048, 2049, 3072, 3073, 5120, 5121, 8191, 8192, 8193, 8196])
def test_selection_at_the_edges(lazyev_lib, n):
    rng = np.random.default_rng(n)
    B = n - W
    eng = lazyev_lib.LazyEviction(1, 1, HKV, HKV, D, B, W, B, alpha=2.0, dtype=torch.float32)
    eng.k_cache[0, 0, :, :B, :] = torch.arange(B, dtype=torch.float32, device="cuda").view(1, -1, 1)
    eng.v_cache.copy_(-eng.k_cache)
    eng.init()
    q = torch.zeros((1, HKV, D), device="cuda")
    out = torch.empty_like(q)
    for step in range(1, T + 1):                                 # nothing reaches alpha = 2
        kv = torch.full((1, HKV, D), float(B + step - 1), device="cuda")
        eng.decode_step(0, step, q, kv, -kv, out)
    assert eng.stats()["len"][0] == n
    pats = _patterns(rng, B)
    for h, (ts, mri) in enumerate(pats):
        eng.ts[0, 0, h, :B] = torch.from_numpy(ts.astype(np.int32)).cuda()
        eng.mri[0, 0, h, :B] = torch.from_numpy(mri.astype(np.int32)).cuda()
    assert eng.evict(0, T) == W
    moved = 0
    for h, (ts, mri) in enumerate(pats):
        keep = select_survivors(mri_centric_score(T, ts, mri, 3), B - W)
        want = np.concatenate([keep, np.arange(B, B + W)])
        assert np.array_equal(eng.pos[0, 0, h, :B].cpu().numpy(), want), h
        assert np.array_equal(eng.ts[0, 0, h, :B].cpu().numpy(), np.concatenate([ts[keep], np.arange(1, W + 1)]))
        assert np.array_equal(eng.mri[0, 0, h, :B].cpu().numpy(), np.concatenate([mri[keep], np.zeros(W, int)]))
        assert np.array_equal(eng.k_cache[0, 0, h, :B, 7].cpu().numpy(), want)
        moved += int((want != np.arange(B)).sum())
    assert eng.stats()["n_rows_moved"][0] == moved
