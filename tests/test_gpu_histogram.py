"""lazyev_mri_histogram against numpy: entries beside and on the edges of a block's span, few and many
bins, one layer and all of them, and per-sequence lengths."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _engine(lazyev_lib, L, S, H, P):
    eng = lazyev_lib.LazyEviction(L, S, H, H, 128, P + 16, 8, P, 0.01, dtype=torch.bfloat16).init()
    gen = torch.Generator(device="cuda").manual_seed(P)
    # most entries 0 or 1, some in every bin and some beyond the last
    m = torch.randint(0, 9000, eng.mri.shape, generator=gen, device="cuda", dtype=torch.int32)
    few = torch.rand(eng.mri.shape, generator=gen, device="cuda") < 0.7
    eng.mri.copy_(torch.where(few, m % 2, m))
    return eng


def _count(mri, n_bins):
    return np.bincount(np.minimum(mri.cpu().numpy().ravel(), n_bins - 1), minlength=n_bins).tolist()


@pytest.mark.parametrize("n_bins", [2, 3, 64, 8192])
@pytest.mark.parametrize("P", [1, 255, 2047, 2048, 2049, 5000])
def test_histogram_counts_every_entry_once(lazyev_lib, P, n_bins):
    eng = _engine(lazyev_lib, 3, 2, 3, P)
    for layer in (-1, 0, 2):
        want = eng.mri[..., :P] if layer < 0 else eng.mri[layer, ..., :P]
        assert eng.mri_histogram(layer, n_bins) == _count(want, n_bins)


def test_histogram_of_sequences_of_different_lengths(lazyev_lib):
    eng = _engine(lazyev_lib, 2, 4, 3, 4200)
    mri = eng.mri.clone()
    lens = [4200, 0, 2049, 7]
    for seq, n in enumerate(lens):
        eng.retire(seq)
        if n:
            eng.admit(seq, n, 0)
    eng.mri.copy_(mri)                             # (admission starts a sequence at MRI = 0)
    want = torch.cat([mri[:, s, :, :n].reshape(-1) for s, n in enumerate(lens)])
    assert eng.mri_histogram(-1, 64) == _count(want, 64)
