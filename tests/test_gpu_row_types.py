"""The single-launch kernel on fp32 rows and on rows of 64 elements, and candidate lists with groups
of eight heads, against the split + merge kernels (variant 0), which take every shape: outputs, TS /
MRI / pos and the caches after decode steps, with an eviction, across the sizes at which the split, the
sub-tile pipeline and the segments of a long run change."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(lazyev_lib, variant, dtype, d, H, group, batch, N, steps, budget, window, blocks=0, alpha=None):
    gen = torch.Generator(device="cuda").manual_seed(N + 10 * group)
    eng = lazyev_lib.LazyEviction(2, batch, group * H, H, d, budget, window, N, alpha or 8.0 / max(N, 16), dtype=dtype)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    eng.set_variant(variant)
    if blocks:
        eng.set_target_blocks(blocks * batch * H)
    out = torch.zeros((steps, 2, batch, group * H, d), dtype=dtype, device="cuda")
    for t in range(1, steps + 1):
        for l in range(2):
            q, kn, vn = (torch.empty((batch, h, d), device="cuda").normal_(generator=gen) for h in (group * H, H, H))
            if N > 8:                              # one head in three reads an entry again
                q[:, ::3] += 4.0 * eng.k_cache[l, :, :1, N // 2].float()
            eng.decode_step(l, t, q.to(dtype), kn.to(dtype), vn.to(dtype), out[t - 1, l])
        eng.evict_all(t)
    st = eng.stats()
    n = st["len"][0]
    state = [x[:, :, :, :n].clone() for x in (eng.ts, eng.mri, eng.pos, eng.k_cache, eng.v_cache)]
    eng.close()
    return out, state, st


def _compare(a, b, dtype):
    (out_a, state_a, st_a), (out_b, state_b, st_b) = a, b
    x, y = out_a.double(), out_b.double()
    err = float(((x - y).norm(dim=-1) / y.norm(dim=-1)).max())
    # fp32: sums of up to some thousand terms in two orders (about 1e-6 at most); bf16: results of two fp32 sums,
    # rounded once each (2^-9 of an element, at most)
    assert err < (1e-5 if dtype == torch.float32 else 2.0 ** -8), err
    for p, q in zip(state_a, state_b):
        assert torch.equal(p, q)
    assert st_a == st_b


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128), ("bf16", 64)])
@pytest.mark.parametrize("group,N", [(1, 3), (2, 15), (3, 16), (8, 62), (7, 129), (8, 700), (5, 2100), (4, 5500)])
def test_row_types_against_the_general_kernels(lazyev_lib, dtype, d, group, N):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    budget, window = max(N - 2, 6), 5
    runs = [_run(lazyev_lib, v, dt, d, 2, group, 2, N, 11, budget, window) for v in (0, 1)]
    _compare(*runs, dt)
    assert runs[0][2]["n_evict_events"] == [2, 2] or N < 8


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128), ("bf16", 64)])
@pytest.mark.parametrize("blocks", [1, 2, 3, 8, 9, 33])
def test_row_types_with_every_kind_of_split(lazyev_lib, dtype, d, blocks):
    """One, several and merged blocks per unit; a single block streams a long run."""
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    runs = [_run(lazyev_lib, v, dt, d, 1, 8, 2, 2300, 4, 4000, 64, blocks=b) for v, b in ((0, 0), (1, blocks))]
    _compare(*runs, dt)


@pytest.mark.parametrize("batch", [36, 70])
def test_row_types_without_list_waves(lazyev_lib, batch):
    """More units than the chip holds blocks with list waves for."""
    runs = [_run(lazyev_lib, v, torch.bfloat16, 64, 4, 8, batch, 400, 3, 4000, 64) for v in (0, 1)]
    _compare(*runs, torch.bfloat16)


@pytest.mark.parametrize("alpha", [1e-30, 2.0])
def test_groups_of_eight_with_every_and_with_no_candidate(lazyev_lib, alpha):
    """Candidate records fill their regions completely, or hold the appended entry alone."""
    for dtype, d in ((torch.bfloat16, 64), (torch.bfloat16, 128), (torch.float32, 128)):
        a, b = (_run(lazyev_lib, v, dtype, d, 2, 8, 2, 333, 9, 320, 4, alpha=alpha) for v in (0, 1))
        for p, q in zip(a[1], b[1]):
            assert torch.equal(p, q)
        assert a[2] == b[2]
