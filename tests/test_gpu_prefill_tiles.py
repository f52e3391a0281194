"""Tracking over the prompt at the edges of its tiles, stages and segments, for every row type and group: the
state the library leaves (wide or narrow tiles, one launch or segments that are joined) against the one that
follows from the weights it exports (Alg. 1 and Eq. 1, no tolerance), and these against weights in
64 bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = [("bf16", 128), ("bf16", 64), ("fp32", 64), ("fp32", 128)]
# (sequences, KV heads, group, positions): of up to three query tiles in one segment and cut; many narrow blocks of few tiles;
# the last eight are shapes of the wide tiles (the first two of them not in all kernels and types), with and without segments
SHAPES = [(1, 1, 1, 1), (1, 1, 2, 15), (2, 1, 3, 16), (1, 2, 5, 17), (1, 1, 7, 63), (1, 1, 4, 64), (1, 1, 8, 65),
          (2, 2, 4, 255), (1, 1, 6, 257), (1, 1, 8, 2100),
          (1, 2, 1, 47), (2, 2, 3, 40), (3, 2, 8, 33), (64, 2, 8, 34), (40, 8, 7, 20), (64, 3, 1, 164), (64, 1, 3, 170),
          (32, 8, 4, 200), (16, 8, 2, 330), (48, 2, 1, 400),
          (64, 8, 1, 70), (16, 4, 8, 300), (8, 4, 7, 513), (64, 2, 3, 129), (128, 16, 1, 33)]


@pytest.mark.parametrize("dtype,d", ROWS)
@pytest.mark.parametrize("S,H,G,P", SHAPES)
def test_prompt_tiles(lazyev_lib, dtype, d, S, H, G, P):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(P * G + d)
    k = torch.empty((S, H, P, d), device="cuda").normal_(generator=gen).to(dt)
    q = (1.5 * torch.empty((S, P, H * G, d), device="cuda").normal_(generator=gen)).to(dt)
    for alpha in (min(0.3, 8.0 / P),) + ((0.0, 2.0) if S * P < 600 else ()):
        runs = []
        for export in (True, False):
            eng = lazyev_lib.LazyEviction(1, S, H * G, H, d, P + 40, 8, P, alpha, dtype=dt)
            eng.k_cache[0, :, :, :P].copy_(k)
            eng.init()
            p = torch.zeros((S, H * G, P, P), device="cuda") if export else None
            eng.prefill_track(0, q, p_out=p)
            runs.append((eng.ts[0, :, :, :P].clone(), eng.mri[0, :, :, :P].clone(), eng.stats()["n_activations"][0]))
            eng.close()
            if export:
                weights = p
        active = (weights.view(S, H, G, P, P) >= alpha).any(2)              # [S, H, query, key]
        active &= torch.ones((P, P), dtype=torch.bool, device="cuda").tril()
        ts = torch.arange(1 - P, 1, dtype=torch.int32, device="cuda").expand(S, H, P).clone()
        mri = torch.zeros_like(ts)
        for i in range(P):
            on, tau = active[:, :, i], i + 1 - P
            mri = torch.where(on, torch.maximum(mri, tau - ts), mri)
            ts = torch.where(on, torch.full_like(ts, tau), ts)
        for got in runs:
            assert torch.equal(got[0], ts) and torch.equal(got[1], mri)
            assert got[2] == int(active.sum())
    # the logits are fp32 sums of d products of about 80 in magnitude together (scaled: 10); each of the d
    # additions is off by 2^-24 of it at most, and a weight by the sum of its logit's error, the
    # log-sum-exp's and one of an exponential: 2 d 2^-24 10 in proportion
    s, pair = 0, (H - 1) * G
    logits = q[s, :, pair:pair + G].double().transpose(0, 1) @ k[s, H - 1].double().T * d ** -0.5
    logits.masked_fill_(~torch.ones((P, P), dtype=torch.bool, device="cuda").tril(), float("-inf"))
    want = torch.softmax(logits, -1)
    got = weights[s, pair:pair + G].double()
    assert float(((got - want).abs() / want.clamp_min(1e-30)).tril().max()) <= 2 * d * 2.0 ** -24 * 10
