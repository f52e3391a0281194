"""The activation test of the prompt tracking at the very edge: alpha is one of the exported weights, or a float
beside it, over the whole range of weights and close to 1, where one weight belongs to many logits.  The state
follows from `exported weight >= alpha` without a tolerance."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _inputs(dt, S, H, G, P, d, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    k = torch.empty((S, H, P, d), device="cuda").normal_(generator=gen)
    k /= k.norm(dim=-1, keepdim=True)
    q = torch.empty((S, P, H, G, d), device="cuda").normal_(generator=gen) * 0.2
    # every query is close to one earlier key, with a strength that leaves weights from 1/2 up to 1 exactly
    which = torch.rand((S, P, H, G), device="cuda", generator=gen) * torch.arange(1, P + 1, device="cuda").view(1, P, 1, 1)
    which = which.long().clamp_max(P - 1)
    hit = torch.stack([k[s][torch.arange(H, device="cuda").view(1, H, 1), which[s]] for s in range(S)])   # [S,P,H,G,d]
    strength = d ** 0.5 * (2.0 + 26.0 * torch.rand((S, P, H, G, 1), device="cuda", generator=gen))
    return k.to(dt), (q + strength * hit).view(S, P, H * G, d).to(dt)


def _track(lazyev_lib, dt, k, q, alpha, export):
    S, H, P, d = k.shape
    eng = lazyev_lib.LazyEviction(1, S, q.shape[2], H, d, P + 40, 8, P, alpha, dtype=dt)
    eng.k_cache[0, :, :, :P].copy_(k)
    eng.init()
    p = torch.zeros((S, q.shape[2], P, P), device="cuda") if export else None
    eng.prefill_track(0, q, p_out=p)
    res = eng.ts[0, :, :, :P].clone(), eng.mri[0, :, :, :P].clone(), eng.stats()["n_activations"][0]
    eng.close()
    return res, p


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("S,H,G,P", [(2, 2, 2, 50), (1, 2, 1, 150), (16, 4, 8, 70)])
def test_threshold_is_met_exactly(lazyev_lib, dtype, d, S, H, G, P):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    k, q = _inputs(dt, S, H, G, P, d, P + d)
    _, p = _track(lazyev_lib, dt, k, q, 0.5, True)
    lower = torch.ones((P, P), dtype=torch.bool, device="cuda").tril()
    seen = np.unique(p[:, :, lower].cpu().numpy())
    picks = [seen[np.searchsorted(seen, x).clip(0, len(seen) - 1)] for x in (1e-6, 0.02, 0.3, 0.5, 0.9, 0.99, 0.996, 0.999, 0.9999, 0.999999)]
    alphas = {np.float32(1.0), np.nextafter(np.float32(1.0), np.float32(0.0))}
    for x in picks:
        alphas |= {x, np.nextafter(x, np.float32(2.0))}
    tau = torch.arange(1 - P, 1, dtype=torch.int32, device="cuda")
    for alpha in sorted(alphas):
        active = (p.view(S, H, G, P, P) >= float(alpha)).any(2) & lower
        ts = tau.expand(S, H, P).clone()
        mri = torch.zeros_like(ts)
        for i in range(P):
            on = active[:, :, i]
            mri = torch.where(on, torch.maximum(mri, tau[i] - ts), mri)
            ts = torch.where(on, tau[i], ts)
        for export in (True, False):
            (got_ts, got_mri, got_n), _ = _track(lazyev_lib, dt, k, q, float(alpha), export)
            assert got_n == int(active.sum()), (alpha, export)
            assert torch.equal(got_ts, ts) and torch.equal(got_mri, mri), (alpha, export)
