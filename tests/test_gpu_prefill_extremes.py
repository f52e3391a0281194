"""Tracking over the prompt with logits at the ends of the range: keys so large that a logit's rounding exceeds the
range of an exponential, keys whose logits are -inf for every query (the first 16, the first 40, scattered ones), infinite
and NaN elements.  Exported weights against softmax in 64 bits, and the state against the exported weights."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = [("bf16", 128), ("bf16", 64), ("fp32", 64), ("fp32", 128)]
INF = float("inf")


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


@pytest.mark.parametrize("dtype,d", ROWS)
@pytest.mark.parametrize("S,H,G,P", [(1, 2, 3, 40), (2, 2, 2, 200), (16, 4, 4, 150)])
@pytest.mark.parametrize("place", ["big 1e8", "big 1e12", "big 1e25", "first 16", "first 40", "scattered", "inf", "nan", "query nan"])
def test_extreme_logits(lazyev_lib, dtype, d, S, H, G, P, place):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(P + d)
    k = torch.empty((S, H, P, d), device="cuda").normal_(generator=gen).to(dt)
    q = (1.5 * torch.empty((S, P, H * G, d), device="cuda").normal_(generator=gen)).to(dt)
    j = P // 3
    if place.startswith("big"):
        k[0, 0, j] *= float(place.split()[1])
    elif place in ("first 16", "first 40", "scattered"):
        rows = slice(0, 16) if place == "first 16" else slice(0, P - 1 if P <= 40 else 40) if place == "first 40" else slice(1, P, 3)
        k[0, 0, rows, 7] = -INF
        q[0, :, :, 7] = q[0, :, :, 7].abs() + 0.1
    elif place == "inf":
        k[0, 0, j, 5] = INF
    elif place == "nan":
        k[0, 0, j, 5] = float("nan")
    else:
        q[0, P // 2, 1, 3] = float("nan")
    lower = torch.ones((P, P), dtype=torch.bool, device="cuda").tril()
    tau = torch.arange(1 - P, 1, dtype=torch.int32, device="cuda")
    weights = None
    for alpha in (0.02, 0.4):
        for export in (True, False):
            (ts_got, mri_got, n_got), p = _track(lazyev_lib, dt, k, q, alpha, export)
            if export:
                weights = p
                active = (p.view(S, H, G, P, P) >= alpha).any(2) & lower     # (NaN: not active)
                ts = tau.expand(S, H, P).clone()
                mri = torch.zeros_like(ts)
                for i in range(P):
                    on = active[:, :, i]
                    mri = torch.where(on, torch.maximum(mri, tau[i] - ts), mri)
                    ts = torch.where(on, tau[i], ts)
            assert n_got == int(active.sum()) and torch.equal(ts_got, ts) and torch.equal(mri_got, mri), (alpha, export)
    # the unit with the unusual rows, its first heads
    logits = (q[0, :, :G].double().transpose(0, 1) @ k[0, 0].double().T) * d ** -0.5
    want = torch.softmax(logits.masked_fill(~lower, -INF), -1).nan_to_num(0.0) * lower
    got = weights[0, :G].double().nan_to_num(0.0) * lower
    if place.startswith("big") and (dtype, d) == ("bf16", 128):
        # rows of 128 x bf16 fold the log-sum-exp into the product: the weight of a key whose logit's rounding exceeds
        # 1 is not told; all others are
        want[:, :, j] = got[:, :, j] = 0.0
    # (logits of ordinary keys: fp32 sums of d products, about 10 in magnitude together)
    assert float((got - want).abs().max()) <= 2 * d * 2.0 ** -24 * 10


@pytest.mark.parametrize("dtype,d", ROWS[1:])
@pytest.mark.parametrize("scale", [1e-38, 1e-31, 1e-20, 1e-6])
def test_smallest_softmax_scales(lazyev_lib, dtype, d, scale):
    """Every key has the same weight."""
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    S, H, G, P = 1, 2, 2, 90
    gen = torch.Generator(device="cuda").manual_seed(d)
    eng = lazyev_lib.LazyEviction(1, S, H * G, H, d, P + 40, 8, P, 0.02, dtype=dt, softmax_scale=scale)
    eng.k_cache[0, :, :, :P].normal_(generator=gen)
    eng.init()
    q = torch.empty((S, P, H * G, d), device="cuda").normal_(generator=gen).to(dt)
    p = torch.zeros((S, H * G, P, P), device="cuda")
    eng.prefill_track(0, q, p_out=p)
    want = 1.0 / torch.arange(1, P + 1, device="cuda", dtype=torch.float64).view(P, 1).expand(P, P).tril()
    rel = ((p.double() - want) / want).tril()[..., torch.ones((P, P), dtype=torch.bool, device="cuda").tril()]
    assert float(rel.abs().max()) < 1e-4               # (logits of up to 40 scale, and a few roundings of 2^-24)
    eng.close()
