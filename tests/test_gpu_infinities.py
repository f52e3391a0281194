"""Infinite and NaN elements in the caches and in the appended rows: the single-launch kernel against the split +
merge kernels (variant 0), which multiply every weight in fp32.  The same elements of the output are +inf, -inf, NaN
and finite; finite ones agree."""
import pytest
import torch

pytestmark = pytest.mark.gpu

ROWS = [("fp32", 64), ("fp32", 128), ("bf16", 64)]


def _run(lazyev_lib, variant, dtype, d, place, value, N, H=2, G=4, S=2, steps=2, blocks=0):
    gen = torch.Generator(device="cuda").manual_seed(N)
    eng = lazyev_lib.LazyEviction(1, S, H * G, H, d, N + 40, 8, N, 0.01, dtype=dtype)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    cols = torch.arange(0, d, 5, device="cuda")    # columns in every register of a row
    sign = torch.where(cols % 2 == 0, value, -value).to(dtype)
    q, kn, vn = (torch.empty((steps, S, h, d), device="cuda").normal_(generator=gen).to(dtype) for h in (H * G, H, H))
    if place == "cached V":
        eng.v_cache[0, 0, :, N // 2, cols] = sign
    elif place == "first V":
        eng.v_cache[0, :, :, 0, cols] = sign
    elif place == "appended V":
        vn[0, :, 0, cols] = sign
    elif place == "cached K":
        eng.k_cache[0, 0, 0, N // 3, 3] = value
    elif place == "query":
        q[0, 1, 2, 7] = value
    elif place == "large K":
        eng.k_cache[0, 0, 0, N // 3] *= value
    eng.init()
    eng.set_variant(variant)
    if N > 2000 or blocks:                         # one block per unit: runs whose logits leave LDS in segments
        eng.set_target_blocks(max(blocks, 1) * S * H)
    out = torch.zeros((steps, S, H * G, d), dtype=dtype, device="cuda")
    for t in range(1, steps + 1):
        eng.decode_step(0, t, q[t - 1], kn[t - 1], vn[t - 1], out[t - 1])
    act = eng.stats()["n_activations"]
    state = [x[:, :, :, :N + steps].clone() for x in (eng.ts, eng.mri)]
    eng.close()
    return out.double(), state, act


@pytest.mark.parametrize("dtype,d", ROWS)
@pytest.mark.parametrize("place", ["cached V", "first V", "appended V", "cached K", "query"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
@pytest.mark.parametrize("N,blocks", [(3, 0), (15, 0), (64, 0), (333, 0), (2600, 0), (2600, 9), (2600, 17), (2600, 33)])
def test_infinite_elements(lazyev_lib, dtype, d, place, value, N, blocks):
    """(Of more than eight blocks a unit, blocks of their own merge the partials, two, four or eight records a lane.)"""
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    (want, state0, act0), (got, state1, act1) = (_run(lazyev_lib, v, dt, d, place, value, N, blocks=blocks) for v in (0, 1))
    assert torch.equal(got.isnan(), want.isnan())
    assert torch.equal(got.isposinf(), want.isposinf()) and torch.equal(got.isneginf(), want.isneginf())
    assert (want.isposinf().any() and want.isneginf().any()) if place.endswith("V") and value == float("inf") else want.isnan().any()
    ok = want.isfinite()
    # two orders of fp32 sums of N + 2 terms, of unit size together; bf16: one rounding of each of two results
    tol = (N + 2) * 2.0 ** -23 if dt == torch.float32 else 2.0 ** -7
    assert float((got - want)[ok].abs().max()) < tol * max(1.0, float(want[ok].abs().max()))
    assert act0 == act1 and all(torch.equal(x, y) for x, y in zip(state0, state1))


@pytest.mark.parametrize("dtype,d", ROWS + [("bf16", 128)])
@pytest.mark.parametrize("value", [1e8, 1e12, 1e25])
@pytest.mark.parametrize("N,blocks", [(3, 0), (64, 0), (333, 0), (2600, 0), (2600, 9), (2600, 17), (2600, 33)])
def test_large_logits(lazyev_lib, dtype, d, value, N, blocks):
    """A key with logits so large that their rounding exceeds the range of an exponential."""
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    (want, state0, act0), (got, state1, act1) = (_run(lazyev_lib, v, dt, d, "large K", value, N, blocks=blocks) for v in (0, 1))
    assert bool(want.isfinite().all()) and bool(got.isfinite().all())
    tol = (N + 2) * 2.0 ** -23 if dt == torch.float32 else 2.0 ** -6
    assert float((got - want).abs().max()) < tol * max(1.0, float(want.abs().max()))
    assert act0 == act1 and all(torch.equal(x, y) for x, y in zip(state0, state1))


@pytest.mark.parametrize("dtype,d", ROWS + [("bf16", 128)])
@pytest.mark.parametrize("N,blocks", [(40, 0), (333, 0), (333, 1), (700, 3), (2600, 1), (2600, 9), (2600, 17), (2600, 33)])
def test_entries_without_weight(lazyev_lib, dtype, d, N, blocks):
    """Runs of entries whose logits are -inf in every head, long enough to fill whole sub-tiles, a wave's first ones among
    them: softmax in 64 bits over the others, and no activation of theirs."""
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    H, G, S, steps = 2, 4, 2, 2
    gen = torch.Generator(device="cuda").manual_seed(N)
    eng = lazyev_lib.LazyEviction(1, S, H * G, H, d, N + 40, 8, N, 0.001, dtype=dt)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    gone = torch.zeros(N, dtype=torch.bool, device="cuda")
    gone[:35] = gone[N // 2:N // 2 + 70] = True
    gone[N - 1] = False
    eng.k_cache[0, :, :, :N][:, :, gone, 5] = -float("inf")
    eng.init()
    if blocks:
        eng.set_target_blocks(blocks * S * H)
    out = torch.zeros((S, H * G, d), dtype=dt, device="cuda")
    for t in range(1, steps + 1):
        q, kn, vn = (torch.empty((S, h, d), device="cuda").normal_(generator=gen).to(dt) for h in (H * G, H, H))
        q[..., 5] = q[..., 5].abs() + 0.125
        eng.decode_step(0, t, q, kn, vn, out)
        k, v = eng.k_cache[0, :, :, :N + t].double(), eng.v_cache[0, :, :, :N + t].double()
        p = torch.softmax(torch.matmul(q.double().view(S, H, G, d), k.transpose(2, 3).contiguous()) * d ** -0.5, dim=-1)
        want = torch.matmul(p, v).view(S, H * G, d)
        err = float(((out.double() - want).norm(dim=-1) / want.norm(dim=-1)).max())
        assert err < (1e-5 if dt == torch.float32 else 2 * 2.0 ** -8), (t, err)
    eng.stats()
    assert bool((eng.ts[0, :, :, :N][:, :, gone] == 0).all()) and bool((eng.ts[0, :, :, :N][:, :, ~gone] > 0).any())
    eng.close()
