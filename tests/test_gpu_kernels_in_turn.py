"""Decode calls of one context that take the two attention kernels in turn, and splits that grow in the course: the
partials of both kernels lie in one area.  Outputs and state against one kernel throughout."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(lazyev_lib, plan, dt, d, S=2, H=3, G=4, N=2300, steps=12):
    gen = torch.Generator(device="cuda").manual_seed(5)
    eng = lazyev_lib.LazyEviction(1, S, G * H, H, d, N + 40, 8, N, 8.0 / N, dtype=dt)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    out = torch.zeros((steps, S, G * H, d), dtype=dt, device="cuda")
    for t in range(1, steps + 1):
        variant, blocks = plan[(t - 1) % len(plan)]
        eng.set_variant(variant)
        if blocks:
            eng.set_target_blocks(blocks * S * H)
        q, k, v = (torch.empty((S, h, d), device="cuda").normal_(generator=gen) for h in (G * H, H, H))
        q[:, ::3] += 4.0 * eng.k_cache[0, :, :1, N // 2].float()
        eng.decode_step(0, t, q.to(dt), k.to(dt), v.to(dt), out[t - 1])
    st = eng.stats()
    state = [x[:, :, :, :N + steps].clone() for x in (eng.ts, eng.mri, eng.pos, eng.k_cache, eng.v_cache)]
    eng.close()
    return out.double(), state, st


@pytest.mark.parametrize("dtype,d", [("fp32", 64), ("fp32", 128), ("bf16", 64)])
@pytest.mark.parametrize("plan", [[(0, 0), (1, 0)], [(1, 2), (1, 7), (0, 0), (1, 9), (1, 36), (0, 0), (1, 4)]])
def test_kernels_in_turn(lazyev_lib, dtype, d, plan):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    (want, state_w, st_w), (got, state_g, st_g) = (_run(lazyev_lib, p, dt, d) for p in ([(0, 0)], plan))
    err = float(((got - want).norm(dim=-1) / want.norm(dim=-1)).max())
    # fp32: sums of some thousand terms in two orders (about 1e-6 at most); bf16: two fp32 sums, rounded once each
    assert err < (1e-5 if dt == torch.float32 else 2.0 ** -8), err
    assert st_w == st_g and all(torch.equal(x, y) for x, y in zip(state_w, state_g))


@pytest.mark.parametrize("units,N", [(128, 700), (172, 700), (192, 700), (192, 6200), (240, 2200), (600, 700)])
def test_more_blocks_than_the_library_would_take(lazyev_lib, units, N):
    """lazyev_set_target_blocks far beyond the chip: as many blocks per unit as the workspace has records for."""
    H, G, d = 4, 7, 128
    outs = []
    for blocks in (0, 100):
        gen = torch.Generator(device="cuda").manual_seed(3)
        S = units // H
        eng = lazyev_lib.LazyEviction(1, S, G * H, H, d, N + 40, 8, N, 8.0 / N)
        eng.k_cache[:, :, :, :N].normal_(generator=gen)
        eng.v_cache[:, :, :, :N].normal_(generator=gen)
        eng.init()
        if blocks:
            eng.set_target_blocks(blocks * units)
        out = torch.zeros((3, S, G * H, d), dtype=torch.bfloat16, device="cuda")
        for t in range(1, 4):
            q, k, v = (torch.empty((S, h, d), device="cuda").normal_(generator=gen).to(torch.bfloat16) for h in (G * H, H, H))
            eng.decode_step(0, t, q, k, v, out[t - 1])
        outs.append((out.double(), eng.stats()["n_activations"]))
        eng.close()
    (a, n_a), (b, n_b) = outs
    # (a weight within rounding of alpha may fall on either side of it: about one in 1e7, of up to 3e7 here)
    assert abs(n_a[0] - n_b[0]) <= 20 and float(((a - b).norm(dim=-1) / a.norm(dim=-1)).max()) < 2 * 2.0 ** -8
