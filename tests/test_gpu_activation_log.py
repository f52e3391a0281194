"""The activation log (single-launch kernel: one bit per entry and call, applied together) against tracking within
every call (variant 0), at the edges of its 32-entry words, 128-entry waves and 512-entry blocks and of its
sets of 32 and 128 calls; layers that hold different numbers of calls when the logs are applied."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(lazyev_lib, variant, P, steps, budget, window, L=3, S=2, H=2, G=2, d=64):
    gen = torch.Generator(device="cuda").manual_seed(P + steps)
    eng = lazyev_lib.LazyEviction(L, S, H * G, H, d, budget, window, P, 0.02, dtype=torch.float32)
    eng.k_cache[:, :, :, :P].normal_(generator=gen)
    eng.v_cache[:, :, :, :P].normal_(generator=gen)
    eng.init()
    eng.set_variant(variant)
    out = torch.empty((S, H * G, d), device="cuda")
    states = []
    for t in range(1, steps + 1):
        for l in range(L):
            q, k, v = (torch.empty((S, h, d), device="cuda").normal_(generator=gen) for h in (H * G, H, H))
            q[:, 0] += (t % 3) * eng.k_cache[l, :, 0, min(P - 1, 3 * (t % 11))]
            eng.decode_step(l, t, q, k, v, out)
            if t == steps // 2 and l == 1:         # two layers of three have taken the step
                eng.stats()
                states += [x[:, :, :, :P].clone() for x in (eng.ts, eng.mri, eng.pos)]
        eng.evict_all(t)
    st = eng.stats()
    states += [x[:, :, :, :st["len"][0]].clone() for x in (eng.ts, eng.mri, eng.pos)]
    eng.close()
    return states, st


# windows beyond 256 calls fill the log before an eviction
@pytest.mark.parametrize("P,steps,budget,window", [(5, 31, 100, 40), (33, 32, 34, 32), (100, 33, 90, 33), (127, 66, 400, 64),
                                                   (480, 65, 512, 64), (300, 129, 300, 128), (512, 130, 300, 128),
                                                   (900, 258, 700, 257), (1400, 300, 1500, 290), (40, 600, 1000, 600)])
def test_logged_calls_against_tracking_at_once(lazyev_lib, P, steps, budget, window):
    (a, st_a), (b, st_b) = (_run(lazyev_lib, v, P, steps, budget, window) for v in (0, 1))
    assert st_a == st_b and sum(st_a["n_activations"]) > 0
    for x, y in zip(a, b):
        assert torch.equal(x, y)
