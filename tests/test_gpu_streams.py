"""Work on a stream of the caller's own, with inputs written on it just before the call, beside another context
on another stream: every kernel runs on its context's stream and contexts share nothing.  Repeated runs give the same bits."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _drive(lazyev_lib, stream, dt, d, seed, S=3, H=2, G=4, P=300, steps=12, window=6):
    """A generator, so that two contexts can take turns."""
    with torch.cuda.stream(stream):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        eng = lazyev_lib.LazyEviction(2, S, H * G, H, d, P - 5, window, P, 0.02, dtype=dt, stream=stream)
        eng.k_cache[:, :, :, :P].normal_(generator=gen)
        eng.v_cache[:, :, :, :P].normal_(generator=gen)
        eng.init()
        out = torch.empty((steps, 2, S, H * G, d), dtype=dt, device="cuda")
        q = torch.empty((S, P, H * G, d), device="cuda").normal_(generator=gen).to(dt)
        for l in range(2):
            eng.prefill_track(l, q)
    yield
    for t in range(1, steps + 1):
        with torch.cuda.stream(stream):
            for l in range(2):
                q, k, v = (torch.empty((S, h, d), device="cuda").normal_(generator=gen).to(dt) for h in (H * G, H, H))
                eng.decode_step(l, t, q, k, v, out[t - 1, l])
            eng.evict_all(t)
        yield
    hist = eng.mri_histogram()
    st = eng.stats()
    n = st["len"][0]
    yield [out] + [x[:, :, :, :n].clone() for x in (eng.ts, eng.mri, eng.pos, eng.k_cache, eng.v_cache)], st, hist
    eng.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 64), ("fp32", 128)])
def test_two_streams_and_the_default_one(lazyev_lib, dtype, d):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    alone = {}
    for seed in (1, 2):
        *_, last = (x for x in _drive(lazyev_lib, torch.cuda.current_stream(), dt, d, seed) if x is not None)
        alone[seed] = last
    pair = {seed: _drive(lazyev_lib, torch.cuda.Stream(), dt, d, seed) for seed in (1, 2)}
    got = {}
    while len(got) < 2:
        for seed, run in pair.items():
            if seed not in got:
                x = next(run)
                if x is not None:
                    got[seed] = x
    for seed in (1, 2):
        (a, st_a, hist_a), (b, st_b, hist_b) = alone[seed], got[seed]
        assert st_a == st_b and hist_a == hist_b and sum(st_a["n_evict_events"]) == 4
        for x, y in zip(a, b):
            assert torch.equal(x, y)
