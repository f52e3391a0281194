"""Queries, appended rows and outputs of a decode call, and the queries of a prompt, that start at any element: the
library asks for no alignment of them.  Same bits as from aligned memory."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _at(x, shift):
    """A copy of x that starts `shift` elements into its memory."""
    y = torch.empty(x.numel() + shift + 8, dtype=x.dtype, device="cuda")[shift:shift + x.numel()].view(x.shape)
    return y.copy_(x)


def _run(lazyev_lib, dt, d, shifts, S=2, H=2, G=3, N=130, steps=5):
    gen = torch.Generator(device="cuda").manual_seed(d)
    eng = lazyev_lib.LazyEviction(1, S, H * G, H, d, N + 30, 8, N, 0.02, dtype=dt)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    qp = torch.empty((S, N, H * G, d), device="cuda").normal_(generator=gen).to(dt)
    eng.prefill_track(0, _at(qp, shifts[0]))
    res = []
    for t in range(1, steps + 1):
        q, k, v = (torch.empty((S, h, d), device="cuda").normal_(generator=gen).to(dt) for h in (H * G, H, H))
        out = _at(torch.zeros((S, H * G, d), dtype=dt, device="cuda"), shifts[3])
        eng.decode_step(0, t, _at(q, shifts[0]), _at(k, shifts[1]), _at(v, shifts[2]), out)
        res.append(out.clone())
    st = eng.stats()
    res += [x[:, :, :, :N + steps].clone() for x in (eng.ts, eng.mri, eng.k_cache, eng.v_cache)]
    eng.close()
    return res, st


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 64), ("fp32", 128)])
def test_buffers_at_any_element(lazyev_lib, dtype, d):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    want, st_w = _run(lazyev_lib, dt, d, (0, 0, 0, 0))
    for shifts in ((1, 2, 3, 1), (3, 1, 1, 2), (2, 3, 2, 3)):
        got, st_g = _run(lazyev_lib, dt, d, shifts)
        assert st_w == st_g and all(torch.equal(x, y) for x, y in zip(want, got)), shifts
