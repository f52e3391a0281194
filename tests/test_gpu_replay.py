"""A captured decode call that is replayed: the inputs are rewritten in place between the replays, with eager work
and synchronisations between them, and every replay's output equals the eager result of the same inputs
bit for bit, for every kind of split and row type."""
import pytest
import torch

pytestmark = pytest.mark.gpu

REPLAYS = 40


def _engine(lazyev_lib, stream, dt, d, S, H, G, N, k, v):
    eng = lazyev_lib.LazyEviction(1, S, H * G, H, d, N + 40, 8, N, 8.0 / N, dtype=dt, stream=stream)
    eng.k_cache[:, :, :, :N].copy_(k)
    eng.v_cache[:, :, :, :N].copy_(v)
    return eng


@pytest.mark.parametrize("calls", [1, 2])
@pytest.mark.parametrize("dtype,d,blocks,N", [("fp32", 64, 3, 700), ("fp32", 128, 8, 900), ("bf16", 64, 6, 900), ("bf16", 128, 2, 700),
                                              ("bf16", 128, 8, 2000), ("bf16", 128, 17, 3000)])
def test_replayed_calls(lazyev_lib, dtype, d, blocks, N, calls):
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    S, H, G = 2, 4, 2
    stream = torch.cuda.Stream()
    gen = torch.Generator(device="cuda").manual_seed(blocks)
    k, v = (torch.empty((1, S, H, N, d), device="cuda").normal_(generator=gen).to(dt) for _ in range(2))
    q, kn, vn = (torch.empty((REPLAYS, calls, S, h, d), device="cuda").normal_(generator=gen).to(dt) for h in (H * G, H, H))
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        want = torch.zeros((REPLAYS, calls, S, H * G, d), dtype=dt, device="cuda")
        eng = _engine(lazyev_lib, stream, dt, d, S, H, G, N, k, v)
        for r in range(REPLAYS):                   # eager: a fresh context for every set of inputs
            eng.init()
            eng.set_target_blocks(blocks * S * H)
            for c in range(calls):
                eng.decode_step(0, 1 + c, q[r, c], kn[r, c], vn[r, c], want[r, c])
        eng.close()
        eng = _engine(lazyev_lib, stream, dt, d, S, H, G, N, k, v).init()
        eng.set_target_blocks(blocks * S * H)
        bufs = [x[0].clone() for x in (q, kn, vn)]
        out = torch.zeros((calls, S, H * G, d), dtype=dt, device="cuda")
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            for c in range(calls):
                eng.decode_step(0, 1 + c, bufs[0][c], bufs[1][c], bufs[2][c], out[c])
        wrong = []
        for r in range(REPLAYS):
            for b, x in zip(bufs, (q, kn, vn)):
                b.copy_(x[r])
            if r % 3 == 1:
                torch.zeros((1 << 20,), device="cuda").add_(1.0)
                stream.synchronize()
            graph.replay()
            if not torch.equal(out, want[r]):
                wrong.append(r)
        assert not wrong, wrong
        # the context goes on from where the captured calls left it
        eng.decode_step(0, 1 + calls, bufs[0][0], bufs[1][0], bufs[2][0], out[0])
        assert eng.stats()["len"] == [N + calls + 1]
        assert bool(out[0].isfinite().all())
    eng.close()
