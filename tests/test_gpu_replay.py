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


@pytest.mark.parametrize("how", ["evict", "stats"])
@pytest.mark.parametrize("G", [7, 8])
def test_replays_after_the_cache_has_grown(lazyev_lib, G, how):
    """The candidate records of 250 entries over four blocks lie elsewhere than those of 257 and more: a call captured at 251
    entries is replayed between eager calls up to 290, and right before what is outstanding is applied (by the
    selection of an eviction, or by a launch of its own).  Outputs against fp64 softmax attention; every row of the cache
    is the one its place (after an eviction, its position) says."""
    S, H, N, W, budget = 2, 4, 250, 40, 280
    stream = torch.cuda.Stream()
    gen = torch.Generator(device="cuda").manual_seed(G)
    q, kn, vn = (torch.empty((W + 1, S, h, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16) for h in (H * G, H, H))
    k, v = (torch.empty((S, H, N + W, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16) for _ in range(2))
    for all_rows, new in ((k, kn), (v, vn)):
        all_rows[:, :, N:] = new[1:].permute(1, 2, 0, 3)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        eng = lazyev_lib.LazyEviction(1, S, H * G, H, 128, budget, W, N, 0.02, stream=stream)
        eng.load_prompt(0, k[:, :, :N], v[:, :, :N])
        eng.init()
        eng.set_target_blocks(4 * S * H)
        out = torch.zeros((W + 1, S, H * G, 128), dtype=torch.bfloat16, device="cuda")
        graph = torch.cuda.CUDAGraph()
        for t in range(1, W + 1):
            if t == 2:                             # (its candidate records go to the second buffer, as those of the last call)
                stream.synchronize()
                with torch.cuda.graph(graph, stream=stream):
                    eng.decode_step(0, t, q[t], kn[t], vn[t], out[t])
                graph.replay()
            else:
                eng.decode_step(0, t, q[t], kn[t], vn[t], out[t])
            if t % 3 == 0 or t == W:
                graph.replay()
        n = N + W
        if how == "evict":
            assert eng.evict(0, W) == n - budget
            n = budget
        assert eng.stats()["len"] == [n]
        for t in range(1, W + 1):
            p = torch.softmax(torch.matmul(k[:, :, :N + t].double(), q[t].double().view(S, H, G, 128).transpose(2, 3).contiguous()) / 128 ** 0.5, dim=2)
            ref = torch.matmul(p.transpose(2, 3).contiguous(), v[:, :, :N + t].double()).view(S, H * G, 128)
            err = (out[t].double() - ref).norm(dim=2) / ref.norm(dim=2)
            assert float(err.max()) < 2 * 2.0 ** -8, (t, float(err.max()))   # (two roundings to bf16 of relative size 2^-9)
        if how == "evict":
            pos = eng.pos[0, :, :, :n].long()
        else:                                      # (what the last call left for its entry's position is gone)
            pos = torch.arange(n, device="cuda").expand(S, H, n).contiguous()
        assert int(pos.min()) >= 0 and int(pos.max()) < N + W and bool((pos.diff(dim=2) > 0).all())
        for cache, rows in ((eng.k_cache, k), (eng.v_cache, v)):
            assert torch.equal(cache[0, :, :, :n], rows.gather(2, pos.unsqueeze(3).expand(-1, -1, -1, 128)))
        eng.close()


def test_replays_between_eager_calls_whose_numbers_start_over(lazyev_lib):
    """Eager calls number their partials with 16 bits, a captured call leaves its partials with one number at every
    replay: an early captured call is replayed before each eager call around the 65536th, whose outputs
    are compared with fp64 softmax attention over what the cache holds."""
    L, H, G, N, steps, captured_at = 64, 8, 2, 250, 1030, 10
    stream = torch.cuda.Stream()
    gen = torch.Generator(device="cuda").manual_seed(5)
    k, v = (torch.empty((L, 1, H, N, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16) for _ in range(2))
    q, kn, vn = (torch.empty((5, 1, h, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16) for h in (H * G, H, H))
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        eng = lazyev_lib.LazyEviction(L, 1, H * G, H, 128, N + steps, 64, N, 0.05, stream=stream)
        eng.k_cache[:, :, :, :N].copy_(k)
        eng.v_cache[:, :, :, :N].copy_(v)
        eng.init()
        eng.set_target_blocks(4 * H)
        out, out_replayed = (torch.zeros((1, H * G, 128), dtype=torch.bfloat16, device="cuda") for _ in range(2))
        graph, launches, wrong = torch.cuda.CUDAGraph(), 0, []
        for t in range(1, steps + 1):
            for layer in range(L):
                x = (t + layer) % 4
                if launches == captured_at:
                    stream.synchronize()
                    with torch.cuda.graph(graph, stream=stream):
                        eng.decode_step(layer, t, q[4], kn[4], vn[4], out_replayed)
                    graph.replay()
                    launches += 1
                    continue
                near = 65526 <= launches < 65610
                if near:
                    graph.replay()
                eng.decode_step(layer, t, q[x], kn[x], vn[x], out)
                launches += 1
                if near:
                    n = N + t
                    kd, vd = eng.k_cache[layer, 0, :, :n].double(), eng.v_cache[layer, 0, :, :n].double()
                    p = torch.softmax(torch.matmul(kd, q[x, 0].double().view(H, G, 128).transpose(1, 2).contiguous()) / 128 ** 0.5, dim=1)
                    ref = torch.matmul(p.transpose(1, 2).contiguous(), vd).view(H * G, 128)
                    err = float(((out[0].double() - ref).norm(dim=1) / ref.norm(dim=1)).max())
                    if not err < 2 * 2.0 ** -8:    # (bf16 weights and a bf16 result: two roundings of relative size 2^-9)
                        wrong.append((launches, err))
        assert launches > 65610 and not wrong, wrong
        eng.close()
