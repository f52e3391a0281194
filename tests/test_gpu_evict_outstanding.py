"""Tracking that is outstanding when an eviction is due: applied by the selection itself, or by launches of its own
(lazyev_stats before the eviction).  Same state bit for bit, places beyond the budget included."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(lazyev_lib, first_stats, per_layer, L, S, group, H, d, dtype, B, W, steps, prompt, last_layer=None):
    gen = torch.Generator(device="cuda").manual_seed(B + W + group)
    eng = lazyev_lib.LazyEviction(L, S, group * H, H, d, B, W, prompt, 8.0 / (B + W), dtype=dtype)
    eng.k_cache[:, :, :, :prompt].normal_(generator=gen)
    eng.v_cache[:, :, :, :prompt].normal_(generator=gen)
    eng.init()
    out = torch.zeros((S, group * H, d), dtype=dtype, device="cuda")
    events = 0
    order = list(range(L)) if last_layer is None else [x for x in range(L) if x != last_layer] + [last_layer]
    for t in range(1, steps + 1):
        for layer in order:
            q, kn, vn = (torch.empty((S, h, d), device="cuda").normal_(generator=gen).to(dtype) for h in (group * H, H, H))
            q = (q.float() + 2.0 * eng.k_cache[layer, :, :, (7 * t) % prompt].float().repeat_interleave(group, dim=1)).to(dtype)
            eng.decode_step(layer, t, q, kn, vn, out)
        if first_stats:
            eng.stats()
        if per_layer:
            events += sum(1 for layer in reversed(range(L)) if eng.evict(layer, t))
        else:
            events += 1 if eng.evict_all(t) else 0
    st = eng.stats()
    state = [x.clone() for x in (eng.ts, eng.mri, eng.pos)] + [eng.k_cache.float().clone(), out.float().clone()]
    eng.close()
    return events, st, state


# the selection's instances hold 2, 3, 5 and 8 entries per thread (2048, 3072, 5120, 8192 entries); 32 calls are applied at a time, 128
# (64 from 5 on) requested together, 256 logged
@pytest.mark.parametrize("L,S,group,H,d,dtype,B,W,steps,prompt", [
    (2, 2, 7, 2, 128, torch.bfloat16, 60, 3, 9, 60), (1, 1, 8, 1, 128, torch.bfloat16, 1000, 33, 66, 1000),
    (3, 1, 4, 2, 64, torch.float32, 2010, 38, 38, 2010), (1, 2, 8, 1, 64, torch.bfloat16, 2000, 49, 49, 2000),
    (2, 1, 7, 1, 128, torch.bfloat16, 2900, 130, 130, 2900), (1, 1, 1, 2, 128, torch.float32, 5000, 65, 65, 5000),
    (1, 1, 7, 1, 128, torch.bfloat16, 8100, 92, 92, 8100), (1, 1, 3, 1, 128, torch.bfloat16, 8150, 43, 43, 8150),
    (1, 1, 7, 1, 128, torch.bfloat16, 400, 270, 270, 400), (2, 1, 5, 1, 64, torch.float32, 90, 40, 80, 20)])
@pytest.mark.parametrize("per_layer", [False, True])
def test_selection_applies_what_is_outstanding(lazyev_lib, per_layer, L, S, group, H, d, dtype, B, W, steps, prompt):
    runs = [_run(lazyev_lib, first, per_layer, L, S, group, H, d, dtype, B, W, steps, prompt) for first in (True, False)]
    assert runs[0][0] == runs[1][0] > 0
    assert runs[0][1] == runs[1][1]
    for x, y in zip(runs[0][2], runs[1][2]):
        assert torch.equal(x, y)


# the layer whose call is the last before the eviction is any of them; 5 entries per thread from 32 units on (31: launches of its own), up
# to 5120 entries
@pytest.mark.parametrize("last_layer", [0, 1, 2])
def test_last_call_of_any_layer(lazyev_lib, last_layer):
    args = (3, 2, 7, 2, 128, torch.bfloat16, 300, 40, 80, 300)
    runs = [_run(lazyev_lib, first, False, *args, last_layer=last_layer) for first in (True, False)]
    assert runs[0][0] == runs[1][0] > 0 and runs[0][1] == runs[1][1]
    for x, y in zip(runs[0][2], runs[1][2]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("L,S,H,B,W", [(1, 32, 1, 3020, 53), (1, 31, 1, 3020, 53), (2, 4, 4, 3019, 53), (1, 8, 4, 5055, 65), (1, 8, 4, 5056, 65),
                                       (1, 8, 4, 4990, 129)])
def test_five_entries_per_thread(lazyev_lib, L, S, H, B, W):
    runs = [_run(lazyev_lib, first, False, L, S, 1, H, 64, torch.bfloat16, B, W, W, B) for first in (True, False)]
    assert runs[0][0] == runs[1][0] > 0 and runs[0][1] == runs[1][1]
    for x, y in zip(runs[0][2], runs[1][2]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("S,first", [(128, 64), (129, 64), (160, 32)])
def test_many_units_as_several_contexts(lazyev_lib, S, first):
    """512 units at once, 516 (tracking in launches of its own, the selection without) and 640: the same state, bit for bit,
    as the same sequences in two contexts of at most 512 units each, whose calls have one block per unit as well."""
    H, group, d, B, W, steps = 4, 2, 64, 70, 9, 27
    gen = torch.Generator(device="cuda").manual_seed(S)
    rnd = lambda *shape: torch.empty(shape, device="cuda").normal_(generator=gen).to(torch.bfloat16)
    k, v, q, kn, vn = rnd(S, H, B, d), rnd(S, H, B, d), rnd(steps, S, group * H, d), rnd(steps, S, H, d), rnd(steps, S, H, d)
    q = (q.float() + 2.0 * k[:, :, 7].float().repeat_interleave(group, dim=1)).to(torch.bfloat16)
    states = []
    for parts in (((0, S),), ((0, first), (first, S))):
        state = []
        for a, b in parts:
            eng = lazyev_lib.LazyEviction(1, b - a, group * H, H, d, B, W, B, 8.0 / (B + W))
            eng.load_prompt(0, k[a:b], v[a:b])
            eng.init()
            eng.set_target_blocks((b - a) * H)
            out = torch.zeros((b - a, group * H, d), dtype=torch.bfloat16, device="cuda")
            for t in range(1, steps + 1):
                eng.decode_step(0, t, q[t - 1, a:b].contiguous(), kn[t - 1, a:b].contiguous(), vn[t - 1, a:b].contiguous(), out)
                assert eng.evict_all(t) == (W if t % W == 0 else 0)
            assert eng.stats()["n_evict_events"] == [steps // W]
            state.append([x[0].clone() for x in (eng.ts, eng.mri, eng.pos)] + [eng.k_cache[0, :, :, :B].clone(), out])
            eng.close()
        states.append([torch.cat(x) for x in zip(*state)])
    for x, y in zip(*states):
        assert torch.equal(x, y)
