"""Partials of a unit handed over between its blocks: up to 8 blocks (an instance of the kernel each) to the unit's last
one, up to 64 to blocks that merge them, two, four or eight records per lane."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _run(lazyev_lib, blocks, N, steps, group):
    H = 2
    gen = torch.Generator(device="cuda").manual_seed(7)
    eng = lazyev_lib.LazyEviction(1, 1, group * H, H, 128, N + 100, 64, N, 8.0 / N)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    if blocks:
        eng.set_target_blocks(blocks * H)
    x = [torch.empty((steps, 1, h, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16)
         for h in (group * H, H, H)]
    out = torch.zeros((steps, 1, group * H, 128), dtype=torch.bfloat16, device="cuda")
    for t in range(1, steps + 1):
        eng.decode_step(0, t, x[0][t - 1], x[1][t - 1], x[2][t - 1], out[t - 1])
    eng.stats()
    k, v = eng.k_cache[0, 0].double(), eng.v_cache[0, 0].double()
    for t in range(1, steps + 1):
        n = N + t
        q = x[0][t - 1, 0].double().view(H, group, 128)
        p = torch.softmax(torch.matmul(q, k[:, :n].transpose(1, 2).contiguous()) / np.sqrt(128.0), dim=-1)
        ref = torch.matmul(p, v[:, :n]).view(group * H, 128)
        # bf16 weights and a bf16 result: two roundings of relative size 2^-9, independent per element
        err = (out[t - 1, 0].double() - ref).norm(dim=1) / ref.norm(dim=1)
        assert float(err.max()) < 2 * 2.0 ** -8, (blocks, t, float(err.max()))
    state = [y[0, 0, :, :N + steps].clone() for y in (eng.ts, eng.mri, eng.pos)]
    eng.close()
    return state


@pytest.mark.parametrize("N,group,blocks", [(4080, 7, (1, 2, 3, 5, 6, 7, 8, 9, 15, 16, 17, 24, 32, 33, 63, 64, 0)),
                                            (150, 4, (1, 2, 3, 0)), (3, 1, (1, 0)), (62, 7, (2, 0)), (13000, 7, (8, 9, 16))])
def test_every_number_of_blocks_gives_the_same_result(lazyev_lib, N, group, blocks):
    """Outputs against fp64 softmax attention; TS / MRI / pos equal whatever the split (a decision
    within rounding of alpha could differ: about one in 1e7, of 1e5 here)."""
    first = None
    for b in blocks:
        state = _run(lazyev_lib, b, N, 6, group)
        if first is None:
            first = state
        for x, y in zip(state, first):
            assert torch.equal(x, y), b


@pytest.mark.parametrize("batch,N", [(12, 700), (20, 700), (24, 6200), (36, 700), (36, 2200)])
def test_more_units_than_blocks_fit_evenly(lazyev_lib, batch, N):
    """48, 80, 96 and 144 units of one launch (3, 2, 5, 1 and 3 blocks per unit; with and without list
    waves): outputs of sampled sequences against fp64 softmax attention."""
    H, group, steps = 4, 7, 3
    gen = torch.Generator(device="cuda").manual_seed(9)
    eng = lazyev_lib.LazyEviction(1, batch, group * H, H, 128, N + 100, 64, N, 8.0 / N)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    out = torch.zeros((batch, group * H, 128), dtype=torch.bfloat16, device="cuda")
    for t in range(1, steps + 1):
        q, kn, vn = (torch.empty((batch, h, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16)
                     for h in (group * H, H, H))
        eng.decode_step(0, t, q, kn, vn, out)
        n = N + t
        for s in (0, batch // 2, batch - 1):
            k, v = eng.k_cache[0, s, :, :n].double(), eng.v_cache[0, s, :, :n].double()
            p = torch.softmax(torch.matmul(q[s].double().view(H, group, 128), k.transpose(1, 2).contiguous()) /
                              np.sqrt(128.0), dim=-1)
            ref = torch.matmul(p, v).view(group * H, 128)
            err = (out[s].double() - ref).norm(dim=1) / ref.norm(dim=1)
            assert float(err.max()) < 2 * 2.0 ** -8, (s, t, float(err.max()))
    assert eng.stats()["len"] == [N + steps]
    eng.close()


def test_launch_numbers_start_over(lazyev_lib):
    """The stamp of a record has 16 bits: 67 layers x 980 steps are more launches than that.  Outputs of the steps
    around the 65536th launch against fp64 softmax attention, and no block gave up waiting."""
    L, H, group, B, W, steps = 67, 2, 7, 130, 60, 980
    gen = torch.Generator(device="cuda").manual_seed(3)
    eng = lazyev_lib.LazyEviction(L, 1, group * H, H, 128, B, W, B, 0.05)
    eng.k_cache[:, :, :, :B].normal_(generator=gen)
    eng.v_cache[:, :, :, :B].normal_(generator=gen)
    eng.init()
    q, kn, vn = (torch.empty((4, 1, h, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16) for h in (group * H, H, H))
    out = torch.zeros((L, 1, group * H, 128), dtype=torch.bfloat16, device="cuda")
    n = B
    for t in range(1, steps + 1):
        x = t % 4
        for layer in range(L):
            eng.decode_step(layer, t, q[x], kn[x], vn[x], out[layer])
        n += 1
        if 976 <= t <= 979:                            # launches 65326 .. 65593
            ref_q = q[x, 0].double().view(H, group, 128)
            k, v = eng.k_cache[:, 0, :, :n].double(), eng.v_cache[:, 0, :, :n].double()
            p = torch.softmax(torch.matmul(ref_q, k.transpose(2, 3).contiguous()) / np.sqrt(128.0), dim=-1)
            ref = torch.matmul(p, v).view(L, group * H, 128)
            err = (out[:, 0].double() - ref).norm(dim=2) / ref.norm(dim=2)
            assert float(err.max()) < 2 * 2.0 ** -8, (t, float(err.max()))   # (two roundings to bf16, as above)
        if eng.evict_all(t):
            n = B
    assert eng.stats()["last_step"] == [steps] * L
    eng.close()


@pytest.mark.parametrize("many,N", [(8, 500), (17, 1100)])
def test_records_left_a_whole_cycle_of_numbers_ago(lazyev_lib, many, N):
    """Launch 100 has eight blocks per unit, or seventeen, whose records other blocks merge; all others up to the next one with
    that number (eager numbers run from 1 to 65534) have two, which leave all but the first of its seven or seventeen records as
    they are.  That launch, over other inputs, must not take them for its own: they are cleared when the numbers start over."""
    L, H, group, steps, period = 64, 8, 2, 1030, 65534
    gen = torch.Generator(device="cuda").manual_seed(4)
    eng = lazyev_lib.LazyEviction(L, 1, group * H, H, 128, N + steps, 64, N, 0.05)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    q, kn, vn = (torch.empty((5, 1, h, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16) for h in (group * H, H, H))
    out = torch.zeros((1, group * H, 128), dtype=torch.bfloat16, device="cuda")
    launches, checked = 0, []
    for t in range(1, steps + 1):
        for layer in range(L):
            launches += 1
            looked_at = launches in (100, period + 100)
            x = launches % 5
            eng.set_target_blocks((many if looked_at else 2) * H)
            eng.decode_step(layer, t, q[x], kn[x], vn[x], out)
            if looked_at:
                k, v = eng.k_cache[layer, 0, :, :N + t].double(), eng.v_cache[layer, 0, :, :N + t].double()
                p = torch.softmax(torch.matmul(k, q[x, 0].double().view(H, group, 128).transpose(1, 2).contiguous()) / np.sqrt(128.0), dim=1)
                ref = torch.matmul(p.transpose(1, 2).contiguous(), v).view(group * H, 128)
                checked.append(float(((out[0].double() - ref).norm(dim=1) / ref.norm(dim=1)).max()))
    assert len(checked) == 2 and max(checked) < 2 * 2.0 ** -8, checked   # (two roundings to bf16, as above)
    assert eng.stats()["last_step"] == [steps] * L
    eng.close()


@pytest.mark.parametrize("group,blocks,N", [(7, 16, 2300), (8, 33, 2300), (1, 17, 2300), (5, 9, 2300), (8, 40, 33300)])
def test_merged_blocks_of_sequences_of_their_own_lengths(lazyev_lib, group, blocks, N):
    """More than eight blocks per unit with per-sequence timing: a full cache, one of fewer sub-tiles than the unit has
    waves, and an empty slot, whose rows of the output stay as they are; launches that fit the chip, and one that does not.  Against
    fp64 softmax attention."""
    H, steps, lens = 2, 3, (N, 70, -1)
    gen = torch.Generator(device="cuda").manual_seed(11)
    eng = lazyev_lib.LazyEviction(1, 3, group * H, H, 128, N + 100, 64, N, 8.0 / N)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    for s, n in enumerate(lens):
        if n < 0:
            eng.retire(s)
        else:
            eng.admit(s, n, 0)
    eng.set_target_blocks(blocks * 3 * H)
    for t in range(1, steps + 1):
        q, kn, vn = (torch.empty((3, h, 128), device="cuda").normal_(generator=gen).to(torch.bfloat16) for h in (group * H, H, H))
        out = torch.full((3, group * H, 128), 7.0, dtype=torch.bfloat16, device="cuda")
        eng.decode_step(0, t, q, kn, vn, out)
        for s, n in enumerate(lens):
            if n < 0:
                assert bool((out[s] == 7.0).all())
                continue
            k, v = eng.k_cache[0, s, :, :n + t].double(), eng.v_cache[0, s, :, :n + t].double()
            p = torch.softmax(torch.matmul(q[s].double().view(H, group, 128), k.transpose(1, 2).contiguous()) / np.sqrt(128.0), dim=-1)
            ref = torch.matmul(p, v).view(group * H, 128)
            err = float(((out[s].double() - ref).norm(dim=1) / ref.norm(dim=1)).max())
            assert err < 2 * 2.0 ** -8, (s, t, err)   # (two roundings to bf16, as above)
    eng.stats()
    eng.close()


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("fp32", 64), ("fp32", 128)])
@pytest.mark.parametrize("batch,blocks,N", [(30, 9, 10500), (30, 10, 11600), (28, 11, 13000), (15, 19, 22500), (18, 32, 10500)])
def test_more_than_eight_blocks_where_the_chip_is_full(lazyev_lib, dtype, d, batch, blocks, N):
    """Units of more than eight blocks in launches of more than two stream blocks per compute unit: the unit's last block merges,
    nine records at a time (fp32 rows of 128: eighteen), a round that is not full, a whole one, one more record, and several.  Outputs
    of sampled sequences against fp64 softmax attention; TS / MRI / pos as with three blocks a unit."""
    H, group, steps = 2, 3, 3
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    states = []
    for b in (3, blocks):
        gen = torch.Generator(device="cuda").manual_seed(13)
        eng = lazyev_lib.LazyEviction(1, batch, group * H, H, d, N + 100, 64, N, 8.0 / N, dtype=dt)
        eng.k_cache[:, :, :, :N].normal_(generator=gen)
        eng.v_cache[:, :, :, :N].normal_(generator=gen)
        eng.init()
        eng.set_target_blocks(b * batch * H)
        out = torch.zeros((batch, group * H, d), dtype=dt, device="cuda")
        for t in range(1, steps + 1):
            q, kn, vn = (torch.empty((batch, h, d), device="cuda").normal_(generator=gen).to(dt) for h in (group * H, H, H))
            eng.decode_step(0, t, q, kn, vn, out)
            for s in (0, batch - 1):
                k, v = eng.k_cache[0, s, :, :N + t].double(), eng.v_cache[0, s, :, :N + t].double()
                p = torch.softmax(torch.matmul(q[s].double().view(H, group, d), k.transpose(1, 2).contiguous()) * d ** -0.5, dim=-1)
                ref = torch.matmul(p, v).view(group * H, d)
                err = float(((out[s].double() - ref).norm(dim=1) / ref.norm(dim=1)).max())
                # (bf16: two roundings, as above; fp32: sums of some thousand terms)
                assert err < (1e-5 if dt == torch.float32 else 2 * 2.0 ** -8), (b, s, t, err)
        eng.stats()
        states.append([x[0, :, :, :N + steps].clone() for x in (eng.ts, eng.mri, eng.pos)])
        eng.close()
    for x, y in zip(*states):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,d,batch,blocks,N", [("fp32", 128, 12, 10, 2000), ("fp32", 128, 9, 13, 2000),
                                                    ("bf16", 128, 10, 12, 13000), ("bf16", 64, 12, 10, 11700), ("fp32", 64, 12, 10, 11700)])
def test_merging_blocks_behind_the_tracking_blocks(lazyev_lib, dtype, d, batch, blocks, N):
    """Launches of more blocks than the chip holds at once, whose merging blocks come last (the first call tracks nothing, so its
    merging blocks come first).  Outputs of sampled sequences against fp64
    softmax attention; TS / MRI / pos and the activations as with three blocks a unit."""
    H, group, steps = 2, 8, 4
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    states = []
    for b in (3, blocks):
        gen = torch.Generator(device="cuda").manual_seed(17)
        eng = lazyev_lib.LazyEviction(1, batch, group * H, H, d, N + 100, 64, N, 8.0 / N, dtype=dt)
        eng.k_cache[:, :, :, :N].normal_(generator=gen)
        eng.v_cache[:, :, :, :N].normal_(generator=gen)
        eng.init()
        eng.set_target_blocks(b * batch * H)
        out = torch.zeros((batch, group * H, d), dtype=dt, device="cuda")
        for t in range(1, steps + 1):
            q, kn, vn = (torch.empty((batch, h, d), device="cuda").normal_(generator=gen).to(dt) for h in (group * H, H, H))
            eng.decode_step(0, t, q, kn, vn, out)
            for s in (0, batch - 1):
                k, v = eng.k_cache[0, s, :, :N + t].double(), eng.v_cache[0, s, :, :N + t].double()
                p = torch.softmax(torch.matmul(q[s].double().view(H, group, d), k.transpose(1, 2).contiguous()) * d ** -0.5, dim=-1)
                ref = torch.matmul(p, v).view(group * H, d)
                err = float(((out[s].double() - ref).norm(dim=1) / ref.norm(dim=1)).max())
                # (bf16: two roundings, as above; fp32: sums of some thousand terms)
                assert err < (1e-5 if dt == torch.float32 else 2 * 2.0 ** -8), (b, s, t, err)
        states.append([eng.stats()["n_activations"]] + [x[0, :, :, :N + steps].clone() for x in (eng.ts, eng.mri, eng.pos)])
        eng.close()
    assert states[0][0] == states[1][0]
    for x, y in zip(states[0][1:], states[1][1:]):
        assert torch.equal(x, y)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("fp32", 64)])
@pytest.mark.parametrize("blocks,N", [(9, 2200), (17, 2200), (33, 2200), (9, 11700)])
def test_merging_blocks_report_a_wait_that_ends(lazyev_lib, dtype, d, blocks, N):
    """Both waits of a merging block, and the one on a single word before them in long runs, with the limit at 0: a block gives
    up as soon as a look finds a record missing.  Every kernel still ends, the next lazyev_stats says so once, and with the
    limit back the outputs are right again (against fp64 softmax attention)."""
    H, group, batch, steps = 2, 4, 2, 12
    dt = torch.float32 if dtype == "fp32" else torch.bfloat16
    gen = torch.Generator(device="cuda").manual_seed(19)
    eng = lazyev_lib.LazyEviction(1, batch, group * H, H, d, N + 100, 64, N, 8.0 / N, dtype=dt)
    eng.k_cache[:, :, :, :N].normal_(generator=gen)
    eng.v_cache[:, :, :, :N].normal_(generator=gen)
    eng.init()
    eng.set_target_blocks(blocks * batch * H)
    out = torch.zeros((batch, group * H, d), dtype=dt, device="cuda")
    eng.set_spin_ticks(0)
    for t in range(1, steps + 1):
        if t == steps - 1:
            torch.cuda.synchronize()
            with pytest.raises(lazyev_lib.LazyevError) as err:
                eng.stats()
            assert err.value.code == lazyev_lib.EEXCHANGE
            eng.set_spin_ticks(2000000)
            assert eng.stats()["len"][0] == N + t - 1        # reported once
        q, kn, vn = (torch.empty((batch, h, d), device="cuda").normal_(generator=gen).to(dt) for h in (group * H, H, H))
        eng.decode_step(0, t, q, kn, vn, out)
        if t >= steps - 1:
            k, v = eng.k_cache[0, :, :, :N + t].double(), eng.v_cache[0, :, :, :N + t].double()
            p = torch.softmax(torch.matmul(q.double().view(batch, H, group, d), k.transpose(2, 3).contiguous()) * d ** -0.5, dim=-1)
            ref = torch.matmul(p, v).view(batch, group * H, d)
            err = float(((out.double() - ref).norm(dim=-1) / ref.norm(dim=-1)).max())
            # (bf16: two roundings, as above; fp32: sums of some thousand terms)
            assert err < (1e-5 if dt == torch.float32 else 2 * 2.0 ** -8), (t, err)
    assert eng.stats()["len"][0] == N + steps
    eng.close()
