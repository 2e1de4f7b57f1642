"""Many rows per KV head: the one-call refresh step (unsplit as two passes of the row-pair kernel; with splits or short
streams as one register-staged pass and a combine) and the per-head refresh (partials by rank, and by head), at ragged
sizes, against the numpy float64 oracle.  Tolerances: those of bf16 storage (fb_testlib)."""
import numpy as np
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


def _wl(B, Hq, Hkv, d, P, Bq):
    return wl.Workload(f"rp_{B}_{Hq}_{Hkv}_{d}_{P}_{Bq}", B, Hq, Hkv, d, P, Bq, 2, 2, "bf16", 1.0)


@pytest.mark.parametrize("B,Hq,Hkv,d,P,Bq,small_ws", [
    (1, 2, 2, 128, 1025, 129, False),     # 129 rows: one row in the second row tile, one key in the last tile
    (1, 4, 1, 128, 512, 65, False),       # 260 rows of 4 heads, 8 tiles
    (2, 2, 1, 64, 2000, 513, False),      # head_dim 64, 1026 rows
    (1, 2, 2, 128, 511, 200, False),      # 8 tiles, the last one ragged
    (1, 2, 2, 128, 500, 200, True),       # the smallest workspace the call accepts
])
def test_refresh_step_in_passes(B, Hq, Hkv, d, P, Bq, small_ws):
    """With splits: one register-staged pass over prefix and block, and the combine."""
    w = _wl(B, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 401)
    steps = wl.make_block_steps(w, 401)
    ora = orc.run_block_dense(Kp, Vp, steps, 2)
    shape, ext = T.shape_of(w), T.Partial(w)
    ws = T.workspace(shape)
    dev = lambda x: T.to_dev(x, "bf16")
    for t, (Q, Kb, Vb) in enumerate(steps):
        q, out = dev(Q), torch.empty_like(dev(Q))
        lse = torch.empty(q.shape[:3], device=T.DEV)
        if t == 0:
            args = (shape, q, dev(Kp), dev(Vp), dev(Kb), dev(Vb), ext.o, ext.m, ext.lse, out, lse)
            n = ws.numel()
            while small_ws:
                try:
                    fb.fb_refresh_step(*args, ws[:n])
                    n -= 256
                except fb.FlashBlockError as e:
                    assert e.status == fb.FB_ERR_WORKSPACE
                    n += 256
                    break
            fb.fb_refresh_step(*args, ws[:n])
        else:
            fb.fb_internal_merge(shape, q, dev(Kb), dev(Vb), ext.o, ext.m, ext.lse, out, lse)
        torch.cuda.synchronize()
        T.assert_close(out.double().cpu().numpy(), ora[t]["out"], "bf16", f"{w.name} step {t} out")
        T.assert_close(lse.double().cpu().numpy(), ora[t]["lse"], "bf16", f"{w.name} step {t} lse", lse=True)
    T.check_partial(ext.numpy(), ora[0]["ext"], "bf16", w.name + " ext")


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq", [
    (16, 16, 128, 512, 2049),             # 8 tiles; 9 row tiles a head, the last with one row; 33 tiles of the block, one key in the last
    (32, 16, 128, 700, 1030),             # heads straddle row tiles and wavefronts
    (16, 16, 64, 577, 2049),
])
def test_refresh_step_without_splits_is_two_row_pair_passes(Hq, Hkv, d, P, Bq):
    """Many rows per KV head, unsplit: neither pass leaves anything in the workspace (the register-staged pass over prefix and
    block does).  The internal pass of this route walks the block's tiles in rotated order.  Every 13th row is compared."""
    w = _wl(1, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 411)
    steps = wl.make_block_steps(w, 411)
    shape, ext = T.shape_of(w), T.Partial(w)
    assert fb.fb_external_heads_splits(shape, 0) == 1 and Hkv * -(-(Hq // Hkv) * Bq // 256) >= 128 and Bq > 448
    ws = torch.full((fb.fb_workspace_bytes(shape, 0, 0, 1),), 0xA5, device=T.DEV, dtype=torch.uint8)
    events = [torch.cuda.Event(enable_timing=True) for _ in range(3)]
    for e in events:
        e.record()                                        # creates the handle
    want_ext = orc.partial(steps[0][0][:, :, ::13], Kp, Vp)
    for t, (Q, Kb, Vb) in enumerate(steps):
        q, kb, vb = (T.to_dev(x, "bf16") for x in (Q, Kb, Vb))
        out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
        if t == 0:
            fb.fb_refresh_step_prof(shape, q, T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16"), kb, vb, ext.o, ext.m, ext.lse, out, lse,
                                    ws, *(e.cuda_event for e in events))
        else:
            fb.fb_internal_merge(shape, q, kb, vb, ext.o, ext.m, ext.lse, out, lse)
        torch.cuda.synchronize()
        want_out, want_lse = orc.merge(want_ext, orc.partial(Q[:, :, ::13], Kb, Vb))
        T.assert_close(out[:, :, ::13].double().cpu().numpy(), want_out, "bf16", f"{w.name} step {t} out")
        T.assert_close(lse[:, :, ::13].double().cpu().numpy(), np.asarray(want_lse), "bf16", f"{w.name} step {t} lse", lse=True)
    assert bool((ws == 0xA5).all())
    assert 0 < events[0].elapsed_time(events[1]) < events[0].elapsed_time(events[2])
    T.check_partial({k: v[:, :, ::13] for k, v in ext.numpy().items()}, want_ext, "bf16", w.name + " ext")


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,masks,hint", [
    (4, 4, 128, 6200, 2900, [[0, 1, 0, 1], [0, 0, 1, 1]], 2),       # two batch elements, 4 splits, other groups in each
    (4, 4, 128, 6200, 2900, [[0, 1, 1, 1], [0, 0, 0, 1]], 2),       # hint too low in one: its third group runs unsplit
    (16, 4, 128, 6200, 700, [[0] * 4 + [0, 0, 1, 1] + [0] * 4 + [1, 0, 0, 1]], 4),      # wavefronts straddle flagged and other heads
    (4, 4, 64, 9300, 2900, [[0, 1, 1, 1]], 3),                      # 6 splits, an odd tile count per range
])
def test_head_wise_refresh_by_rank(Hq, Hkv, d, P, Bq, masks, hint):
    """Split partials by rank among the flagged KV groups: the first flagged group's are where group 0's would be by head, though
    group 0 is not flagged.  Every 131st row is compared."""
    B = len(masks)
    w = _wl(B, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 413)
    (Q, _, _), _ = wl.make_block_steps(w, 413)
    shape, part, on = T.shape_of(w), T.Partial(w), np.array(masks, dtype=bool)
    assert not on[0, :Hq // Hkv].any()
    part.o.fill_(7), part.m.fill_(8), part.lse.fill_(9)
    n = fb.fb_workspace_bytes(shape, 0, 0, fb.fb_external_heads_splits(shape, hint))
    ws = torch.full((n,), 0xA5, device=T.DEV, dtype=torch.uint8)
    fb.fb_external_partial_heads(shape, T.to_dev(Q, "bf16"), T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16"),
                                 torch.tensor(masks, dtype=torch.uint8, device=T.DEV), part.o, part.m, part.lse, ws, hint)
    torch.cuda.synchronize()
    assert not bool((ws[:Hq // Hkv * Bq * d * 4] == 0xA5).all())
    got, want = {k: v[:, :, ::131] for k, v in part.numpy().items()}, orc.partial(Q[:, :, ::131], Kp, Vp)
    T.check_partial({k: v[on] for k, v in got.items()}, {k: v[on] for k, v in want.items()}, "bf16", w.name)
    assert (got["o"][~on] == 7).all() and (got["m"][~on] == 8).all() and (got["lse"][~on] == 9).all()


@pytest.mark.parametrize("P,Bq,mask,ns,by_rank", [
    (64 * 96, 1287, [0, 1, 1, 1, 1, 1, 0, 0], 4, True),           # 12 tiles per stream, and one tile fewer
    (64 * 95, 1287, [0, 1, 1, 1, 1, 1, 0, 0], 4, False),
    (64 * 300, 260, [0, 0, 0, 0, 0, 1, 0, 0], 11, True),          # 22 workgroups
    (64 * 300, 520, [0, 0, 1, 1, 1, 1, 0, 0], 12, False),         # twice 12 splits of 12 row tiles: a second round
    (64 * 175, 145, [0] * 4 + [1] * 23 + [0] * 5, 6, False),      # four heads to a KV group: the same with 24
    (64 * 192, 128, [0] * 4 + [1] * 23 + [0] * 5, 15, True),      # 16 (8 splits; 15 hold the partials): one round
])
def test_head_wise_refresh_by_rank_or_not(P, Bq, mask, ns, by_rank):
    """Both sides of the rule's lines: by rank the first flagged group's partials stand where group 0's would."""
    w = _wl(1, len(mask), 8, 128, P, Bq)
    print(f"[case] {w.name}", flush=True)
    Kp, Vp = wl.make_prefix(w, 421)
    (Q, _, _), _ = wl.make_block_steps(w, 421)
    shape, part, on = T.shape_of(w), T.Partial(w), np.array([mask], dtype=bool)
    part.o.fill_(7), part.m.fill_(8), part.lse.fill_(9)
    assert fb.fb_external_heads_splits(shape, sum(mask)) == ns
    ws = torch.full((fb.fb_workspace_bytes(shape, 0, 0, ns),), 0xA5, device=T.DEV, dtype=torch.uint8)
    fb.fb_external_partial_heads(shape, *(T.to_dev(x, "bf16") for x in (Q, Kp, Vp)), torch.tensor([mask], dtype=torch.uint8, device=T.DEV),
                                 part.o, part.m, part.lse, ws, sum(mask))
    torch.cuda.synchronize()
    assert bool((ws[:len(mask) // 8 * Bq * 128 * 4] != 0xA5).any()) == by_rank
    got, want = {k: v[:, :, ::131] for k, v in part.numpy().items()}, orc.partial(Q[:, :, ::131], Kp, Vp)
    T.check_partial({k: v[on] for k, v in got.items()}, {k: v[on] for k, v in want.items()}, "bf16", w.name)
    assert (got["o"][~on] == 7).all() and (got["m"][~on] == 8).all() and (got["lse"][~on] == 9).all()


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,mask,hint,step", [
    (8, 2, 128, 3300, 40, [0, 1, 0, 0, 0, 0, 1, 1], 3, 1),      # 160 rows of 4 heads: wavefronts straddle flagged and other heads
    (4, 4, 128, 3300, 300, [0, 0, 1, 0], 1, 1),                 # one head
    (4, 4, 128, 3300, 300, [1, 0, 1, 1], 1, 1),                 # hint too low
    (6, 3, 128, 5000, 90, [0, 0, 0, 1, 1, 0], 2, 1),            # groups 1 and 2 of 3
    (8, 8, 128, 9300, 2080, [1, 0, 1, 1, 0, 0, 1, 1], 5, 41),   # by rank: 3 ranges, 6 splits
    (4, 4, 128, 2100, 300, [0, 0, 1, 0], 1, 1),                 # 33 tiles
    (4, 4, 128, 530, 300, [1, 0, 1, 0], 0, 1),                  # no hint, one split
    (2, 2, 64, 3300, 1030, [0, 1], 1, 7),
])
def test_head_wise_refresh(Hq, Hkv, d, P, Bq, mask, hint, step):
    """Every step-th row is compared with the oracle."""
    w = _wl(1, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 403)
    (Q, _, _), _ = wl.make_block_steps(w, 403)
    shape, part = T.shape_of(w), T.Partial(w)
    part.o.fill_(7), part.m.fill_(8), part.lse.fill_(9)
    hm = torch.tensor([mask], dtype=torch.uint8, device=T.DEV)
    ws = T.workspace(shape, n_splits=fb.fb_external_heads_splits(shape, hint))
    fb.fb_external_partial_heads(shape, T.to_dev(Q, "bf16"), T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16"), hm, part.o, part.m,
                                 part.lse, ws, hint)
    torch.cuda.synchronize()
    got, want = {k: v[:, :, ::step] for k, v in part.numpy().items()}, orc.partial(Q[:, :, ::step], Kp, Vp)
    on = np.array(mask, dtype=bool)
    T.check_partial({k: v[:, on] for k, v in got.items()}, {k: v[:, on] for k, v in want.items()}, "bf16", w.name)
    assert (got["o"][:, ~on] == 7).all() and (got["m"][:, ~on] == 8).all() and (got["lse"][:, ~on] == 9).all()


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,active,ns", [
    (4, 2, 128, 6300, 3300, 2, 2),      # both KV groups flagged: 8 group partials by rank; 2 splits hold 6
    (8, 8, 128, 9300, 2080, 7, 2),      # 28 and 24
    (8, 8, 128, 9300, 2080, 5, 3),      # 30 and 32: they fit
])
def test_head_wise_refresh_does_not_depend_on_the_workspace(Hq, Hkv, d, P, Bq, active, ns):
    """The documented workspace and a larger one: the same result bit for bit.  One for the pass's ns splits is taken too."""
    w = _wl(1, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 405)
    (Q, _, _), _ = wl.make_block_steps(w, 405)
    shape = T.shape_of(w)
    q, kp, vp = (T.to_dev(x, "bf16") for x in (Q, Kp, Vp))
    hm = torch.tensor([[0] * (Hq - active) + [1] * active], dtype=torch.uint8, device=T.DEV)
    documented = fb.fb_workspace_bytes(shape, 0, 0, fb.fb_external_heads_splits(shape, active))
    by_rank = (2 * ns * min(active, Hkv)) * (Hq // Hkv) * Bq * (d + 2) * 4
    assert documented >= by_rank and documented >= fb.fb_workspace_bytes(shape, 0, 0, ns)
    got = []
    for n in (documented, 4 * documented, fb.fb_workspace_bytes(shape, 0, 0, ns)):
        part = T.Partial(w)
        part.o.zero_(), part.m.zero_(), part.lse.zero_()
        fb.fb_external_partial_heads(shape, q, kp, vp, hm, part.o, part.m, part.lse,
                                     torch.empty(n, device=T.DEV, dtype=torch.uint8), active)
        torch.cuda.synchronize()
        got.append(part)
    for a, b in zip((got[0].o, got[0].m, got[0].lse), (got[1].o, got[1].m, got[1].lse)):
        assert torch.equal(a, b)
    on, step = slice(Hq - active, Hq), 131
    want = {k: v[:, on] for k, v in orc.partial(Q[:, :, ::step], Kp, Vp).items()}
    for part in got:
        T.check_partial({k: v[:, on, ::step] for k, v in part.numpy().items()}, want, "bf16", w.name)


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,mask", [
    (8, 8, 128, 3000, 1000, [0, 0, 0, 0, 0, 1, 0, 0]),       # 47 tiles, 8 row tiles: 5 splits of 9 or 10 tiles
    (4, 4, 128, 3000, 1000, [1, 0, 1, 1]),                   # 11 splits, as without a hint
    (8, 4, 64, 2000, 64, [0, 0, 1, 1, 0, 0, 0, 0]),          # 128 rows, one KV group
    (4, 4, 128, 130, 200, [0, 1, 0, 0]),                     # three tiles: one split
    (4, 4, 128, 1000, 200, [0, 1, 0, 0]),                    # 16 tiles: the least that is split
])
def test_hint_on_a_short_stream(Hq, Hkv, d, P, Bq, mask):
    """With the hint no fewer splits than without, from 16 tiles on; the documented workspace and the smallest one that is accepted."""
    w = _wl(1, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 407)
    (Q, _, _), _ = wl.make_block_steps(w, 407)
    shape, hint, on = T.shape_of(w), sum(mask), np.array(mask, dtype=bool)
    ns = fb.fb_external_heads_splits(shape, hint)
    assert ns >= (fb.fb_external_heads_splits(shape, 0) if P >= 1000 else 1)
    hm = torch.tensor([mask], dtype=torch.uint8, device=T.DEV)
    want = {k: v[:, on] for k, v in orc.partial(Q[:, :, ::17], Kp, Vp).items()}
    for size in (fb.fb_workspace_bytes(shape, 0, 0, ns), fb.fb_workspace_bytes(shape, 0, 0, 1)):
        part = T.Partial(w)
        fb.fb_external_partial_heads(shape, T.to_dev(Q, "bf16"), T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16"), hm, part.o, part.m,
                                     part.lse, torch.empty(size, device=T.DEV, dtype=torch.uint8), hint)
        torch.cuda.synchronize()
        T.check_partial({k: v[:, on, ::17] for k, v in part.numpy().items()}, want, "bf16", f"{w.name} {size}")


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq", [
    (36, 18, 128, 600, 960),              # a block of 15 whole tiles: register-staged internal pass
    (32, 16, 128, 900, 961),              # 16 tiles, one key in the last: the streaming kernel, its prefix pass as well (15 tiles)
    (32, 16, 64, 600, 1024),
])
def test_internal_pass_around_16_tiles(Hq, Hkv, d, P, Bq):
    test_refresh_step_without_splits_is_two_row_pair_passes(Hq, Hkv, d, P, Bq)


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,masks,hint,step", [
    # 260 rows of 4 heads: the flagged ones' fill one row tile, a part of it, two (all four heads)
    (32, 8, 128, 36000, 65, ["0000", "1000", "0001", "0101", "1111", "0010", "1101", "0000"], 8, 7),
    # 320 rows of 8 heads: every other head; all but one (280 rows: 24 in the second tile); the last head alone
    (32, 4, 128, 74000, 40, ["00000000", "01010101", "11111011", "00000001"], 4, 7),
    (16, 2, 64, 49000, 140, ["00000000", "10010110"], 2, 31),
    (16, 4, 128, 19000, 700, ["0000", "0101", "1000", "0110"], 2, 61),      # hint too low: the third flagged group unsplit, with gaps
])
def test_head_wise_refresh_by_rank_with_gaps(Hq, Hkv, d, P, Bq, masks, hint, step):
    """Several query heads per KV head, some of them flagged: row tiles are cut from the flagged heads' rows.  Every step-th row is
    compared; no row of another head is written, in the workspace either."""
    w = _wl(1, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 419)
    (Q, _, _), _ = wl.make_block_steps(w, 419)
    on = np.array([[int(c) for c in "".join(masks)]], dtype=bool)
    shape, part, G = T.shape_of(w), T.Partial(w), Hq // Hkv
    part.o.fill_(7), part.m.fill_(8), part.lse.fill_(9)
    n = fb.fb_workspace_bytes(shape, 0, 0, fb.fb_external_heads_splits(shape, hint))
    ws = torch.full((n,), 0xA5, device=T.DEV, dtype=torch.uint8)
    fb.fb_external_partial_heads(shape, T.to_dev(Q, "bf16"), T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16"),
                                 torch.from_numpy(on.astype(np.uint8)).to(T.DEV), part.o, part.m, part.lse, ws, hint)
    torch.cuda.synchronize()
    # the first flagged group's partials of the first split stand at the beginning of the workspace, by row of the group
    rank0 = (ws[:G * Bq * d * 4].view(G, Bq * d * 4) != 0xA5).any(1).cpu().numpy()
    first = next(m for m in masks if "1" in m)
    assert rank0.tolist() == [c == "1" for c in first]
    got, want = {k: v[:, :, ::step] for k, v in part.numpy().items()}, orc.partial(Q[:, :, ::step], Kp, Vp)
    T.check_partial({k: v[on] for k, v in got.items()}, {k: v[on] for k, v in want.items()}, "bf16", w.name)
    assert (got["o"][~on] == 7).all() and (got["m"][~on] == 8).all() and (got["lse"][~on] == 9).all()
