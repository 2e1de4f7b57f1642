"""Routes of the many-row (row-pair) streaming kernel: the one-call refresh step as passes and the per-head refresh, at
ragged sizes, against the numpy float64 oracle.  Tolerances: those of bf16 storage (fb_testlib)."""
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
    (1, 2, 2, 128, 1025, 129, False),     # 129 rows: the smallest row-pair group, one key past the tile, two splits
    (1, 4, 1, 128, 512, 65, False),       # 260 rows, 8 tiles: one split, the pass writes the partial itself
    (2, 2, 1, 64, 2000, 513, False),      # head_dim 64 from 1024 rows on
    (1, 2, 2, 128, 511, 200, False),      # 8 tiles, the last one ragged
    (1, 2, 2, 128, 500, 200, True),       # the smallest workspace the call accepts
])
def test_refresh_step_in_passes(B, Hq, Hkv, d, P, Bq, small_ws):
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


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,mask,hint,step", [
    (8, 2, 128, 3300, 40, [0, 1, 0, 0, 0, 0, 1, 1], 3, 1),      # 160 rows of 4 heads: wavefronts straddle flagged and other heads
    (4, 4, 128, 3300, 300, [0, 0, 1, 0], 1, 1),                 # one head, its even and its odd tiles
    (4, 4, 128, 3300, 300, [1, 0, 1, 1], 1, 1),                 # hint too low: the groups beyond it run unsplit
    (6, 3, 128, 5000, 90, [0, 0, 0, 1, 1, 0], 2, 1),            # partials of groups 1 and 2 in the slots of the first two
    (8, 8, 128, 9300, 2080, [1, 0, 1, 1, 0, 0, 1, 1], 5, 41),   # 3 ranges, 6 splits, an odd tile count per range
    (4, 4, 128, 2100, 300, [0, 0, 1, 0], 1, 1),                 # too few tiles: 128-row workgroups, as without a hint
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
    (4, 4, 128, 130, 200, [0, 1, 0, 0]),                     # three tiles
])
def test_hint_on_a_short_stream(Hq, Hkv, d, P, Bq, mask):
    """With the hint no fewer splits than without; the documented workspace and the smallest one that is accepted."""
    w = _wl(1, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 407)
    (Q, _, _), _ = wl.make_block_steps(w, 407)
    shape, hint, on = T.shape_of(w), sum(mask), np.array(mask, dtype=bool)
    ns = fb.fb_external_heads_splits(shape, hint)
    assert ns >= fb.fb_external_heads_splits(shape, 0)
    hm = torch.tensor([mask], dtype=torch.uint8, device=T.DEV)
    want = {k: v[:, on] for k, v in orc.partial(Q[:, :, ::17], Kp, Vp).items()}
    for size in (fb.fb_workspace_bytes(shape, 0, 0, ns), fb.fb_workspace_bytes(shape, 0, 0, 1)):
        part = T.Partial(w)
        fb.fb_external_partial_heads(shape, T.to_dev(Q, "bf16"), T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16"), hm, part.o, part.m,
                                     part.lse, torch.empty(size, device=T.DEV, dtype=torch.uint8), hint)
        torch.cuda.synchronize()
        T.check_partial({k: v[:, on, ::17] for k, v in part.numpy().items()}, want, "bf16", f"{w.name} {size}")
