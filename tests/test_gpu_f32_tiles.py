"""The fp32 pass at the edges of its workgroup tiles (16, 32 and 64 group-flattened rows, 64-key tiles in quarters of 16,
split counts above the tile count) against the numpy float64 oracle.  Tolerance: the 1e-5 max-abs of fp32 storage."""
import numpy as np
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


def _wl(B, Hq, Hkv, d, P, Bq, S=2, R=2, **kw):
    return wl.Workload(f"f32_{B}_{Hq}_{Hkv}_{d}_{P}_{Bq}", B, Hq, Hkv, d, P, Bq, S, R, "f32", 1.0, **kw)


@pytest.mark.parametrize("B,Hq,Hkv,d,P,Bq,n_splits", [
    (1, 1, 1, 64, 1, 1, 0),          # one row, one key
    (1, 2, 2, 128, 15, 16, 0),       # one whole row block, keys of one quarter only (one missing)
    (1, 2, 1, 64, 17, 8, 0),         # 16 rows of two heads, second quarter holds one key
    (1, 3, 1, 128, 48, 11, 0),       # 33 rows: 64-row tile with one row in its third block
    (2, 4, 2, 64, 64, 16, 0),        # 32-row tile, exactly one key tile
    (1, 4, 2, 128, 130, 9, 9),       # 18 rows, more splits than tiles
    (1, 4, 1, 64, 129, 16, 2),       # 64 rows, one key in the last tile
    (1, 5, 1, 128, 200, 13, 3),      # 65 rows: a second row tile with one row
    (1, 8, 1, 64, 1000, 33, 1),      # 264 rows, one split: the kernel writes the final partial
])
def test_row_and_key_tile_edges(B, Hq, Hkv, d, P, Bq, n_splits):
    w = _wl(B, Hq, Hkv, d, P, Bq)
    print(f"[case] {w.name} n_splits={n_splits}", flush=True)
    Kp, Vp = wl.make_prefix(w, 301)
    steps = wl.make_block_steps(w, 301)
    ora = orc.run_block_dense(Kp, Vp, steps, 2)
    for g, o in zip(T.run_dense_block_gpu(w, Kp, Vp, steps, R=2, n_splits=n_splits), ora):
        T.assert_close(g["out"], o["out"], "f32", w.name + " out")
        T.assert_close(g["lse"], o["lse"], "f32", w.name + " lse", lse=True)
        T.check_partial(g["ext"], o["ext"], "f32", w.name + " ext")
    # the fused pass: the block's own keys are one more workgroup
    shape, ext = T.shape_of(w), T.Partial(w)
    Q, Kb, Vb = steps[0]
    q = T.to_dev(Q, "f32")
    out = torch.empty_like(q)
    fb.fb_refresh_step(shape, q, T.to_dev(Kp, "f32"), T.to_dev(Vp, "f32"), T.to_dev(Kb, "f32"), T.to_dev(Vb, "f32"),
                       ext.o, ext.m, ext.lse, out, None, T.workspace(shape))
    torch.cuda.synchronize()
    T.assert_close(out.double().cpu().numpy(), ora[0]["out"], "f32", w.name + " refresh_step out")
    T.check_partial(ext.numpy(), ora[0]["ext"], "f32", w.name + " refresh_step ext")


def test_internal_pass_with_64_row_workgroups():
    """Enough workgroups for the 64-row form of the internal pass (256 of them, 65 rows each)."""
    w = _wl(32, 20, 4, 64, 0, 13, S=1)
    (Q, Kb, Vb), = wl.make_block_steps(w, 303)
    q = T.to_dev(Q, "f32")
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
    fb.fb_internal_merge(T.shape_of(w), q, T.to_dev(Kb, "f32"), T.to_dev(Vb, "f32"), None, None, None, out, lse)
    torch.cuda.synchronize()
    part = orc.partial(Q, Kb, Vb)
    T.assert_close(out.double().cpu().numpy(), orc.normalized(part), "f32", "internal out")
    T.assert_close(lse.double().cpu().numpy(), part["lse"], "f32", "internal lse", lse=True)


@pytest.mark.parametrize("ext", ["none", "empty", "partial"])
@pytest.mark.parametrize("B,Hq,Hkv,d,Bq", [
    (1, 1, 1, 64, 1), (1, 3, 1, 128, 1), (2, 6, 2, 64, 4), (1, 8, 2, 128, 8), (1, 4, 4, 128, 15), (1, 4, 2, 64, 16), (1, 3, 3, 128, 16),
    (1, 4, 2, 128, 17),                                              # one key too many for a wavefront per row
    (16, 32, 1, 64, 8), (17, 32, 1, 64, 8), (40, 32, 8, 64, 8),      # 4096 rows; 4352 of one KV head, and of 8 with 32 each
])
def test_internal_pass_over_few_keys(B, Hq, Hkv, d, Bq, ext):
    P = 0 if ext == "empty" else 70
    w = _wl(B, Hq, Hkv, d, P, Bq, S=1)
    Kp, Vp = wl.make_prefix(w, 311)
    (Q, Kb, Vb), = wl.make_block_steps(w, 311)
    shape, part = T.shape_of(w), T.Partial(w)
    q, parts = T.to_dev(Q, "f32"), (None, None, None)
    inn = orc.partial(Q, Kb, Vb)
    want_out, want_lse = orc.normalized(inn), inn["lse"]
    if ext != "none":
        kp, vp = (T.to_dev(Kp, "f32"), T.to_dev(Vp, "f32")) if P else (None, None)
        fb.fb_external_partial(shape, q, kp, vp, part.o, part.m, part.lse, T.workspace(shape))
        parts = (part.o, part.m, part.lse)
        want_out, want_lse = orc.merge(orc.partial(Q, Kp, Vp), inn)
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
    fb.fb_internal_merge(shape, q, T.to_dev(Kb, "f32"), T.to_dev(Vb, "f32"), *parts, out, lse)
    torch.cuda.synchronize()
    T.assert_close(out.double().cpu().numpy(), want_out, "f32", w.name + " out")
    T.assert_close(lse.double().cpu().numpy(), np.asarray(want_lse), "f32", w.name + " lse", lse=True)


@pytest.mark.parametrize("P", [1, 3, 15, 16, 17])
@pytest.mark.parametrize("Hq,Hkv,d,Bq", [(1, 1, 64, 1), (6, 2, 128, 13), (4, 4, 64, 70)])
def test_prefix_of_few_keys(Hq, Hkv, d, Bq, P):
    w = _wl(2, Hq, Hkv, d, P, Bq, S=1, R=1)
    Kp, Vp = wl.make_prefix(w, 313)
    (Q, _, _), = wl.make_block_steps(w, 313)
    shape, part = T.shape_of(w), T.Partial(w)
    fb.fb_external_partial(shape, T.to_dev(Q, "f32"), T.to_dev(Kp, "f32"), T.to_dev(Vp, "f32"), part.o, part.m, part.lse,
                           T.workspace(shape))
    torch.cuda.synchronize()
    T.check_partial(part.numpy(), orc.partial(Q, Kp, Vp), "f32", w.name)


def test_few_keys_with_an_infinite_last_value():
    """The last key's value row is infinite and its weight is not 0: infinities, and no NaN, where the row is added."""
    w = _wl(1, 2, 1, 64, 0, 5, S=1)
    (Q, Kb, Vb), = wl.make_block_steps(w, 315)
    Vb[..., -1, :] = np.inf
    q = T.to_dev(Q, "f32")
    out = torch.empty_like(q)
    fb.fb_internal_merge(T.shape_of(w), q, T.to_dev(Kb, "f32"), T.to_dev(Vb, "f32"), None, None, None, out, None)
    torch.cuda.synchronize()
    assert bool(torch.isposinf(out).all())


@pytest.mark.parametrize("Bq", [7, 20, 40])
def test_unselected_key_blocks_are_never_touched(Bq):
    """Sparse reuse: an infinity in a key block that another head of the group selected leaves this head's rows alone."""
    w = _wl(1, 4, 2, 128, 320, Bq, key_block=64, topk=1)
    Kp, Vp = wl.make_prefix(w, 305)
    (Q, _, _), _ = wl.make_block_steps(w, 305)
    Vp[0, :, 64:128] = np.inf                                        # block 1, selected by heads 0 and 2 only
    idx = torch.tensor([[[1], [3], [1], [4]]], device=T.DEV, dtype=torch.int32)
    shape, res, ext = T.shape_of(w), T.Partial(w), T.Partial(w)
    res.o.zero_(), res.m.fill_(-np.inf), res.lse.fill_(-np.inf)
    fb.fb_sparse_external_residual(shape, fb.FB_SPARSE_REUSE, T.to_dev(Q, "f32"), T.to_dev(Kp, "f32"), T.to_dev(Vp, "f32"),
                                   64, 1, idx, res.o, res.m, res.lse, ext.o, ext.m, ext.lse, T.workspace(shape, 64, 1))
    torch.cuda.synchronize()
    got = ext.numpy()
    for h, blk in ((1, 3), (3, 4)):
        keys = slice(64 * blk, 64 * blk + 64)
        want = orc.partial(Q[:, h:h + 1], Kp[:, h // 2:h // 2 + 1, keys], Vp[:, h // 2:h // 2 + 1, keys])
        T.check_partial({k: v[:, h:h + 1] for k, v in got.items()}, want, "f32", f"head {h}")


@pytest.mark.parametrize("d,P,Bq,key_block,topk", [
    (128, 700, 20, 64, 4), (128, 1029, 40, 128, 3),       # 32-row workgroups, one and two to a head
    (64, 700, 20, 64, 4), (64, 1029, 40, 128, 3),         # 32 and 64 rows
    (128, 257, 65, 64, 5), (64, 257, 65, 64, 0),          # three row tiles (two), all and none of the key blocks selected
])
def test_sparse_refresh_and_reuse(d, P, Bq, key_block, topk):
    w = _wl(2, 4, 2, d, P, Bq, key_block=key_block, topk=topk)
    print(f"[case] {w.name} key_block={key_block} topk={topk}", flush=True)
    Kp, Vp = wl.make_prefix(w, 307)
    steps = wl.make_block_steps(w, 307)
    ora = orc.run_block_sparse(Kp, Vp, steps, 2, key_block, topk)
    idx = {0: ora[0]["idx"]} if topk else None
    for g, o in zip(T.run_sparse_block_gpu(w, Kp, Vp, steps, idx_per_refresh=idx, R=2), ora):
        T.assert_close(g["out"], o["out"], "f32", w.name + " out")
        T.check_partial(g["ext"], o["ext"], "f32", w.name + " sel(+)res")
        T.check_partial(g["residual"], o["residual"], "f32", w.name + " residual")


@pytest.mark.parametrize("d,P,Bq,mask", [
    (128, 700, 10, [0, 1, 1, 0]), (128, 700, 20, [1, 0, 0, 0]), (64, 1029, 40, [0, 1, 0, 1]), (128, 1029, 40, [1, 1, 0, 1]),
    (64, 65, 65, [0, 0, 0, 1]),
])
def test_head_wise_refresh(d, P, Bq, mask):
    w = _wl(2, 4, 2, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 309)
    (Q, _, _), _ = wl.make_block_steps(w, 309)
    shape, part = T.shape_of(w), T.Partial(w)
    part.o.fill_(7), part.m.fill_(8), part.lse.fill_(9)
    on = np.array([mask, mask[::-1]], dtype=bool)                    # another choice per batch element
    ns = fb.fb_external_heads_splits(shape, sum(mask))
    fb.fb_external_partial_heads(shape, T.to_dev(Q, "f32"), T.to_dev(Kp, "f32"), T.to_dev(Vp, "f32"),
                                 torch.from_numpy(on.astype(np.uint8)).to(T.DEV), part.o, part.m, part.lse,
                                 T.workspace(shape, n_splits=ns), sum(mask))
    torch.cuda.synchronize()
    got, want = part.numpy(), orc.partial(Q, Kp, Vp)
    T.check_partial({k: v[on] for k, v in got.items()}, {k: v[on] for k, v in want.items()}, "f32", w.name)
    assert (got["o"][~on] == 7).all() and (got["m"][~on] == 8).all() and (got["lse"][~on] == 9).all()
