"""Streaming passes that take two tiles per barrier: at head_dim 64, where each of the two wavefronts of a row group has one key
half of both (dense, sparse), and the refresh step with few splits, where each has one whole tile and the internal pass folds
the splits.  Odd and even tile counts around the ring's length, ragged last tiles, every row-group count, against the numpy
float64 oracle.  Tolerances: those of bf16 storage (fb_testlib)."""
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Bq", [4, 12, 25])                 # 16, 48, 100 rows per KV group: 1, 2, 4 row groups
@pytest.mark.parametrize("P,n_splits", [(64 * 8, 1), (64 * 8 + 1, 1), (64 * 10, 1), (64 * 11 - 63, 1), (64 * 17 + 5, 2)])
def test_dense(P, n_splits, Bq):
    w = wl.Workload(f"wt_{P}_{Bq}", 1, 8, 2, 64, P, Bq, 2, 2, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 501)
    steps = wl.make_block_steps(w, 501)
    ora = orc.run_block_dense(Kp, Vp, steps, 2)
    for g, o in zip(T.run_dense_block_gpu(w, Kp, Vp, steps, R=2, n_splits=n_splits), ora):
        T.assert_close(g["out"], o["out"], "bf16", w.name + " out")
        T.check_partial(g["ext"], o["ext"], "bf16", w.name + " ext")


@pytest.mark.parametrize("P,key_block,topk", [(64 * 32, 64, 9), (64 * 33 + 7, 128, 3), (64 * 41, 64, 40)])
def test_sparse(P, key_block, topk):
    """Fewer than 8 tiles per split: the register-staged kernel."""
    w = wl.Workload(f"wts_{P}_{topk}", 2, 16, 8, 64, P, 20, 3, 3, "bf16", 1.0, key_block=key_block, topk=topk)
    Kp, Vp = wl.make_prefix(w, 503)
    steps = wl.make_block_steps(w, 503)
    ora = orc.run_block_sparse(Kp, Vp, steps, 3, key_block, topk)
    for g, o in zip(T.run_sparse_block_gpu(w, Kp, Vp, steps, idx_per_refresh={0: ora[0]["idx"]}, R=3), ora):
        T.assert_close(g["out"], o["out"], "bf16", w.name + " out")
        T.check_partial(g["ext"], o["ext"], "bf16", w.name + " sel(+)res")
        T.check_partial(g["residual"], o["residual"], "bf16", w.name + " residual")


@pytest.mark.parametrize("G,Bq", [(1, 5), (2, 21), (3, 33)])       # 5, 42, 99 rows: 1, 2, 4 row groups
@pytest.mark.parametrize("P,key_block,topk", [
    (64 * 9 + 7, 64, 4),             # 10 tiles in one split: one tile per barrier
    (64 * 9 + 7, 128, 3),
    (64 * 24, 64, 7),                # from 24 tiles per split on: two
    (64 * 25 + 7, 128, 9),
    (128 * 12 + 30, 128, 11),        # the last key block's second tile lies past the end: an entry of the reuse list without keys
])
def test_sparse_streams(P, key_block, topk, G, Bq):
    B, Hkv = 16, 16                  # 256 KV groups: unsplit, at least 8 tiles per workgroup
    w = wl.Workload(f"wtl_{P}_{topk}_{G}", B, Hkv * G, Hkv, 64, P, Bq, 2, 2, "bf16", 1.0, key_block=key_block, topk=topk)
    Kp, Vp = wl.make_prefix(w, 507)
    steps = wl.make_block_steps(w, 507)
    ora = orc.run_block_sparse(Kp, Vp, steps, 2, key_block, topk)
    for g, o in zip(T.run_sparse_block_gpu(w, Kp, Vp, steps, idx_per_refresh={0: ora[0]["idx"]}, R=2), ora):
        T.assert_close(g["out"], o["out"], "bf16", w.name + " out")
        T.check_partial(g["ext"], o["ext"], "bf16", w.name + " sel(+)res")
        T.check_partial(g["residual"], o["residual"], "bf16", w.name + " residual")


@pytest.mark.parametrize("B,Hq,Hkv,d,P,Bq", [
    (6, 16, 8, 128, 2700, 31),       # 10 splits: one register-staged pass and a combine
    (6, 16, 8, 128, 4000, 31),       # 62 rows per KV head, 6 splits folded by the internal pass
    (16, 8, 4, 128, 3000, 9),        # 18 rows
    (10, 8, 4, 128, 4100, 64),       # 128 rows, a block of one whole tile
    (16, 8, 4, 64, 9000, 24),        # head_dim 64, one round of workgroups, fewer than 44 tiles per split
    (16, 8, 4, 64, 12000, 24),       # more
    (16, 8, 4, 64, 12100, 33),       # a block of two 32-key tiles
    (20, 8, 4, 64, 9100, 33),        # more than one round, more than 32 tiles
    (40, 8, 4, 128, 700, 40),        # too short for the streaming kernel
])
def test_refresh_step_with_few_splits(B, Hq, Hkv, d, P, Bq):
    """Folded by the internal pass: no partial of the block's own keys goes through the workspace (its place, behind the splits',
    stays as it was)."""
    w = wl.Workload(f"fs_{B}_{d}_{P}_{Bq}", B, Hq, Hkv, d, P, Bq, 2, 2, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 505)
    steps = wl.make_block_steps(w, 505)
    ora = orc.run_block_dense(Kp, Vp, steps, 2)
    shape, ext, ws = T.shape_of(w), T.Partial(w), T.workspace(T.shape_of(w)).fill_(0xA5)
    kp, vp = T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16")
    for t, step in enumerate(steps):
        q, kb, vb = (T.to_dev(x, "bf16") for x in step)
        out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
        if t == 0:
            fb.fb_refresh_step(shape, q, kp, vp, kb, vb, ext.o, ext.m, ext.lse, out, lse, ws)
        else:
            fb.fb_internal_merge(shape, q, kb, vb, ext.o, ext.m, ext.lse, out, lse)
        torch.cuda.synchronize()
        T.assert_close(out.double().cpu().numpy(), ora[t]["out"], "bf16", f"{w.name} step {t} out")
        T.assert_close(lse.double().cpu().numpy(), ora[t]["lse"], "bf16", f"{w.name} step {t} lse", lse=True)
    rows, ns = B * Hq * Bq, fb.fb_external_heads_splits(shape, 0)
    behind = ns * rows * d * 4 + 2 * 256 * -(-ns * rows * 4 // 256)
    assert bool((ws[behind:behind + rows * d * 4] == 0xA5).all()) == (P not in (2700, 9000, 12100, 700))
    T.check_partial(ext.numpy(), ora[0]["ext"], "bf16", w.name + " ext")
