"""fp32 passes over keys and values that hold infinities, on both sides of the row count from which the products are made of bf16 parts
(64-row workgroups: more than 32 rows and enough workgroups; head_dim 64 from four tiles a workgroup on, from six in the internal pass).  A key whose score is -inf for a row is left out of it; an infinite value
makes its own column infinite and no other.  Against the numpy float64 oracle without those keys and with a finite value there."""
import numpy as np
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu

COLUMN = 5                                # of the infinite value


def _inputs(w, seed, at, drop):
    """Keys `drop` score -inf in every row (columns 0 and 1 of the queries are negative and positive), value `at` is infinite."""
    Kp, Vp = wl.make_prefix(w, seed)
    Q, Kb, Vb = wl.make_block_steps(w, seed)[0]
    Q[..., 0], Q[..., 1] = -np.abs(Q[..., 0]) - 0.25, np.abs(Q[..., 1]) + 0.25
    K, V = (Kp, Vp) if w.prefix_len else (Kb, Vb)
    kept = [i for i in range(K.shape[2]) if i not in drop]
    plain = K[:, :, kept].copy(), V[:, :, kept].copy()
    for n, i in enumerate(drop):
        K[:, :, i, n % 2] = np.inf if n % 2 == 0 else -np.inf
    V[:, :, at, COLUMN] = np.inf
    return Q, Kp, Vp, Kb, Vb, plain


def _check(a, want, what):
    assert np.isposinf(a[..., COLUMN]).all(), f"{what}: the infinite value's column"
    a, want = np.delete(a, COLUMN, -1), np.delete(want, COLUMN, -1)
    T.assert_close(a, want, "f32", what)


def _normalized(part):
    return part["o"] * np.exp(part["m"] - part["lse"])[..., None]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Bq,n_splits", [(1, 32, 200), (1, 33, 200), (2, 50, 200), (1, 40, 129), (2, 50, 65)])
def test_external_pass(Hq, Bq, n_splits, d):
    w = wl.Workload(f"if_{Hq}_{Bq}_{d}", 1, Hq, 1, d, 64 * 201 + 9, Bq, 1, 1, "f32", 1.0)
    print(f"[case] {w.name}", flush=True)
    Q, Kp, Vp, _, _, (K, V) = _inputs(w, 351, 70, [3, 64 * 100, 64 * 201 + 8])
    shape, ext = T.shape_of(w), T.Partial(w)
    fb.fb_external_partial_ex(shape, *(T.to_dev(x, "f32") for x in (Q, Kp, Vp)), ext.o, ext.m, ext.lse, n_splits,
                              T.workspace(shape, n_splits=n_splits))
    got, want = ext.numpy(), orc.partial(Q, K, V)
    T.assert_close(got["lse"], want["lse"], "f32", w.name + " lse", lse=True)
    _check(_normalized(got), orc.normalized(want), w.name)


@pytest.mark.parametrize("Bq", [8, 32])                     # 32 and 128 rows per KV head
def test_refresh_step(Bq):
    w = wl.Workload(f"ir_{Bq}", 1, 32, 8, 128, 4111, Bq, 1, 1, "f32", 1.0)
    print(f"[case] {w.name}", flush=True)
    Q, Kp, Vp, Kb, Vb, (K, V) = _inputs(w, 353, 4110, [0, 2000])
    shape, ext = T.shape_of(w), T.Partial(w)
    q, kp, vp, kb, vb = (T.to_dev(x, "f32") for x in (Q, Kp, Vp, Kb, Vb))
    out = torch.empty_like(q)
    fb.fb_refresh_step(shape, q, kp, vp, kb, vb, ext.o, ext.m, ext.lse, out, None, T.workspace(shape))
    part = orc.partial(Q, K, V)
    got = ext.numpy()
    T.assert_close(got["lse"], part["lse"], "f32", w.name + " lse", lse=True)
    _check(_normalized(got), orc.normalized(part), w.name + " ext")
    _check(out.double().cpu().numpy(), orc.merge(part, orc.partial(Q, Kb, Vb))[0], w.name + " out")


@pytest.mark.parametrize("B,Bq", [(2, 80), (32, 80), (11, 336)])           # 16- and 64-row workgroups, these without parts and with
def test_internal_pass(B, Bq):
    w = wl.Workload(f"ii_{B}_{Bq}", B, 8, 4, 64, 0, Bq, 1, 1, "f32", 1.0)
    print(f"[case] {w.name}", flush=True)
    Q, _, _, Kb, Vb, (K, V) = _inputs(w, 355, 79, [10, 64])
    q = T.to_dev(Q, "f32")
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
    fb.fb_internal_merge(T.shape_of(w), q, T.to_dev(Kb, "f32"), T.to_dev(Vb, "f32"), None, None, None, out, lse)
    part = orc.partial(Q, K, V)
    T.assert_close(lse.double().cpu().numpy(), part["lse"], "f32", w.name + " lse", lse=True)
    _check(out.double().cpu().numpy(), orc.normalized(part), w.name)


@pytest.mark.parametrize("Bq", [20, 40])                    # 32- and 64-row workgroups, one query head each
def test_sparse_refresh(Bq):
    """The infinite value is among the selected keys: the residual partial stays finite."""
    w = wl.Workload(f"is_{Bq}", 4, 8, 4, 64, 64 * 40 + 9, Bq, 1, 1, "f32", 1.0, key_block=64, topk=2)
    print(f"[case] {w.name}", flush=True)
    Q, Kp, Vp, _, _, (K, V) = _inputs(w, 357, 70, [5, 64 * 30])
    shape, res, ext = T.shape_of(w), T.Partial(w), T.Partial(w)
    idx = torch.tensor([1, 17], device=T.DEV, dtype=torch.int32).expand(4, 8, 2).contiguous()
    fb.fb_sparse_external_residual(shape, fb.FB_SPARSE_REFRESH, T.to_dev(Q, "f32"), T.to_dev(Kp, "f32"), T.to_dev(Vp, "f32"), 64, 2, idx,
                                   res.o, res.m, res.lse, ext.o, ext.m, ext.lse, T.workspace(shape, 64, 2))
    got, want = ext.numpy(), orc.partial(Q, K, V)
    T.assert_close(got["lse"], want["lse"], "f32", w.name + " lse", lse=True)
    _check(_normalized(got), orc.normalized(want), w.name)
    unselected = [i for i in range(w.prefix_len) if i // 64 not in (1, 17) and i not in (5, 64 * 30)]
    T.check_partial(res.numpy(), orc.partial(Q, Kp[:, :, unselected], Vp[:, :, unselected]), "f32", w.name + " residual")


def test_heads_and_paged_passes():
    """The other two forms of the pass, 64-row workgroups."""
    w = wl.Workload("ih", 8, 8, 8, 64, 64 * 40, 40, 1, 1, "f32", 1.0)
    print(f"[case] {w.name}", flush=True)
    Q, Kp, Vp, _, _, (K, V) = _inputs(w, 359, 70, [5, 64 * 30])
    want = orc.partial(Q, K, V)
    shape = T.shape_of(w)
    q, kp, vp = (T.to_dev(x, "f32") for x in (Q, Kp, Vp))
    tables = torch.arange(8 * 40, device=T.DEV, dtype=torch.int32).reshape(8, 40)
    pools = [x.reshape(8, 8, 40, 64, 64).transpose(1, 2).reshape(320, 8, 64, 64).contiguous() for x in (kp, vp)]
    lens = torch.full((8,), w.prefix_len, device=T.DEV, dtype=torch.int32)
    kv = fb.make_paged_kv(*pools, tables, lens)
    for form in ("heads", "paged"):
        ext, ws = T.Partial(w), T.workspace(shape, n_splits=8)
        if form == "heads":
            fb.fb_external_partial_heads(shape, q, kp, vp, torch.ones(8, 8, device=T.DEV, dtype=torch.uint8), ext.o, ext.m, ext.lse, ws, 0)
        else:
            fb.fb_external_partial_paged(shape, q, kv, ext.o, ext.m, ext.lse, ws, n_splits=8)
        got = ext.numpy()
        T.assert_close(got["lse"], want["lse"], "f32", form + " lse", lse=True)
        _check(_normalized(got), orc.normalized(want), form)
