"""fp32 storage, short: the one-wavefront internal pass over 17 to 64 keys (edges of its 16-key groups, of its 16-row blocks, with and
without a cached partial, with infinities in the last key's values) and the refresh step in one launch (prefix of no, one, several
and ragged tiles; the largest stream it takes and one tile more), against the numpy float64 oracle at the fp32 tolerances of
fb_testlib."""
import numpy as np
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


def _wl(B, Hq, Hkv, d, P, Bq):
    return wl.Workload(f"f32s_{B}_{Hq}_{Hkv}_{d}_{P}_{Bq}", B, Hq, Hkv, d, P, Bq, 2, 2, "f32", 1.0)


@pytest.mark.parametrize("B,Hq,Hkv,d,P,Bq", [
    (1, 2, 1, 128, 70, 17),       # one key in the second 16-key group; 34 rows: two in the third block
    (1, 3, 3, 128, 64, 32),       # two whole groups, two whole row blocks a head
    (2, 2, 2, 64, 40, 33),        # one key in the third group
    (1, 4, 2, 64, 130, 48),
    (1, 2, 2, 128, 129, 49),      # one key in the fourth group
    (1, 1, 1, 64, 65, 64),
    (1, 4, 4, 64, 0, 16),         # empty prefix: nothing but the block
    (1, 4, 4, 64, 256, 16),       # 4 + 1 tiles, the most at head_dim 64
    (1, 4, 4, 64, 257, 16),       # one more: splits
    (1, 2, 2, 128, 128, 20),      # 2 + 1 tiles
    (1, 2, 2, 128, 1, 70),        # a prefix of one key, a block of two tiles
])
def test_block(B, Hq, Hkv, d, P, Bq):
    """A refresh step in one call, then a reuse step."""
    w = _wl(B, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 611)
    steps = wl.make_block_steps(w, 611)
    ora = orc.run_block_dense(Kp, Vp, steps, 2)
    shape, ext = T.shape_of(w), T.Partial(w)
    ws = T.workspace(shape)
    dev = lambda x: T.to_dev(x, "f32")
    for t, (Q, Kb, Vb) in enumerate(steps):
        q, out = dev(Q), torch.empty_like(dev(Q))
        lse = torch.empty(q.shape[:3], device=T.DEV)
        if t == 0:
            fb.fb_refresh_step(shape, q, dev(Kp) if P else None, dev(Vp) if P else None, dev(Kb), dev(Vb), ext.o, ext.m, ext.lse, out, lse, ws)
        else:
            fb.fb_internal_merge(shape, q, dev(Kb), dev(Vb), ext.o, ext.m, ext.lse, out, lse)
        torch.cuda.synchronize()
        T.assert_close(out.double().cpu().numpy(), ora[t]["out"], "f32", f"{w.name} step {t} out")
        T.assert_close(lse.double().cpu().numpy(), ora[t]["lse"], "f32", f"{w.name} step {t} lse", lse=True)
    T.check_partial(ext.numpy(), ora[0]["ext"], "f32", w.name + " ext")


@pytest.mark.parametrize("Bq", [17, 40, 63])
def test_internal_pass_without_partial_and_with_infinite_values(Bq):
    """No cached partial; and a last key whose values are infinite: rows past the end are copies of it and must not add to it (an
    infinity times a weight of 0 would be NaN in every column)."""
    w = _wl(1, 2, 2, 128, 64, Bq)
    (Q, Kb, Vb), _ = wl.make_block_steps(w, 612)
    Vb = Vb.copy()
    Vb[0, 0, -1, :64] = np.inf
    q, k, v = (T.to_dev(x, "f32") for x in (Q, Kb, Vb))
    out = torch.empty_like(q)
    fb.fb_internal_merge(T.shape_of(w), q, k, v, None, None, None, out, None)
    torch.cuda.synchronize()
    got = out.double().cpu().numpy()
    assert np.isposinf(got[0, 0, :, :64]).all()
    s = np.einsum("hqd,hkd->hqk", Q[0].astype(np.float64), Kb[0].astype(np.float64)) / np.sqrt(128)
    p = np.exp(s - s.max(-1, keepdims=True))
    p /= p.sum(-1, keepdims=True)
    want = np.einsum("hqk,hkd->hqd", p, np.where(np.isinf(Vb[0]), 0.0, Vb[0]).astype(np.float64))
    assert np.abs(got[0, 1] - want[1]).max() <= 1e-5 and np.abs(got[0, 0, :, 64:] - want[0, :, 64:]).max() <= 1e-5


@pytest.mark.parametrize("n,d", [(3, 64), (4, 128), (7, 64), (13, 128), (16, 64), (16, 128)])
def test_one_denominator_per_row(n, d):
    """At most 16 keys (one wavefront per row): every key's value row is one number repeated, so all columns of an output row are the
    same sum over the same denominator and have to be equal bit for bit, with and without a cached partial, which is constant
    over the columns as well."""
    B, H, Bq = 4, 8, n
    g = torch.Generator(device=T.DEV)
    g.manual_seed(613 + n + d)
    normal = lambda *s: torch.randn(s, generator=g, device=T.DEV)
    q, k = normal(B, H, Bq, d), normal(B, H, Bq, d)
    v, eo = (normal(B, H, Bq, 1).expand(B, H, Bq, d).contiguous() for _ in range(2))
    em = normal(B, H, Bq)
    shape = fb.make_shape(B, H, H, d, Bq, 64, "f32")
    for ext in ((None, None, None), (eo, em, em + 1)):
        out = torch.empty_like(q)
        fb.fb_internal_merge(shape, q, k, v, *ext, out, None)
        torch.cuda.synchronize()
        uneven = (out != out[..., :1]).any(-1).sum().item()
        assert uneven == 0, f"{uneven} of {B * H * Bq} rows"


@pytest.mark.parametrize("B,Hq,Hkv,d,P,Bq,one", [
    (1, 2, 2, 128, 64, 20, True),         # 2 tiles
    (1, 2, 2, 128, 128, 20, False),       # 3 tiles, 4 workgroups of 16 rows
    (4, 8, 8, 128, 128, 49, True),        # 3 tiles, 128 workgroups
    (2, 8, 8, 128, 64, 100, True),        # a block of two tiles, 112 workgroups
    (4, 8, 8, 128, 129, 49, False),       # 4 tiles
    (4, 4, 4, 64, 200, 70, False),        # head_dim 64: 6 tiles
    (2, 8, 2, 64, 190, 70, True),         # 5 tiles
])
def test_refresh_step_in_one_launch(B, Hq, Hkv, d, P, Bq, one):
    """One launch leaves the workspace alone, the splits and their combine do not; both against the oracle."""
    w = _wl(B, Hq, Hkv, d, P, Bq)
    Kp, Vp = wl.make_prefix(w, 615)
    steps = wl.make_block_steps(w, 615)
    ora = orc.run_block_dense(Kp, Vp, steps, 2)
    shape, ext, dev = T.shape_of(w), T.Partial(w), lambda x: T.to_dev(x, "f32")
    ws = torch.full((fb.fb_workspace_bytes(shape),), 0xA5, device=T.DEV, dtype=torch.uint8)
    Q, Kb, Vb = steps[0]
    q, out = dev(Q), torch.empty_like(dev(Q))
    fb.fb_refresh_step(shape, q, dev(Kp), dev(Vp), dev(Kb), dev(Vb), ext.o, ext.m, ext.lse, out, None, ws)
    torch.cuda.synchronize()
    assert bool((ws == 0xA5).all()) == one
    T.assert_close(out.double().cpu().numpy(), ora[0]["out"], "f32", f"{w.name} out")
    T.check_partial(ext.numpy(), ora[0]["ext"], "f32", w.name + " ext")
