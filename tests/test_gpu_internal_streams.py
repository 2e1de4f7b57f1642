"""Internal pass in two streams of tiles per row group (1, 2 and 4 row groups of 32 rows a workgroup), around the tile counts and
workgroup counts where the rule takes it: against the numpy float64 oracle, with and without a cached partial, into the queries' place."""
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,Bq", [
    (1, 2, 2, 193),          # one row group: 4 tiles, the last of one key
    (1, 4, 2, 320),          # 5 whole tiles, an odd number of them
    (2, 2, 1, 700),          # 11 tiles, ragged
    (1, 8, 8, 1024),         # 256 workgroups of one row group
    (1, 8, 8, 1025),         # two row groups
    (1, 64, 16, 130),        # 520 rows per KV head, 3 tiles: two row groups (head_dim 128)
    (1, 30, 30, 321),        # two row groups, 6 tiles
    (3, 20, 20, 385),        # four row groups, 7 tiles
])
def test_internal_streams(B, Hq, Hkv, Bq, d):
    w = wl.Workload(f"is_{B}_{Hq}_{Bq}_{d}", B, Hq, Hkv, d, 64, Bq, 2, 2, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 701)
    steps = wl.make_block_steps(w, 701)
    want = orc.run_block_dense(Kp, Vp, steps, 2)
    shape, ext, ws, k, v = T.shape_of(w), T.Partial(w), T.workspace(T.shape_of(w)), T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16")
    q0 = T.to_dev(steps[0][0], "bf16")
    fb.fb_external_partial(shape, q0, k, v, ext.o, ext.m, ext.lse, ws)
    q, kb, vb = (T.to_dev(x, "bf16") for x in steps[1])
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
    fb.fb_internal_merge(shape, q, kb, vb, ext.o, ext.m, ext.lse, out, lse)
    T.assert_close(out.double().cpu().numpy(), want[1]["out"], "bf16", w.name + " out")
    T.assert_close(lse.double().cpu().numpy(), want[1]["lse"], "bf16", w.name + " lse", lse=True)
    inner = torch.empty_like(q)
    fb.fb_internal_merge(shape, q, kb, vb, None, None, None, inner)
    T.assert_close(inner.double().cpu().numpy(), orc.normalized(want[1]["int"]), "bf16", w.name + " without a cached partial")
    fb.fb_internal_merge(shape, q, kb, vb, ext.o, ext.m, ext.lse, q)
    assert torch.equal(q, out)
