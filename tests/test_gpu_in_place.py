"""A step whose output takes the place of its queries (out is q) gives what it gives with a buffer of its own, on every kernel
that writes `out`.  Both are compared with the numpy float64 oracle; tolerances: those of the storage type (fb_testlib)."""
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,B,Hq,Hkv,d,P,Bq", [
    ("bf16", 1, 32, 8, 128, 70, 32),      # few rows, one tile: one wavefront per 32 rows x 32 columns, were it not in place
    ("bf16", 1, 8, 2, 64, 70, 16),
    ("bf16", 1, 3, 3, 128, 70, 64),
    ("bf16", 12, 16, 8, 128, 70, 31),     # more of them than that kernel takes
    ("bf16", 70, 4, 2, 64, 70, 40),       # 128-row workgroups, each row in one wavefront
    ("bf16", 1, 16, 16, 128, 70, 449),    # beyond one tile
    ("bf16", 6, 16, 8, 128, 4000, 31),    # refresh step: splits folded by the internal pass
    ("bf16", 1, 32, 8, 128, 4200, 32),    # refresh step: one kernel folds, attends and merges
    ("bf16", 3, 8, 8, 128, 64 * 88, 5),   # refresh step: pieces, and the same kernel over a block of odd length
    ("bf16", 1, 8, 8, 128, 64 * 60, 700), # refresh step by streams of even and odd tiles; reuse step in two streams
    ("bf16", 3, 24, 8, 64, 64 * 216, 43), # by streams: fold kernel
    ("bf16", 9, 24, 8, 128, 64 * 28, 43), # by streams: combine and internal pass
    ("f32", 1, 4, 4, 64, 256, 16),
    ("f32", 1, 3, 1, 128, 70, 25),
])
def test_output_in_the_queries_place(dtype, B, Hq, Hkv, d, P, Bq):
    w = wl.Workload(f"ip_{dtype}_{B}_{Hq}_{d}_{P}_{Bq}", B, Hq, Hkv, d, P, Bq, 1, 1, dtype, 1.0)
    print(f"[case] {w.name}", flush=True)
    Kp, Vp = wl.make_prefix(w, 701)
    steps = wl.make_block_steps(w, 701)
    (want,) = orc.run_block_dense(Kp, Vp, steps, 1)
    shape, ext, ws = T.shape_of(w), T.Partial(w), T.workspace(T.shape_of(w))
    q, kb, vb = (T.to_dev(x, dtype) for x in steps[0])
    kp, vp = T.to_dev(Kp, dtype), T.to_dev(Vp, dtype)
    apart, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
    for step in ("refresh", "reuse"):
        for out in (apart, q.clone()):
            src = q if out is apart else out
            if step == "refresh":
                fb.fb_refresh_step(shape, src, kp, vp, kb, vb, ext.o, ext.m, ext.lse, out, lse, ws)
            else:
                fb.fb_internal_merge(shape, src, kb, vb, ext.o, ext.m, ext.lse, out, lse)
            torch.cuda.synchronize()
            T.assert_close(out.double().cpu().numpy(), want["out"], dtype, f"{w.name} {step} out")
            T.assert_close(lse.double().cpu().numpy(), want["lse"], dtype, f"{w.name} {step} lse", lse=True)
        T.check_partial(ext.numpy(), want["ext"], dtype, f"{w.name} {step} ext")
