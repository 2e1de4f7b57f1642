"""The one-wavefront-per-workgroup internal pass (few rows, at most 64 keys) at its edges, against the numpy float64 oracle:
key counts around its 16- and 32-key steps, row remainders, both head dims, with an external partial, with an empty one and
without; and the sizes on both sides of the rule that selects it.  Tolerances: those of bf16 storage (fb_testlib)."""
import numpy as np
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext", ["none", "empty", "partial"])
@pytest.mark.parametrize("B,Hq,Hkv,d,Bq", [
    (1, 1, 1, 64, 1), (1, 3, 1, 128, 11), (2, 4, 2, 128, 15), (1, 8, 2, 64, 16), (1, 4, 4, 128, 17), (1, 2, 1, 64, 31),
    (1, 8, 2, 128, 32), (1, 2, 2, 128, 33), (1, 3, 1, 64, 63), (1, 4, 2, 128, 64),
    (4, 32, 8, 128, 32), (5, 32, 8, 128, 32), (1, 32, 8, 128, 61), (1, 40, 8, 128, 61),      # 512 / 640 and 256 / 320 wavefronts
])
def test_internal_pass(B, Hq, Hkv, d, Bq, ext):
    P = 0 if ext == "empty" else 70
    w = wl.Workload(f"iw_{B}_{Hq}_{d}_{Bq}", B, Hq, Hkv, d, P, Bq, 1, 1, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 601)
    (Q, Kb, Vb), = wl.make_block_steps(w, 601)
    shape, part = T.shape_of(w), T.Partial(w)
    q = T.to_dev(Q, "bf16")
    parts = (None, None, None)
    want_out, want_lse = (lambda p: (orc.normalized(p), p["lse"]))(orc.partial(Q, Kb, Vb))
    if ext != "none":
        kp, vp = (T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16")) if P else (None, None)
        fb.fb_external_partial(shape, q, kp, vp, part.o, part.m, part.lse, T.workspace(shape))
        parts = (part.o, part.m, part.lse)
        want_out, want_lse = orc.merge(orc.partial(Q, Kp, Vp), orc.partial(Q, Kb, Vb))
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
    fb.fb_internal_merge(shape, q, T.to_dev(Kb, "bf16"), T.to_dev(Vb, "bf16"), *parts, out, lse)
    torch.cuda.synchronize()
    T.assert_close(out.double().cpu().numpy(), want_out, "bf16", w.name + " out")
    T.assert_close(lse.double().cpu().numpy(), np.asarray(want_lse), "bf16", w.name + " lse", lse=True)
