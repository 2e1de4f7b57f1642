"""fb_select_topk: the form with a workspace (mean queries and block scores spread over the chip, in one kernel where a KV group has
few rows and at most eight heads, else in two) selects what the one-kernel form without a workspace does, index by index; and both
equal numpy's choice on scores that are exact in fp32 (small integers), with many ties, at the edges of the 256-thread passes."""
import numpy as np
import pytest
import torch

from paper_2602_05305_amd import flashblock as fb

import fb_testlib as T

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,Hq,Hkv,d,Bq,nblk,topk,dtype", [
    (1, 32, 8, 128, 32, 1024, 256, "bf16"),
    (2, 16, 2, 128, 33, 257, 100, "bf16"),      # eight heads a group, three rows a thread
    (1, 8, 1, 64, 64, 256, 256, "bf16"),        # 512 rows, the most; everything selected
    (1, 8, 1, 64, 65, 255, 1, "bf16"),          # one row more: two kernels
    (1, 9, 1, 128, 4, 300, 17, "bf16"),         # nine heads: two kernels
    (1, 4, 4, 128, 1, 1, 1, "bf16"),
    (1, 4, 2, 128, 32, 77, 30, "f32"),          # four rows a thread
    (1, 4, 2, 128, 41, 77, 30, "f32"),          # five: two kernels
    (2, 6, 2, 64, 7, 700, 300, "f32"),
])
def test_selection(B, Hq, Hkv, d, Bq, nblk, topk, dtype):
    rng = np.random.default_rng([B, Hq, Bq, nblk])
    # every row of a head different, small integers whose column sums are multiples of the row count (the last row makes up for
    # the rest, at most Bq - 1 <= 64 and so exact in bf16): means, products and sums are small integers
    q = rng.integers(-2, 3, (B, Hq, 1, d)) + rng.integers(-2, 3, (B, Hq, Bq, d))
    q[:, :, -1] -= q.sum(2) % Bq
    mean = q.sum(2) // Bq
    q = q.astype(np.float64)
    kp = rng.integers(-1, 2, (B, Hkv, nblk, d)).astype(np.float64)
    kp[:, :, :, 8:] = 0                          # few distinct scores
    shape = fb.make_shape(B, Hq, Hkv, d, Bq, nblk * 64, dtype)
    qt, kt = T.to_dev(q, dtype), torch.from_numpy(kp).float().to(T.DEV)
    ws = torch.empty(fb.fb_select_workspace_bytes(shape, 64), device=T.DEV, dtype=torch.uint8)
    got = []
    for w in (ws, None):
        sel = torch.full((B, Hq, topk), -7, device=T.DEV, dtype=torch.int32)
        fb.fb_select_topk(shape, qt, kt, 64, topk, sel, w)
        torch.cuda.synchronize()
        got.append(sel.cpu().numpy())
    assert (got[0] == got[1]).all()
    k = min(topk, nblk)
    for b in range(B):
        for h in range(Hq):
            score = kp[b, h // (Hq // Hkv)] @ mean[b, h]
            want = np.sort(np.lexsort((np.arange(nblk), -score))[:k])
            assert (got[0][b, h, :k] == want).all() and (got[0][b, h, k:] == -1).all()
