"""Single fp32 products on both sides of the row count from which they are made of bf16 parts (64-row workgroups): one column of a query
against a key and against the same key rounded to bf16, so that the two weights' ratio is the difference of two large scores."""
import numpy as np
import pytest
import torch

from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


def _bf16(x):
    return torch.from_numpy(x).to(torch.bfloat16).float().numpy()


def _factors(rng, n):
    """In [1, 2): half of them anywhere, half with the lowest bits that the upper and middle of three parts leave as large as can be."""
    anywhere = 1 + rng.integers(0, 1 << 23, n) / (1 << 23)
    ties = 1 + rng.integers(0, 4, n) / 128 + (254.5 - rng.integers(0, 4, n)) / 32768
    return np.where(rng.integers(0, 2, n) == 0, anywhere, ties).astype(np.float32)


@pytest.mark.parametrize("B,Bq", [(2, 80), (32, 80), (11, 336)])           # 16- and 64-row workgroups; head_dim 64: parts in the last
@pytest.mark.parametrize("d", [64, 128])
def test_score_products_lose_no_more_than_fp32_rounding(B, Bq, d):
    """A score of one product is off by its rounding to fp32 (2^-24 of it) and, in parts, by the cross terms left out (2^-24 again; the
    rounded key has no lower parts and so none of these): the difference of the two is within 3 x 2^-24 of the score.  The sums of
    the small terms, whose roundings are 2^-8 of that, and the weights (exponents below 12, so 1e-6) come on top."""
    w = wl.Workload(f"sp_{B}_{Bq}_{d}", B, 8, 4, d, 0, Bq, 1, 1, "f32", 1.0)
    print(f"[case] {w.name}", flush=True)
    rng = np.random.default_rng(371)
    Q, K, V = (np.zeros((B, h, Bq, d), np.float32) for h in (8, 4, 4))
    Q[..., 0] = 64 * _factors(rng, B * 8 * Bq).reshape(B, 8, Bq)
    Q[..., 1] = 1.0
    K[..., 1] = -65536.0 * 16                                # all other keys: far below
    exact, rounded = 70, 5
    K[:, :, exact, 0] = 64 * _factors(rng, B * 4).reshape(B, 4)
    K[:, :, rounded, 0] = _bf16(K[:, :, exact, 0].copy())
    K[:, :, [exact, rounded], 1] = 0.0
    V[:, :, exact, 2] = V[:, :, rounded, 3] = 1.0
    q = T.to_dev(Q, "f32")
    out = torch.empty_like(q)
    fb.fb_internal_merge(T.shape_of(w), q, T.to_dev(K, "f32"), T.to_dev(V, "f32"), None, None, None, out, None)
    got = out.double().cpu().numpy()
    got = np.log(got[..., 2]) - np.log(got[..., 3])
    pair = K[:, np.arange(8) // 2][:, :, [exact, rounded], 0].astype(np.float64)         # [B, 8, 2]
    scores = Q[..., :1].astype(np.float64) * pair[:, :, None] * d ** -0.5               # [B, 8, Bq, 2]
    want = scores[..., 0] - scores[..., 1]
    bound = scores.max(-1) * (3 + 0.1) * 2.0 ** -24 + 2e-6
    over = np.abs(got - want) / bound
    worst, rows = float(over.max()), int((over > 1).sum())
    assert worst <= 1, f"{worst:.2f} times the bound, {rows} of {over.size} rows"
