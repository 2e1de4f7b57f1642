"""Row-pair layouts of the streaming kernel: 32 rows per wavefront and two tiles a trip for streams of 8 to 13 tiles, 64 rows and four
written-out tiles a trip, operands and loads of the next tiles requested inside the present one, from 14 on.  Where their tile
walks can go wrong: streams ending with a whole tile, with one key, with one key missing; every remainder modulo the trip; the
ragged tile first, in the middle and last in the rotated order (several KV heads and splits rotate differently); row counts
around a wavefront's 64 and a workgroup's 256.  Scores spread over many log2 units with planted outliers, so that the reference moves in mid-stream.
Against the numpy float64 oracle, tolerances of bf16 storage (fb_testlib)."""
import numpy as np
import pytest

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T
from test_gpu_large_scores import _inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,n_splits", [
    (4, 2, 128, 512, 65, 1),          # 8 whole tiles; 130 rows: two of the third wavefront
    (4, 2, 128, 513, 96, 1),          # 9 tiles, one key in the last; 192 rows: three whole wavefronts
    (6, 3, 128, 639, 97, 1),          # 10 tiles, one key missing
    (5, 5, 128, 700, 257, 1),         # 11 tiles; one row in the second row tile
    (3, 3, 128, 1100, 256, 2),        # two splits of 9 tiles
    (8, 8, 128, 833, 129, 1),         # 14 tiles, eight rotations
    (2, 2, 64, 577, 1025, 1),         # head_dim 64: 10 tiles, one row in the fifth row tile
    (2, 1, 64, 1023, 600, 2),         # two splits of 8 tiles
])
def test_external_partial(Hq, Hkv, d, P, Bq, n_splits):
    w = wl.Workload(f"rows64_{Hq}_{Hkv}_{d}_{P}_{Bq}", 1, Hq, Hkv, d, P, Bq, 1, 1, "bf16", 1.0)
    print(f"[case] {w.name} n_splits={n_splits}", flush=True)
    Kp, Vp, steps = _inputs(w, 977)
    ora = orc.run_block_dense(Kp, Vp, steps, 1, scale=0.7)
    gpu = T.run_dense_block_gpu(w, Kp, Vp, steps, n_splits=n_splits, scale=0.7)
    assert orc.scores(steps[0][0], Kp, 0.7).std() / np.log(2.0) >= 5.0
    T.check_partial(gpu[0]["ext"], ora[0]["ext"], "bf16", w.name + " ext")
    T.assert_close(gpu[0]["out"], ora[0]["out"], "bf16", w.name + " out")


@pytest.mark.parametrize("Hq,Hkv,d,P,Bq,n_splits", [
    (4, 2, 128, 832, 65, 1),          # 13 whole tiles: the longest of the short layout
    (4, 2, 128, 896, 65, 1),          # 14 whole tiles; 130 rows: two of the third wavefront
    (4, 2, 128, 897, 96, 1),          # 15 tiles, one key in the last; 192 rows: three whole wavefronts
    (6, 3, 128, 1023, 97, 1),         # 16 tiles, one key missing
    (5, 5, 128, 1084, 257, 1),        # 17 tiles; one row in the second row tile
    (3, 3, 128, 1800, 256, 2),        # splits of 15 and 14 tiles
    (8, 8, 128, 1217, 129, 1),        # 20 tiles, eight rotations
    (20, 20, 128, 961, 130, 1),       # 16 tiles, every rotation
    (2, 2, 64, 1027, 1025, 1),        # head_dim 64: 17 tiles, one row in the fifth row tile
    (2, 1, 64, 1919, 600, 2),         # two splits of 15 tiles
])
def test_external_partial_around_14_tiles(Hq, Hkv, d, P, Bq, n_splits):
    test_external_partial(Hq, Hkv, d, P, Bq, n_splits)
