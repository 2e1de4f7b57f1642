"""head_dim 64 streaming pass: the two wavefronts of a row group take alternate tiles, two per barrier.  Odd and even tile
counts around the ring's length, ragged last tiles, every row-group count, dense and sparse, against the numpy float64
oracle.  Tolerances: those of bf16 storage (fb_testlib)."""
import pytest

from oracle import flashblock_oracle as orc
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
    w = wl.Workload(f"wts_{P}_{topk}", 2, 16, 8, 64, P, 20, 3, 3, "bf16", 1.0, key_block=key_block, topk=topk)
    Kp, Vp = wl.make_prefix(w, 503)
    steps = wl.make_block_steps(w, 503)
    ora = orc.run_block_sparse(Kp, Vp, steps, 3, key_block, topk)
    for g, o in zip(T.run_sparse_block_gpu(w, Kp, Vp, steps, idx_per_refresh={0: ora[0]["idx"]}, R=3), ora):
        T.assert_close(g["out"], o["out"], "bf16", w.name + " out")
        T.check_partial(g["ext"], o["ext"], "bf16", w.name + " sel(+)res")
        T.check_partial(g["residual"], o["residual"], "bf16", w.name + " residual")
