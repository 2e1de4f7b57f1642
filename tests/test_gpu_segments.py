"""Dense passes whose workgroups take even pieces of a walk through reference segments (24 KV groups: 10 pieces of 11 segments), and the
fold kernel over blocks that are no multiple of its four rows: against the same pass with one workgroup per segment, and against
the numpy float64 oracle."""
import pytest
import torch

from oracle import flashblock_oracle as orc
from paper_2602_05305_amd import flashblock as fb
from paper_2602_05305_amd import workloads as wl

import fb_testlib as T

pytestmark = pytest.mark.gpu


def _normalised(e):
    return e.o.double() * (e.m - e.lse).double().exp()[..., None]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,G,Bq,P", [
    (3, 1, 8, 64 * 88),              # the shortest segments: 8 tiles
    (3, 2, 31, 64 * 97 - 31),        # 62 rows, a ragged last tile with one key for the second key half
    (3, 4, 25, 64 * 163 + 5),        # 100 rows, segments of 14 and 15 tiles
    (5, 1, 32, 64 * 131 + 40),       # 40 groups: 6 pieces of 7 segments
])
def test_pieces_keep_the_segments_references(B, G, Bq, P, d):
    """Weights are rounded against the same references, so the two ways differ by fp32 sums only: 1e-5 of the RMS, where another
    reference moves single values by some 1e-2 of it."""
    w = wl.Workload(f"sg_{B}_{G}_{P}_{d}", B, 8 * G, 8, d, P, Bq, 1, 1, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 601)
    q = T.to_dev(wl.make_block_steps(w, 601)[0][0], "bf16")
    k, v = T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16")
    shape, pieces, segments = T.shape_of(w), T.Partial(w), T.Partial(w)
    nseg = -(-256 // (8 * B))
    assert fb.fb_external_splits(shape) == 256 // (8 * B) == nseg - 1
    fb.fb_external_partial(shape, q, k, v, pieces.o, pieces.m, pieces.lse, T.workspace(shape))
    fb.fb_external_partial_ex(shape, q, k, v, segments.o, segments.m, segments.lse, nseg, T.workspace(shape, n_splits=nseg))
    a, b = _normalised(pieces), _normalised(segments)
    assert float((a - b).abs().max()) <= 1e-5 * float(b.square().mean().sqrt())
    assert float((pieces.lse - segments.lse).abs().max()) <= 2e-6 * max(1.0, float(segments.lse.abs().max()))


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("G,Bq,P", [(1, 1, 64 * 88), (4, 3, 64 * 90 + 1), (2, 33, 64 * 91 - 1), (4, 31, 64 * 109 + 7), (1, 63, 64 * 93)])
def test_refresh_step_of_odd_blocks(G, Bq, P, d):
    w = wl.Workload(f"so_{G}_{Bq}_{P}_{d}", 3, 8 * G, 8, d, P, Bq, 2, 2, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 603)
    steps = wl.make_block_steps(w, 603)
    shape, ext = T.shape_of(w), T.Partial(w)
    ws, k, v = T.workspace(shape), T.to_dev(Kp, "bf16"), T.to_dev(Vp, "bf16")
    for (Q, Kb, Vb), want in zip(steps, orc.run_block_dense(Kp, Vp, steps, 2)):
        q, kb, vb = (T.to_dev(x, "bf16") for x in (Q, Kb, Vb))
        out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
        if Q is steps[0][0]:
            fb.fb_refresh_step(shape, q, k, v, kb, vb, ext.o, ext.m, ext.lse, out, lse, ws)
        else:
            fb.fb_internal_merge(shape, q, kb, vb, ext.o, ext.m, ext.lse, out, lse)
        T.assert_close(out.double().cpu().numpy(), want["out"], "bf16", w.name + " out")
        T.check_partial(ext.numpy(), want["ext"], "bf16", w.name + " ext")


def test_workspace_sized_by_the_split_count():
    """fb_external_splits is the number of pieces; what it sizes holds the passes that ask for a partial per segment."""
    w = wl.Workload("sw", 3, 8, 8, 128, 64 * 88, 9, 1, 1, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 607)
    step = wl.make_block_steps(w, 607)[0]
    want = orc.run_block_dense(Kp, Vp, [step], 1)[0]
    q, kb, vb, k, v = (T.to_dev(x, "bf16") for x in (*step, Kp, Vp))
    shape, ext, out = T.shape_of(w), T.Partial(w), torch.empty_like(q)
    ws = T.workspace(shape, n_splits=fb.fb_external_splits(shape))
    fb.fb_external_partial(shape, q, k, v, ext.o, ext.m, ext.lse, ws)
    T.check_partial(ext.numpy(), want["ext"], "bf16", "external")
    fb.fb_refresh_step(shape, q, k, v, kb, vb, ext.o, ext.m, ext.lse, out, None, ws)
    T.check_partial(ext.numpy(), want["ext"], "bf16", "step ext")
    T.assert_close(out.double().cpu().numpy(), want["out"], "bf16", "step out")


@pytest.mark.parametrize("factor", [2.0, 8.0])
@pytest.mark.parametrize("Bq", [8, 5])
def test_references_that_move_between_segments(Bq, factor):
    """Some keys outweigh the others by 30 or 130 powers of two for one row: the next segment's reference lies as far below, and what a
    workgroup that walks on has accumulated is scaled up (or, farther apart than 32, its reference stays)."""
    w = wl.Workload(f"sm_{Bq}_{factor}", 3, 8, 8, 128, 64 * 88, Bq, 1, 1, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 605)
    steps = wl.make_block_steps(w, 605)
    for at in range(7, w.prefix_len, 64 * 8 + 11):
        Kp[:, :, at] = wl.round_storage(factor * steps[0][0][:, :, 1], "bf16")
    shape, ext = T.shape_of(w), T.Partial(w)
    q, kb, vb, k, v = (T.to_dev(x, "bf16") for x in (*steps[0], Kp, Vp))
    want = orc.run_block_dense(Kp, Vp, steps, 1)[0]
    fb.fb_external_partial(shape, q, k, v, ext.o, ext.m, ext.lse, T.workspace(shape))
    T.check_partial(ext.numpy(), want["ext"], "bf16", w.name + " ext")
    out = torch.empty_like(q)
    fb.fb_refresh_step(shape, q, k, v, kb, vb, ext.o, ext.m, ext.lse, out, None, T.workspace(shape))
    T.assert_close(out.double().cpu().numpy(), want["out"], "bf16", w.name + " out")
    T.check_partial(ext.numpy(), want["ext"], "bf16", w.name + " ext of the step")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("factor", [2.0, 3.0, 4.0, 4.5])
def test_similarity_of_partials_whose_reference_moved_down(factor, d):
    """One tile outweighs all others, for every row by another 25 to 75 powers of two, and a workgroup that has passed it walks into
    the next segment: what it leaves can be squared and summed in fp32, and is what one workgroup per segment leaves, up to fp32 sums."""
    w = wl.Workload(f"sd_{factor}_{d}", 3, 8, 8, d, 64 * 88, 8, 1, 1, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 613)
    (Q, _, _), = wl.make_block_steps(w, 613)
    for r in range(8):
        Kp[:, :, 64 * 35 + 7 * r] = wl.round_storage(factor * (128 / d) ** 0.5 * Q[:, :, r], "bf16")
    q, k, v = (T.to_dev(x, "bf16") for x in (Q, Kp, Vp))
    shape, pieces, segments = T.shape_of(w), T.Partial(w), T.Partial(w)
    fb.fb_external_partial(shape, q, k, v, pieces.o, pieces.m, pieces.lse, T.workspace(shape))
    fb.fb_external_partial_ex(shape, q, k, v, segments.o, segments.m, segments.lse, 11, T.workspace(shape, n_splits=11))
    a, b = _normalised(pieces), _normalised(segments)
    # (m and lse of either are rounded to 2^-24 of themselves, and enter the normalised row through e^(m - lse))
    bound = 1e-5 * b.square().mean().sqrt() + b.abs() * segments.lse.double().abs()[..., None] * 2.0 ** -22
    assert bool(((a - b).abs() <= bound).all()), float(((a - b).abs() - bound).max())
    for left, right in ((pieces, pieces), (pieces, segments)):
        sim = torch.empty(3, 8, device=T.DEV)
        fb.fb_head_similarity(shape, left.o, right.o, sim)
        assert float((sim - 1).abs().max()) <= 1e-5, f"{sim}"


@pytest.mark.parametrize("B,Hq,Hkv,d,P,Bq", [
    (1, 8, 8, 128, 64 * 60, 700),        # 6 splits of 10 tiles, the least; the block's 11 tiles in two streams
    (1, 8, 8, 64, 64 * 71 + 9, 641),     # a ragged last tile, a block of one row more than whole tiles
    (1, 12, 6, 128, 64 * 97 - 1, 650),   # 1300 rows per KV head, 5 splits
    (1, 1, 1, 128, 64 * 52 * 14, 640),   # 104 streams of few rows: the combine takes a workgroup per row
    (1, 2, 2, 64, 64 * 22 * 20 + 1, 700),
    (9, 24, 8, 128, 64 * 30 + 3, 43),    # 129 rows, 2 splits: combine and internal pass
    (4, 24, 8, 64, 64 * 144 + 31, 43),   # 4 splits, more than 4096 rows: the same
    (3, 24, 8, 64, 64 * 216 + 5, 43),    # 6 splits, 3096 rows: fold kernel
    (3, 24, 8, 128, 64 * 216 - 9, 43),
])
def test_refresh_step_in_streams_of_even_and_odd_tiles(B, Hq, Hkv, d, P, Bq):
    """More than 128 rows per KV head in several splits; a workspace without room for the streams gets the former route."""
    w = wl.Workload(f"st_{B}_{Hq}_{d}_{P}", B, Hq, Hkv, d, P, Bq, 1, 1, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 609)
    step = wl.make_block_steps(w, 609)[0]
    want = orc.run_block_dense(Kp, Vp, [step], 1)[0]
    q, kb, vb, k, v = (T.to_dev(x, "bf16") for x in (*step, Kp, Vp))
    shape = T.shape_of(w)
    ns = -(-256 // (B * Hkv * -(-(Hq // Hkv * Bq) // 128)))
    rows = B * Hq * Bq
    full, small = (sum(-(-n * rows * x * 4 // 256) * 256 for n in sets for x in (d, 1, 1)) + 256 for sets in ((2 * ns, 2), (ns, 1)))
    assert fb.fb_workspace_bytes(shape) == full, "not the route of this test"
    results, outs = [], []
    for size in (fb.fb_workspace_bytes(shape), small):
        ext, ws = T.Partial(w), torch.zeros(size, device=T.DEV, dtype=torch.uint8)
        out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
        fb.fb_refresh_step(shape, q, k, v, kb, vb, ext.o, ext.m, ext.lse, out, lse, ws)
        T.assert_close(out.double().cpu().numpy(), want["out"], "bf16", w.name + " out")
        T.assert_close(lse.double().cpu().numpy(), want["lse"], "bf16", w.name + " lse", lse=True)
        T.check_partial(ext.numpy(), want["ext"], "bf16", w.name + " ext")
        results.append(_normalised(ext))
        outs.append(out.double())
        # partials are written beyond where a route of one stream a split would put them, or not
        written = int(ws.nonzero().max()) + 1
        assert written > small if size == full else written <= small
    # the same references: fp32 sums only
    assert float((results[0] - results[1]).abs().max()) <= 1e-5 * float(results[1].square().mean().sqrt())
    # and the merged output rounded to bf16 (one step of it where a sum falls on the other side of a boundary, 2^-7 at most), or with the
    # block's weights rounded to bf16 on one route and not on the other, 2^-9 each
    assert float((outs[0] - outs[1]).abs().max()) <= 2.0 ** -7 * float(outs[1].abs().max())


@pytest.mark.parametrize("B,Hq,Hkv,d,P,Bq", [
    (1, 4, 4, 128, 64 * 512 + 5, 8),     # 64 splits: two rows a workgroup
    (3, 1, 1, 64, 64 * 688, 5),          # 85 pieces, two rows a workgroup, a block of odd length
    (3, 2, 1, 128, 64 * 688 + 1, 5),     # 85 pieces, one row
    (1, 2, 2, 128, 64 * 1024, 4),        # 128 splits, one row
])
def test_fold_of_many_splits(B, Hq, Hkv, d, P, Bq):
    w = wl.Workload(f"fm_{B}_{Hkv}_{d}_{Bq}", B, Hq, Hkv, d, P, Bq, 1, 1, "bf16", 1.0)
    Kp, Vp = wl.make_prefix(w, 611)
    step = wl.make_block_steps(w, 611)[0]
    want = orc.run_block_dense(Kp, Vp, [step], 1)[0]
    q, kb, vb, k, v = (T.to_dev(x, "bf16") for x in (*step, Kp, Vp))
    shape, ext, out, lse = T.shape_of(w), T.Partial(w), torch.empty_like(q), torch.empty(q.shape[:3], device=T.DEV)
    assert fb.fb_external_splits(shape) > 4 * 1024 // d
    for call in ("step", "external"):
        if call == "step":
            fb.fb_refresh_step(shape, q, k, v, kb, vb, ext.o, ext.m, ext.lse, out, lse, T.workspace(shape))
            T.assert_close(out.double().cpu().numpy(), want["out"], "bf16", w.name + " out")
            T.assert_close(lse.double().cpu().numpy(), want["lse"], "bf16", w.name + " lse", lse=True)
        else:
            fb.fb_external_partial(shape, q, k, v, ext.o, ext.m, ext.lse, T.workspace(shape))
        T.check_partial(ext.numpy(), want["ext"], "bf16", w.name + " ext by " + call)
