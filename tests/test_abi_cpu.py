"""Host-only checks of the C ABI: the library loads, exports every symbol the header declares,
and every argument error is reported before anything touches a GPU."""
import ctypes
import os
import re

import pytest

from paper_2602_05305_amd import flashblock as fb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADERS = [os.path.join(ROOT, "include", n) for n in sorted(os.listdir(os.path.join(ROOT, "include"))) if n.endswith(".h")]


def _declared():
    names = set()
    for h in HEADERS:
        text = re.sub(r"/\*.*?\*/", "", open(h).read(), flags=re.S)
        names |= set(re.findall(r"\b(fb_[a-z_]+)\s*\(", text))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    lib = fb.load_library()
    names = _declared()
    assert {"fb_external_partial", "fb_internal_merge", "fb_sparse_external_residual"} <= set(names)
    for n in names:
        assert hasattr(lib, n), n
    assert set(names) == set(fb.exported_symbols())
    assert fb.fb_version() == 110
    for n in names:   # the binding offers the same names
        assert hasattr(fb, n) or n in ("fb_status_string", "fb_last_hip_error"), n


def test_struct_layout_matches_header():
    assert ctypes.sizeof(fb.fb_shape) == 36
    assert fb.fb_shape.scale.offset == 32


def _ok_shape(**kw):
    base = dict(batch=1, n_q_heads=4, n_kv_heads=2, head_dim=64, block_len=16, prefix_len=256, dtype="f32")
    base.update(kw)
    return fb.make_shape(**base)


@pytest.mark.parametrize("kw,status", [
    (dict(), fb.FB_OK),
    (dict(batch=0), fb.FB_ERR_SHAPE),
    (dict(n_q_heads=5), fb.FB_ERR_SHAPE),
    (dict(n_q_heads=66, n_kv_heads=2), fb.FB_ERR_SHAPE),
    (dict(block_len=0), fb.FB_ERR_SHAPE),
    (dict(prefix_len=-1), fb.FB_ERR_SHAPE),
    (dict(prefix_len=0), fb.FB_OK),
    (dict(head_dim=96), fb.FB_ERR_UNSUPPORTED),
    (dict(head_dim=0), fb.FB_ERR_SHAPE),
    (dict(dtype=7), fb.FB_ERR_DTYPE),
    (dict(scale=-1.0), fb.FB_ERR_SHAPE),
    (dict(scale=float("nan")), fb.FB_ERR_SHAPE),
    (dict(scale=float("inf")), fb.FB_ERR_SHAPE),
    (dict(dtype="bf16", head_dim=128), fb.FB_OK),
])
def test_check_shape(kw, status):
    assert fb.fb_check_shape(_ok_shape(**kw)) == status


def test_struct_size_is_checked():
    s = _ok_shape()
    s.struct_size = 8
    assert fb.fb_check_shape(s) == fb.FB_ERR_SHAPE
    assert fb.load_library().fb_check_shape(None) == fb.FB_ERR_NULL


def test_workspace_and_split_queries():
    s = _ok_shape()
    assert fb.fb_external_splits(s) >= 1
    assert fb.fb_workspace_bytes(s) >= 256
    assert fb.fb_workspace_bytes(s, 0, 0, 8) >= 8 * 64 * (64 + 2) * 4
    assert fb.fb_workspace_bytes(s, 64, 2) > fb.fb_workspace_bytes(s)
    assert fb.fb_workspace_bytes(s, 48, 2) == 0             # key_block not a multiple of 64
    assert fb.fb_workspace_bytes(s, 0, 0, 1000) == 0
    assert fb.fb_workspace_bytes(_ok_shape(batch=0)) == 0
    big = _ok_shape(dtype="bf16", head_dim=128, n_q_heads=32, n_kv_heads=8, block_len=32, prefix_len=131072)
    assert fb.fb_external_splits(big) == 32      # one 8-wavefront workgroup per CU: 256 CUs / 8 KV heads


TOO_SMALL = 256                      # below one split partial of _ok_shape (the general query also covers fb_refresh_step)
FAKE = ctypes.c_void_p(0x1000)       # aligned, never dereferenced: validation fails first
ODD = ctypes.c_void_p(0x1004)


def test_external_partial_error_paths():
    lib = fb.load_library()
    s = _ok_shape()
    ws_bytes = fb.fb_workspace_bytes(s)
    call = lib.fb_external_partial
    assert call(ctypes.byref(s), None, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, None, FAKE, FAKE, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, None, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), ODD, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_ALIGN
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, ODD, FAKE, ws_bytes, None) == fb.FB_ERR_ALIGN
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None, ws_bytes, None) == fb.FB_ERR_WORKSPACE
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, TOO_SMALL, None) == fb.FB_ERR_WORKSPACE
    bad = _ok_shape(head_dim=96)
    assert call(ctypes.byref(bad), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_UNSUPPORTED
    ex = lib.fb_external_partial_ex
    assert ex(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 257, FAKE, 1 << 30, None) == fb.FB_ERR_SHAPE
    assert ex(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, -1, FAKE, 1 << 30, None) == fb.FB_ERR_SHAPE
    assert ex(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, 16, FAKE, TOO_SMALL, None) in (
        fb.FB_ERR_WORKSPACE,)


def test_external_partial_heads_error_paths():
    lib = fb.load_library()
    s = _ok_shape()
    ws_bytes = fb.fb_workspace_bytes(s)
    call = lib.fb_external_partial_heads
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, None, 0, FAKE, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, 0, FAKE, FAKE, FAKE, FAKE, TOO_SMALL, None) == fb.FB_ERR_WORKSPACE
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, ODD, 0, ODD, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_ALIGN  # mask may be unaligned, o may not
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, -1, FAKE, FAKE, FAKE, FAKE, ws_bytes, None) == fb.FB_ERR_SHAPE
    # the hint changes the split count where few heads leave the GPU underfilled
    video = _ok_shape(dtype="bf16", head_dim=128, n_q_heads=12, n_kv_heads=12, block_len=4680, prefix_len=37440)
    assert fb.fb_external_heads_splits(video, 0) == fb.fb_external_splits(video) == 1
    assert fb.fb_external_heads_splits(video, 12) == 1
    assert fb.fb_external_heads_splits(video, 6) == 1            # 222 workgroups: one round either way
    assert fb.fb_external_heads_splits(video, 3) == 2
    assert fb.fb_external_heads_splits(video, 1) == 6            # 37 row tiles x 6 = 222 workgroups, one round
    assert fb.fb_external_heads_splits(video, -1) == 0


@pytest.mark.parametrize("heads,kv,rows,prefix", [(8, 8, 1000, 3000), (12, 12, 1000, 16000), (32, 8, 64, 8000), (4, 4, 40, 100),
                                                  (12, 12, 4680, 37440), (10, 5, 300, 0), (32, 1, 9, 700)])
def test_a_hint_on_a_short_stream_never_means_fewer_splits(heads, kv, rows, prefix):
    """Where a split of the flagged groups that fill 256 workgroups would have fewer than 8 tiles, from 16 tiles on."""
    s = _ok_shape(dtype="bf16", head_dim=128, n_q_heads=heads, n_kv_heads=kv, block_len=rows, prefix_len=prefix)
    tiles, plain, short = -(-prefix // 64), fb.fb_external_heads_splits(s, 0), 0
    for active in range(1, heads):
        groups = min(active, kv) * -(-heads // kv * rows // 128)
        if 16 <= tiles < 8 * (256 // groups):
            short += 1
            assert fb.fb_external_heads_splits(s, active) >= max(plain, min(tiles // 8, 7), 1), active
    assert short > 0 or prefix in (37440, 0, 100, 700)


def _paged(**kw):
    base = dict(struct_size=ctypes.sizeof(fb.fb_paged_kv), num_pages=8, page_size=64, max_pages=4,
                k_pool=0x1000, v_pool=0x1000, block_table=0x1000, prefix_lens=0x1000)
    base.update(kw)
    return fb.fb_paged_kv(**base)


def test_external_partial_paged_error_paths():
    lib = fb.load_library()
    s = _ok_shape()                       # prefix_len 256 = 4 pages of 64
    ws_bytes = fb.fb_workspace_bytes(s, 0, 0, fb.fb_paged_splits(s))
    call = lib.fb_external_partial_paged
    tail = (FAKE, FAKE, FAKE, 0, FAKE, ws_bytes, None)
    assert ctypes.sizeof(fb.fb_paged_kv) == 48
    assert call(ctypes.byref(s), FAKE, None, *tail) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), None, ctypes.byref(_paged()), *tail) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(struct_size=40)), *tail) == fb.FB_ERR_SHAPE
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(block_table=None)), *tail) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(prefix_lens=None)), *tail) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(k_pool=None)), *tail) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(page_size=96)), *tail) == fb.FB_ERR_UNSUPPORTED
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(page_size=0)), *tail) == fb.FB_ERR_SHAPE
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(num_pages=0)), *tail) == fb.FB_ERR_SHAPE
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(max_pages=3)), *tail) == fb.FB_ERR_SHAPE   # 3*64 < 256
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged(v_pool=0x1004)), *tail) == fb.FB_ERR_ALIGN
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged()), FAKE, FAKE, FAKE, 0, FAKE, TOO_SMALL, None) == fb.FB_ERR_WORKSPACE
    assert call(ctypes.byref(s), FAKE, ctypes.byref(_paged()), FAKE, FAKE, FAKE, 300, FAKE, 1 << 30, None) == fb.FB_ERR_SHAPE


def test_internal_merge_error_paths():
    lib = fb.load_library()
    s = _ok_shape()
    call = lib.fb_internal_merge
    assert call(ctypes.byref(s), None, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None, None) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, None, None, None) == fb.FB_ERR_NULL
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, None, FAKE, FAKE, None, None) == fb.FB_ERR_NULL  # 2 of 3
    assert call(ctypes.byref(s), FAKE, FAKE, ODD, FAKE, FAKE, FAKE, FAKE, None, None) == fb.FB_ERR_ALIGN
    assert call(ctypes.byref(s), FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, FAKE, ODD, None) == fb.FB_ERR_ALIGN


def test_refresh_step_error_paths():
    lib = fb.load_library()
    s = _ok_shape()
    ws_bytes = fb.fb_workspace_bytes(s)
    call = lib.fb_refresh_step
    ok = [FAKE] * 9 + [None, FAKE, ws_bytes, None]       # q kp vp kb vb o m lse out | lse_out ws bytes stream
    for i in (0, 3, 4, 5, 6, 7, 8):
        a = list(ok); a[i] = None
        assert call(ctypes.byref(s), *a) == fb.FB_ERR_NULL, i
    a = list(ok); a[1] = None
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_NULL                       # prefix_len > 0 needs k_prefix
    a = list(ok); a[8] = ODD
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_ALIGN
    a = list(ok); a[10] = None
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_WORKSPACE
    a = list(ok); a[11] = ws_bytes - 1
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_WORKSPACE
    assert call(ctypes.byref(_ok_shape(head_dim=96)), *ok) == fb.FB_ERR_UNSUPPORTED


def test_sparse_error_paths():
    lib = fb.load_library()
    s = _ok_shape()
    ws_bytes = fb.fb_workspace_bytes(s, 64, 2)
    call = lib.fb_sparse_external_residual
    args = [FAKE] * 3 + [64, 2, FAKE] + [FAKE] * 6 + [FAKE, ws_bytes, None]
    assert call(ctypes.byref(s), 3, *args) == fb.FB_ERR_SHAPE                       # bad mode
    a = list(args); a[5] = None; a[13] = TOO_SMALL
    assert call(ctypes.byref(s), 2, *a) == fb.FB_ERR_WORKSPACE                      # same-selection reuse takes no sel_idx
    a = list(args); a[3] = 48
    assert call(ctypes.byref(s), 0, *a) == fb.FB_ERR_UNSUPPORTED                    # key_block % 64
    a = list(args); a[3] = 0
    assert call(ctypes.byref(s), 0, *a) == fb.FB_ERR_SHAPE
    a = list(args); a[4] = -1
    assert call(ctypes.byref(s), 0, *a) == fb.FB_ERR_SHAPE
    a = list(args); a[5] = None
    assert call(ctypes.byref(s), 0, *a) == fb.FB_ERR_NULL                           # topk > 0 needs idx
    a = list(args); a[6] = None
    assert call(ctypes.byref(s), 1, *a) == fb.FB_ERR_NULL
    a = list(args); a[13] = ws_bytes - 1
    assert call(ctypes.byref(s), 0, *a) == fb.FB_ERR_WORKSPACE
    a = list(args); a[0] = ODD
    assert call(ctypes.byref(s), 0, *a) == fb.FB_ERR_ALIGN
    assert lib.fb_pool_keys(ctypes.byref(s), FAKE, 32, FAKE, None) == fb.FB_ERR_UNSUPPORTED
    assert lib.fb_pool_keys(ctypes.byref(s), None, 64, FAKE, None) == fb.FB_ERR_NULL
    assert lib.fb_select_topk(ctypes.byref(s), None, FAKE, 64, 2, FAKE, None, 0, None) == fb.FB_ERR_NULL
    assert lib.fb_select_topk(ctypes.byref(s), FAKE, FAKE, 64, 2, ODD, None, 0, None) == fb.FB_ERR_ALIGN
    n = fb.fb_select_workspace_bytes(s, 64)
    heads = s.batch * s.n_q_heads
    assert n >= heads * (s.head_dim + -(-s.prefix_len // 64)) * 4 and n % 256 == 0
    assert fb.fb_select_workspace_bytes(s, 48) == 0
    assert lib.fb_select_topk(ctypes.byref(s), FAKE, FAKE, 64, 2, FAKE, FAKE, n - 1, None) == fb.FB_ERR_WORKSPACE
    assert lib.fb_select_topk(ctypes.byref(s), FAKE, FAKE, 64, 2, FAKE, ODD, n, None) == fb.FB_ERR_ALIGN
    huge = _ok_shape(prefix_len=64 * 16385)
    assert lib.fb_pool_keys(ctypes.byref(huge), FAKE, 64, FAKE, None) == fb.FB_ERR_UNSUPPORTED


def test_select_topk_mass_error_paths():
    lib = fb.load_library()
    s = _ok_shape()
    n = fb.fb_select_mass_workspace_bytes(s, 64)
    assert n >= 64 * 4 * 4                           # 64 rows x 4 key blocks, floats
    assert fb.fb_select_mass_workspace_bytes(s, 48) == 0
    assert fb.fb_select_mass_workspace_bytes(_ok_shape(batch=0), 64) == 0
    call = lib.fb_select_topk_mass
    ok = [FAKE, FAKE, FAKE, 64, 2, FAKE, None, FAKE, n, None]     # q k lse key_block topk idx mass ws bytes stream
    for i in (0, 1, 2, 5):
        a = list(ok); a[i] = None
        assert call(ctypes.byref(s), *a) == fb.FB_ERR_NULL, i
    a = list(ok); a[3] = 48
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_UNSUPPORTED
    a = list(ok); a[4] = -1
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_SHAPE
    a = list(ok); a[4] = 0
    assert call(ctypes.byref(s), *a) == fb.FB_OK                  # nothing to select, nothing launched
    a = list(ok); a[6] = ODD
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_ALIGN
    a = list(ok); a[7] = None
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_WORKSPACE
    a = list(ok); a[8] = n - 1
    assert call(ctypes.byref(s), *a) == fb.FB_ERR_WORKSPACE
    assert call(ctypes.byref(_ok_shape(prefix_len=0)), *ok) == fb.FB_OK


def test_status_strings():
    lib = fb.load_library()
    seen = {lib.fb_status_string(i).decode() for i in range(8)}
    assert len(seen) == 8 and all(s.startswith("FB_") for s in seen)
    assert lib.fb_status_string(99).decode().startswith("unknown")


def test_binding_has_no_cpu_fallback(monkeypatch, tmp_path):
    monkeypatch.setattr(fb, "_lib", None)
    monkeypatch.setattr(fb, "LIB_PATH", str(tmp_path / "missing.so"))
    with pytest.raises(RuntimeError, match="no CPU fallback"):
        fb.load_library()


def test_bench_refuses_more_than_one_gpu():
    """This build has no multi-GPU part: bench.py --gpus N > 1 exits with a message (before touching any GPU)."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True, text=True,
                       timeout=60, cwd=ROOT)
    assert r.returncode != 0 and "one GPU" in r.stderr


def test_header_is_plain_c_and_links(tmp_path):
    """include/flashblock.h is a C header (C99, no C++ needed) and a C program links against the library."""
    import shutil
    import subprocess
    if shutil.which("gcc") is None:
        pytest.skip("no gcc")
    src = tmp_path / "use.c"
    src.write_text('#include "flashblock.h"\n#include <stdio.h>\n'
                   "int main(void) {\n"
                   "  fb_shape s = {sizeof(fb_shape), 1, 4, 2, 64, 16, 256, FB_F32, 0.0f};\n"
                   "  fb_paged_kv kv; kv.struct_size = sizeof kv; (void)kv;\n"
                   '  printf("%d %d %d %zu\\n", fb_version(), (int)fb_check_shape(&s), (int)fb_external_splits(&s),\n'
                   "         fb_workspace_bytes(&s, 0, 0, 0));\n"
                   "  return 0;\n}\n")
    exe = tmp_path / "use"
    libdir = os.path.dirname(fb.LIB_PATH)
    r = subprocess.run(["gcc", "-std=c99", "-pedantic", "-Wall", "-Werror", "-I", os.path.join(ROOT, "include"), str(src),
                        "-o", str(exe), "-L", libdir, "-l:libflashblock.so", f"-Wl,-rpath,{libdir}",
                        "-Wl,-rpath,/opt/rocm/lib", "-L/opt/rocm/lib"], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr
    out = subprocess.run([str(exe)], capture_output=True, text=True, timeout=60)
    assert out.returncode == 0, out.stderr
    ver, ok, splits, ws = out.stdout.split()
    assert int(ver) == 110 and int(ok) == fb.FB_OK and int(splits) >= 1 and int(ws) >= 256


def test_builtin_workspace_entry_rejects_on_the_host():
    """The entry point for callers that cannot allocate: size and argument checks come before any HIP call."""
    assert fb.fb_builtin_workspace_bytes() == 20 * 1024 * 1024
    lib = fb.load_library()
    video = fb.make_shape(1, 12, 12, 128, 4680, 37440, "bf16")
    one = ctypes.c_void_p(16)
    assert lib.fb_external_partial_builtin_ws(ctypes.byref(video), one, one, one, one, one, one, None) == fb.FB_ERR_WORKSPACE
    small = fb.make_shape(1, 4, 4, 64, 16, 256, "f32")
    assert lib.fb_external_partial_builtin_ws(ctypes.byref(small), None, one, one, one, one, one, None) == fb.FB_ERR_NULL
    bad = fb.make_shape(1, 4, 3, 64, 16, 256, "f32")
    assert lib.fb_external_partial_builtin_ws(ctypes.byref(bad), one, one, one, one, one, one, None) == fb.FB_ERR_SHAPE


def test_external_kernel_name_over_few_fp32_keys():
    name = lambda *a: fb.fb_external_kernel_name(fb.make_shape(*a))
    assert name(1, 4, 4, 64, 16, 16, "f32") == "attn_f32_few_kernel<64, 0>"
    assert name(1, 4, 4, 64, 16, 17, "f32") == name(16, 32, 4, 64, 16, 16, "f32") == name(1, 4, 4, 64, 16, 0, "f32") == "attn_f32_kernel<64, 0>"
    assert name(64, 32, 32, 128, 32, 3, "f32") == "attn_f32_few_kernel<128, 0>"      # many rows, 32 to a KV head


def test_external_kernel_name_follows_the_launch_rules():
    """Host-only query the benchmark labels its roofline with: streaming kernel (with 1, 2 or 4 row groups per workgroup) for up
    to 128 rows per KV group and at least 8 tiles per split, register-staged kernel for short prefixes, fp32 kernel for fp32."""
    name = lambda *a: fb.fb_external_kernel_name(fb.make_shape(*a))
    assert name(1, 32, 8, 128, 32, 32768, "bf16") == "attn_stream_kernel<128, 0, 0, 4>"       # 128 rows per KV group
    assert name(1, 32, 8, 128, 16, 32768, "bf16") == "attn_stream_kernel<128, 0, 0, 2>"       # 64 rows
    assert name(1, 32, 8, 128, 8, 131072, "bf16") == "attn_stream_kernel<128, 0, 0, 1>"       # 32 rows
    assert name(1, 12, 12, 128, 4680, 37440, "bf16") == "attn_stream_kernel<128, 0, 2, 4>"    # row-pair layout
    assert name(1, 32, 8, 128, 8, 4096, "bf16").startswith("attn_bf16_kernel<128, 0, 64, 4, ")  # short prefix: register-staged
    assert name(1, 32, 8, 64, 32, 32768, "bf16") == "attn_stream_kernel<64, 0, 0, 4>"
    assert name(1, 4, 4, 64, 16, 256, "f32") == "attn_f32_kernel<64, 0>"
    bad = fb.make_shape(1, 4, 3, 64, 16, 256, "f32")
    assert fb.fb_external_kernel_name(bad) == ""


@pytest.mark.parametrize("kw,layout", [
    (dict(prefix_len=13 * 64), 4), (dict(prefix_len=13 * 64 + 1), 2),        # one split: 13 and 14 tiles
    (dict(prefix_len=27 * 64), 4),                                           # three splits of 9
    (dict(head_dim=64, block_len=200, prefix_len=13 * 64), 4), (dict(head_dim=64, block_len=200, prefix_len=40000), 2),
])
def test_dense_row_pairs_by_tiles_per_split(kw, layout):
    shape = _ok_shape(**dict(dict(n_q_heads=64, n_kv_heads=8, head_dim=128, block_len=32, dtype="bf16"), **kw))
    assert fb.fb_external_kernel_name(shape) == f"attn_stream_kernel<{shape.head_dim}, 0, {layout}, 4>"


def test_native_calls_marshal_as_the_python_ones():
    """The native form of the binding passes the same C arguments, in the same order, as the Python functions it stands for."""
    import ctypes
    import inspect
    if fb._fbcall is None:
        pytest.skip("fb_call.c is not built")

    class Tensor:
        def __init__(self, at):
            self.at = at

        def data_ptr(self):
            return self.at

        def numel(self):
            return self.at // 16

        def element_size(self):
            return 4

    python = {"__name__": fb.__name__, "__file__": fb.__file__, "__package__": fb.__package__}
    exec(compile(inspect.getsource(fb).split("\n# The entry points in native form")[0], fb.__file__, "exec"), python)
    seen = []
    take = ctypes.CFUNCTYPE(ctypes.c_int, *[ctypes.c_int64] * 20)(lambda *a: seen.append(a) or 0)
    shape, kv = _ok_shape(), fb.fb_paged_kv()
    for name, kinds in fb._KINDS.items():
        fn = python[name]
        names = list(inspect.signature(fn).parameters)
        values = {n: shape if n == "shape" else kv if n == "kv" else 7 + i if n in ("key_block", "topk", "mode", "n_splits", "n_active_heads", "stream")
                  else Tensor(4096 * (i + 1)) for i, n in enumerate(names)}
        for left_out in ([], ["lse_out", "mass_out", "o_part"], [n for n in names if n in ("workspace",) and name == "fb_select_topk"]):
            args = {n: None if n in left_out else v for n, v in values.items()}
            want = []

            class Lib:
                def __getattr__(self, _):
                    return lambda *a: want.append(a) or 0
            python["load_library"] = Lib
            fn(**args)
            kinds_, order = kinds if isinstance(kinds, tuple) else (kinds, " ".join(names))
            native = fb._fbcall.Call(name, tuple(names), fn.__defaults__ or (), kinds_, tuple(names.index(x) for x in order.split()),
                                     lambda _: ctypes.cast(take, ctypes.c_void_p).value, lambda: 0, fb._check, fb.fb_shape, fb.fb_paged_kv)
            native(*args.values()) if not left_out else native(**args)
            flat = [ctypes.addressof(a._obj) if hasattr(a, "_obj") else a or 0 for a in want[0]]
            assert list(seen[-1][:len(flat)]) == flat and not any(seen[-1][len(flat):]), name


def test_native_calls_are_used_as_functions_are():
    """What a function of the module could be asked for, a native call can: signature, name, documentation, module, pickling, copying,
    weak references, a class attribute of it is a method."""
    import copy
    import inspect
    import pickle
    import weakref
    if fb._fbcall is None:
        pytest.skip("fb_call.c is not built")
    for name in fb._KINDS:
        call = getattr(fb, name)
        fn = call.__wrapped__
        assert inspect.signature(call) == inspect.signature(fn) and list(inspect.signature(call).parameters)[0] == "shape"
        assert call.__name__ == call.__qualname__ == name and call.__module__ == fb.__name__ and call.__doc__ == fn.__doc__
        assert pickle.loads(pickle.dumps(call)) is call and copy.deepcopy(call) is call and copy.copy(call) is call
        assert weakref.ref(call)() is call
        with pytest.raises(AttributeError):
            call.no_such_attribute

    class Holder:
        step = fb.fb_internal_merge
    holder = Holder()
    assert inspect.ismethod(holder.step) and holder.step.__self__ is holder and Holder.step is fb.fb_internal_merge


def test_native_calls_take_and_refuse_what_the_python_functions_do():
    """Arguments that are not plain integers, tensors and structures, and faulty calls, end as they do without the native form."""
    if fb._fbcall is None:
        pytest.skip("fb_call.c is not built")

    class Tensor:
        def __init__(self, at=4096):
            self.at = at

        def data_ptr(self):
            return self.at

        def numel(self):
            return 1 << 20

        def element_size(self):
            return 1

    class Stream:
        cuda_stream = 12345

    bad, t = _ok_shape(n_kv_heads=3), Tensor()              # a shape that is refused before anything is launched
    splits = dict(shape=bad, q=t, k_prefix=t, v_prefix=t, o_part=t, m_part=t, lse_part=t, n_splits=1, workspace=t, stream=0)

    def outcome(fn, *args, **kw):
        try:
            return fn(*args, **kw)
        except Exception as e:
            return type(e), str(e)
    cases = [(), dict(n_splits=ctypes.c_int32(2)), dict(stream=ctypes.c_void_p(0)), dict(stream=ctypes.c_void_p(64)), dict(stream=Stream()),
             dict(stream=2.5), dict(stream=ctypes.c_int64(3)), dict(n_splits=2.5), dict(n_splits=None), dict(n_splits=True), dict(n_splits=1 << 40),
             dict(shape=ctypes.byref(bad)), dict(shape=None), dict(shape=fb.fb_paged_kv()), dict(q=None), dict(q=7), dict(q=Tensor(None)),
             dict(q=Tensor(1.5)), dict(q=Tensor(ctypes.c_void_p(64))), dict(workspace=None), dict(workspace=9), dict(unknown=1)]
    for changed in cases:
        kw = dict(splits, **dict(changed))
        assert outcome(fb.fb_external_partial_ex, **kw) == outcome(fb.fb_external_partial_ex.__wrapped__, **kw), changed
    assert outcome(fb.fb_external_partial_ex, **splits)[0] is fb.FlashBlockError
    values = list(splits.values())
    for args, kw in ((values, {}), (values[:-1], dict(stream=0)), (values[:3], {}), (values + [1], {}), (values, dict(q=t)), ([], {}),
                     (values[:2], dict(q=t, n_splits=1))):
        assert outcome(fb.fb_external_partial_ex, *args, **kw) == outcome(fb.fb_external_partial_ex.__wrapped__, *args, **kw), (args, kw)
    # a workspace that may be left out
    args = (bad, t, t, 64, 2, t)
    for rest in ((), (None,), (t,), (None, 0), (t, 0)):
        kw = {} if len(rest) == 2 else dict(stream=0)
        assert outcome(fb.fb_select_topk, *args, *rest, **kw) == outcome(fb.fb_select_topk.__wrapped__, *args, *rest, **kw)
    # no other exception of an argument's own is taken for one of these

    class Interrupted(Tensor):
        def data_ptr(self):
            raise KeyboardInterrupt
    with pytest.raises(KeyboardInterrupt):
        fb.fb_external_partial_ex(**dict(splits, q=Interrupted()))


def test_the_library_is_usable_without_the_native_calls(tmp_path, monkeypatch, capfd):
    """No compiler for fb_call.c: a message, nothing stale left, and the Python functions make the calls."""
    import subprocess
    import sys
    import sysconfig
    from paper_2602_05305_amd import build as fb_build
    assert fb_build.CALL_LIB.endswith("_fbcall" + sysconfig.get_config_var("EXT_SUFFIX"))
    monkeypatch.setattr(fb_build, "CALL_LIB", str(tmp_path / os.path.basename(fb_build.CALL_LIB)))
    for left in (fb_build.CALL_LIB, tmp_path / "_fbcall.so"):
        open(left, "w").close()
    for cc in ("/no/such/compiler", "false"):
        monkeypatch.setenv("CC", cc)
        fb_build._build_call()
        assert os.listdir(tmp_path) == [] and "not built" in capfd.readouterr().err
    code = ("import sys; sys.modules['paper_2602_05305_amd._fbcall'] = None\n"
            "from paper_2602_05305_amd import flashblock as fb\n"
            "import types; assert fb._fbcall is None and isinstance(fb.fb_internal_merge, types.FunctionType)\n"
            "try: fb.fb_internal_merge(fb.make_shape(1, 4, 3, 64, 16, 256, 'f32'), None, None, None, None, None, None, None, None, 0)\n"
            "except fb.FlashBlockError as e: assert e.status == fb.FB_ERR_SHAPE\n"
            "else: sys.exit('no error')\n")
    r = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=120, cwd=ROOT)
    assert r.returncode == 0, r.stderr


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("B,Hq,Hkv,Bq,P", [(3, 8, 8, 9, 16913), (5, 8, 8, 32, 8424), (11, 4, 4, 48, 92023), (15, 16, 8, 25, 3000),
                                           (1, 32, 8, 32, 32768), (1, 12, 12, 4680, 37440)])
def test_workspace_of_the_librarys_split_count_holds_its_own_passes(B, Hq, Hkv, Bq, P, d):
    """Passes in pieces ask for a partial per reference segment, more than there are pieces."""
    shape = fb.make_shape(B, Hq, Hkv, d, Bq, P, "bf16")
    rows = B * Hq * Bq
    splits = fb.fb_external_splits(shape)
    if Hq // Hkv * Bq <= 128:
        splits = max(splits, -(-256 // (B * Hkv)))
    held = sum(-(-n * rows * x * 4 // 256) * 256 for n in (splits, 1) for x in (d, 1, 1))
    assert fb.fb_workspace_bytes(shape, n_splits=fb.fb_external_splits(shape)) >= held
    assert fb.fb_workspace_bytes(shape) >= held


@pytest.mark.parametrize("B,Hq,Hkv,d,Bq,ns,tiles,streams", [
    (1, 8, 8, 128, 640, 7, 70, True), (1, 8, 8, 128, 640, 7, 69, False),        # 10 tiles a split, and one fewer altogether
    (1, 8, 8, 128, 639, 7, 70, False), (1, 12, 6, 64, 650, 4, 56, True),        # blocks from 640 tokens on
    (1, 1, 1, 64, 640, 52, 52 * 16, True), (1, 1, 1, 64, 640, 52, 52 * 16 - 1, False),           # head_dim 64: few heads in many splits
    (1, 2, 2, 64, 700, 22, 220, True), (1, 1, 1, 128, 640, 52, 520, True),
    (1, 1, 1, 64, 4096, 8, 8 * 32, True), (1, 1, 1, 64, 4096, 8, 8 * 33, False),                 # one round of fewer than 8 heads
    (1, 4, 2, 64, 2048, 4, 4 * 96, False), (1, 4, 2, 64, 2048, 4, 4 * 160, True), (2, 4, 4, 64, 2048, 2, 2 * 80, True),
    (1, 1, 1, 64, 1024, 32, 32 * 64, False), (1, 1, 1, 64, 1024, 32, 32 * 80, True),
    (9, 24, 8, 64, 43, 2, 28, True), (9, 24, 8, 64, 43, 2, 27, False),          # one-tile blocks: combine and internal pass
    (3, 24, 8, 128, 43, 6, 6 * 36, True), (3, 24, 8, 128, 43, 6, 6 * 36 - 1, False),             # fold kernel
    (10, 64, 8, 64, 43, 2, 31, False), (8, 64, 8, 64, 43, 2, 31, True),          # 640 workgroups for 480, 512 for 384
    (4, 64, 4, 64, 62, 2, 63, False), (4, 64, 4, 64, 62, 2, 64, True), (4, 64, 4, 128, 62, 2, 28, True),       # one round of 256
    (2, 32, 4, 128, 59, 8, 8 * 48 - 1, False), (2, 32, 4, 128, 59, 8, 8 * 48, True), (2, 32, 4, 64, 59, 8, 8 * 36, True),      # few heads of many rows
    (1, 64, 4, 128, 59, 8, 8 * 64 - 1, False), (1, 64, 4, 128, 59, 8, 8 * 64, True),
    (7, 96, 12, 64, 45, 2, 260, False), (7, 96, 12, 128, 48, 2, 159, False), (7, 96, 12, 128, 48, 2, 160, True), (7, 72, 12, 128, 42, 2, 40, True),
])
def test_refresh_steps_by_streams(B, Hq, Hkv, d, Bq, ns, tiles, streams):
    """Which refresh steps of many rows run as streams of even and odd tiles, on both sides of every line of the rule: they want room
    for twice the splits and two partials of the block."""
    shape = fb.make_shape(B, Hq, Hkv, d, Bq, 64 * tiles, "bf16")
    rows = B * Hq * Bq
    held = sum(-(-n * rows * x * 4 // 256) * 256 for n in (2 * ns, 2) for x in (d, 1, 1)) + 256
    assert ns == -(-256 // (B * Hkv * -(-Hq // Hkv * Bq // 128)))
    got = fb.fb_workspace_bytes(shape)
    assert got == held if streams else got < held
