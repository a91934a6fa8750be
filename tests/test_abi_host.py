"""CPU-only checks of the C-ABI library: it loads, exports every symbol that
include/msla.h declares, and rejects bad arguments on the host before any
launch (so none of these calls touches a GPU)."""
import ctypes
import os
import re

import pytest

from paper_2205_14756_amd import build as msla_build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

OK, INVALID, UNSUPPORTED, WORKSPACE = 0, -1, -2, -3
F32, F16, BF16 = 0, 1, 2


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(msla_build.LIB):
        msla_build.build(True)
    return ctypes.CDLL(msla_build.LIB)


def declared_functions():
    text = open(os.path.join(ROOT, "include", "msla.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(msla_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(lib):
    names = declared_functions()
    assert set(names) == {"msla_error_string", "msla_workspace_bytes", "msla_forward", "msla_forward_opts", "msla_forward_profiled",
                          "msla_core_forward",
                          "msla_multiscale_state", "msla_multiscale_state_static", "msla_linear",
                          "msla_ffn_workspace_bytes", "msla_ffn_forward", "msla_block_workspace_bytes", "msla_block_forward",
                          "msla_softmax_attention", "msla_linear_attention_backward_workspace_bytes",
                          "msla_linear_attention_backward"}
    for n in names:
        assert getattr(lib, n) is not None
    from paper_2205_14756_amd import msla
    assert set(msla.EXPORTS) == set(names)
    for n in names:
        if n != "msla_error_string":
            assert callable(getattr(msla, n))


def test_error_strings(lib):
    lib.msla_error_string.restype = ctypes.c_char_p
    seen = set()
    for code in (0, -1, -2, -3, -4, 17):
        s = lib.msla_error_string(code)
        assert s and len(s) > 3
        seen.add(s)
    assert len(seen) == 6


def _ws(lib, B, C, H, W, heads, d, scales, dt):
    arr = (ctypes.c_int * max(1, len(scales)))(*scales)
    out = ctypes.c_size_t(12345)
    st = lib.msla_workspace_bytes(B, C, H, W, heads, d, arr, len(scales), dt, ctypes.byref(out))
    return st, out.value


def test_workspace_bytes(lib):
    st, n = _ws(lib, 8, 256, 64, 128, 16, 16, [5], F16)
    assert st == OK
    T, Ct, S = 8 * 64 * 128, 256, 2
    # at least the multi-scale Q map and the raw K/V map, and not absurdly more
    assert T * S * Ct * 2 + T * 2 * Ct * 2 <= n <= T * S * Ct * 2 + T * 2 * Ct * 2 + (64 << 20)
    st32, n32 = _ws(lib, 1, 64, 32, 32, 4, 16, [5], F32)
    assert st32 == OK and n32 >= 1024 * (2 * 64 + 2 * 64) * 4
    assert _ws(lib, 1, 64, 32, 32, 4, 16, [], F32)[0] == OK
    # invalid
    assert _ws(lib, 0, 64, 32, 32, 4, 16, [5], F32)[0] == INVALID
    assert _ws(lib, 1, 64, 32, 32, 4, 16, [4], F32)[0] == INVALID      # even kernel
    assert _ws(lib, 1, 64, 32, 32, 4, 16, [5], 9)[0] == INVALID        # bad dtype
    assert _ws(lib, 1, 64, -3, 32, 4, 16, [5], F32)[0] == INVALID
    assert lib.msla_workspace_bytes(1, 64, 32, 32, 4, 16, None, 1, F32, ctypes.byref(ctypes.c_size_t())) == INVALID
    assert lib.msla_workspace_bytes(1, 64, 32, 32, 4, 16, None, 0, F32, None) == INVALID
    # unsupported
    assert _ws(lib, 1, 64, 32, 32, 8, 8, [5], F32)[0] == OK            # head_dim 8 and 32: the plain kernels
    assert _ws(lib, 1, 64, 32, 32, 2, 32, [5], F16)[0] == OK
    assert _ws(lib, 1, 96, 32, 32, 4, 24, [5], F32)[0] == UNSUPPORTED  # head_dim not in {8, 16, 32}
    assert _ws(lib, 1, 64, 32, 32, 4, 16, [9], F32)[0] == UNSUPPORTED   # kernel sizes other than 3, 5, 7
    assert _ws(lib, 1, 64, 32, 32, 4, 16, [7], F32)[0] == OK
    assert _ws(lib, 1, 60, 32, 32, 4, 16, [5], F32)[0] == UNSUPPORTED  # C not a multiple of 16
    # a failed query leaves *bytes alone
    assert _ws(lib, 1, 64, 32, 32, 4, 16, [9], F32)[1] == 12345


def _fwd(lib, x=0x1000, wq=0x1000, wd=0x1000, wg=0x1000, wp=0x1000, out=0x2000, ws=0x3000, ws_bytes=1 << 40,
         B=1, C=64, H=32, W=32, heads=4, d=16, scales=(5,), eps=1e-15, dt=F32, layout=0):
    lib.msla_forward.argtypes = [ctypes.c_void_p] * 7 + [ctypes.c_size_t] + [ctypes.c_int] * 6 + \
        [ctypes.POINTER(ctypes.c_int), ctypes.c_int, ctypes.c_float, ctypes.c_int, ctypes.c_int, ctypes.c_void_p]
    arr = (ctypes.c_int * max(1, len(scales)))(*scales)
    return lib.msla_forward(x, wq, wd, wg, wp, out, ws, ws_bytes, B, C, H, W, heads, d, arr, len(scales),
                            eps, dt, layout, None)


def test_forward_rejects_bad_arguments_before_launching(lib):
    # every call below fails validation, so the fake pointers are never dereferenced or passed to HIP
    assert _fwd(lib, x=None) == INVALID
    assert _fwd(lib, out=None) == INVALID
    assert _fwd(lib, ws=None) == INVALID
    assert _fwd(lib, wd=None) == INVALID
    assert _fwd(lib, x=0x1004) == INVALID            # misaligned
    assert _fwd(lib, eps=-1.0) == INVALID
    assert _fwd(lib, eps=float("nan")) == INVALID
    assert _fwd(lib, layout=5) == INVALID
    assert _fwd(lib, scales=(2,)) == INVALID
    assert _fwd(lib, H=0) == INVALID
    assert _fwd(lib, layout=1, C=256) == UNSUPPORTED  # channel-planar needs C <= 2 * heads * head_dim
    assert _fwd(lib, d=24, C=96) == UNSUPPORTED
    assert _fwd(lib, d=32, heads=2, C=256, layout=1) == UNSUPPORTED   # ... with heads of 32: C <= 3 * heads * head_dim
    assert _fwd(lib, d=8, heads=3, C=32, layout=1) == UNSUPPORTED      # an odd number of heads of 8: not at all
    assert _fwd(lib, d=32, heads=2, ws_bytes=1024) == WORKSPACE
    assert _fwd(lib, scales=(9,)) == UNSUPPORTED
    assert _fwd(lib, ws_bytes=1024) == WORKSPACE


def test_other_entry_points_reject_bad_arguments(lib):
    vp, i = ctypes.c_void_p, ctypes.c_int
    ip = ctypes.POINTER(ctypes.c_int)
    lib.msla_core_forward.argtypes = [vp] * 5 + [ctypes.c_size_t] + [i] * 5 + [ip, i, ctypes.c_float, i, vp]
    lib.msla_multiscale_state.argtypes = [vp] * 6 + [ctypes.c_size_t] + [i] * 5 + [ip, i, i, vp]
    lib.msla_linear.argtypes = [vp, vp, vp, ctypes.c_long, i, i, i, vp]
    sc = (ctypes.c_int * 1)(5)
    assert lib.msla_core_forward(None, 0x1000, 0x1000, 0x1000, 0x1000, 1 << 40, 1, 8, 8, 2, 16, sc, 1, 1e-15, F16, None) == INVALID
    assert lib.msla_core_forward(0x1000, 0x1000, 0x1000, 0x1000, 0x1000, 16, 1, 8, 8, 2, 16, sc, 1, 1e-15, F16, None) == WORKSPACE
    assert lib.msla_core_forward(0x1000, 0x1000, 0x1000, 0x1000, 0x1000, 1 << 40, 1, 8, 8, 2, 24, sc, 1, 1e-15, F16, None) == UNSUPPORTED
    assert lib.msla_multiscale_state(0x1000, 0x1000, 0x1000, None, None, 0x1000, 1 << 40, 1, 8, 8, 2, 16, sc, 1, F16, None) == INVALID
    assert lib.msla_multiscale_state(0x1000, 0x1000, 0x1000, None, 0x1000, 0x1000, 8, 1, 8, 8, 2, 16, sc, 1, F16, None) == WORKSPACE
    assert lib.msla_linear(None, 0x1000, 0x1000, 10, 16, 16, F16, None) == INVALID
    assert lib.msla_linear(0x1000, 0x1000, 0x1000, 0, 16, 16, F16, None) == INVALID
    assert lib.msla_linear(0x1000, 0x1000, 0x1000, 10, 24, 16, F16, None) == UNSUPPORTED
    assert lib.msla_linear(0x1000, 0x1000, 0x1000, 10, 16, 16, 7, None) == INVALID


def test_product_path_does_not_touch_the_oracle():
    pkg = os.path.join(ROOT, "paper_2205_14756_amd")
    for dirpath, _, files in os.walk(pkg):
        for f in files:
            if f.endswith((".py", ".h", ".hip", ".cpp")):
                text = open(os.path.join(dirpath, f)).read()
                assert "msla_oracle" not in text, os.path.join(dirpath, f)
                assert not re.search(r"^\s*(import|from)\s+\S*oracle", text, flags=re.M), os.path.join(dirpath, f)


def test_bench_refuses_more_than_one_gpu():
    """This build runs on one GPU; asked for more, the bench says so and does not start."""
    import subprocess
    import sys
    r = subprocess.run([sys.executable, os.path.join(ROOT, "bench.py"), "--gpus", "2"], capture_output=True,
                       text=True, timeout=120)
    assert r.returncode != 0
    assert "one GPU" in (r.stderr + r.stdout)
    assert not any(line.startswith("{") for line in r.stdout.splitlines())


def test_forward_opts_rejects_unknown_bits_and_stage_bits_with_nchw(lib):
    sc = (ctypes.c_int * 1)(5)
    vp = ctypes.c_void_p
    lib.msla_forward_opts.argtypes = [vp] * 7 + [ctypes.c_size_t] + [ctypes.c_int] * 6 + [ctypes.POINTER(ctypes.c_int), ctypes.c_int,
                                                                                          ctypes.c_float, ctypes.c_int, ctypes.c_int, vp, ctypes.c_uint]
    lib.msla_forward_opts.restype = ctypes.c_int
    p = vp(0x1000)      # never dereferenced: every check below fails on the host
    call = lambda layout, opts: lib.msla_forward_opts(p, p, p, p, p, p, p, 1 << 40, 1, 64, 8, 8, 4, 16, sc, 1, 1e-15, F16,
                                                      layout, None, opts)
    assert call(0, 64) == INVALID and call(0, 0x80000000) == INVALID
    assert call(1, 2) == UNSUPPORTED and call(1, 16 | 1) == UNSUPPORTED


def _fp32_chunks(lib, B, H, W, heads, scales):
    """Workgroups a state in the fp32 aggregation, from the size of the workspace that holds their partial states."""
    up = lambda v: (v + 255) // 256 * 256
    T, Ct, states = B * H * W, 16 * heads, B * heads * (1 + len(scales))
    fixed = up(T * (1 + len(scales)) * Ct * 4) + up((T + 31) // 32 * 32 * 2 * Ct * 4) + up(states * 1088) + up(states * 2048) + up(states * 4)
    st, n = _ws(lib, B, Ct, H, W, heads, 16, scales, F32)
    assert st == OK
    return [c for c in range(1, 1025) if fixed + up(states * c * 1088) == n]


@pytest.mark.parametrize("B,H,W,heads,scales,chunks", [
    (1, 32, 32, 4, (5,), 4),                # four tiles: one each
    (4, 64, 128, 8, (5,), 16),              # 512 workgroups are one round of two a compute unit
    (6, 50, 144, 14, (5,), 6),              # 504 in one round, not 588 in two
    (20, 40, 40, 15, (3, 5), 3),            # 900 in two rounds with 4 tiles, not 600 in two with 5
    (6, 50, 144, 14, (7,), 3),              # 7x7, one workgroup a compute unit: 252
    (32, 16, 16, 12, (7,), 2),              # 768 in three rounds of one tile, not 384 in two of two
    (2, 64, 128, 400, (5,), 1),             # more states than places
])
def test_fp32_workgroups_fill_whole_rounds(lib, B, H, W, heads, scales, chunks):
    assert chunks in _fp32_chunks(lib, B, H, W, heads, scales)


def _f16_chunks(lib, B, H, W, heads, scales):
    """The same for the 16-bit matrix-core aggregation."""
    up = lambda v: (v + 255) // 256 * 256
    T, Ct, states = B * H * W, 16 * heads, B * heads * (1 + len(scales))
    fixed = up(T * (1 + len(scales)) * Ct * 2) + up((T + 31) // 32 * 32 * 2 * Ct * 2) + up(states * 1088) + up(states * 2048) + up(states * 4)
    st, n = _ws(lib, B, Ct, H, W, heads, 16, scales, F16)
    assert st == OK
    return [c for c in range(1, 1025) if fixed + up(states * c * 1088) == n]


@pytest.mark.parametrize("B,H,W,heads,scales,chunks", [
    (8, 64, 128, 16, (5,), 2),              # 256 workgroups, 8 tiles each
    (5, 90, 90, 11, (5,), 4),               # 220 in one round with 5 tiles, not 275 in two with 4
    (3, 64, 100, 17, (3, 5), 2),            # two scales share the chip: 102 of each in one round, not 153 in two
    (9, 100, 100, 6, (3,), 4),              # 216 in one round
    (2, 64, 128, 400, (5,), 1),             # more states than places
    (9, 23, 113, 19, (7,), 2),              # a 7x7 scale: the general kernel, two workgroups a compute unit, 342 of them
    (10, 72, 24, 22, (3, 7), 2),
])
def test_matrix_core_workgroups_fill_whole_rounds(lib, B, H, W, heads, scales, chunks):
    assert chunks in _f16_chunks(lib, B, H, W, heads, scales)


# (dtype 1: fp16, 2: bf16; B, C, H, W, hidden) -> rows of a block of the one-launch FFN, 0: two launches.  Us of two launches /
# blocks of four / of eight rows
@pytest.mark.parametrize("shape,rows", [
    ((1, 8, 128, 1, 4096, 512), 0),         # one row of tokens
    ((2, 8, 128, 1, 4096, 512), 0),
    ((1, 16, 128, 2, 512, 512), 0),
    ((1, 8, 128, 4096, 1, 512), 0),         # one column
    ((1, 4096, 64, 1, 1, 256), 0),          # images of one token, of 3 x 3, 4 x 4 and 7 x 7
    ((1, 2048, 128, 3, 3, 512), 0),
    ((1, 1024, 64, 4, 4, 256), 0),
    ((2, 512, 256, 7, 7, 1024), 0),
    ((1, 64, 256, 17, 17, 1024), 0),        # 17 = 16 + 1 columns, 4 x 4 + 1 rows
    ((1, 1, 128, 4, 16, 2048), 0),          # many slabs for one workgroup
    ((2, 1, 128, 32, 32, 768), 0),
    ((2, 5, 112, 114, 222, 224), 8),        # a hidden size that the two launches' slabs of 64 and passes of 192 channels pad most
    ((2, 15, 160, 181, 231, 80), 8),
    ((1, 9, 176, 44, 159, 176), 4),         # four rounds of 64 tokens before three of 128
    ((2, 8, 256, 64, 96, 1024), 4),         # three before two
    ((1, 1, 128, 64, 128, 512), 4),
    ((2, 1, 32, 8, 32, 64), 4),
    ((1, 8, 256, 64, 128, 1024), 8),
    ((2, 8, 256, 64, 128, 1024), 8),
    ((1, 8, 128, 64, 128, 512), 8),
    ((0, 1, 128, 64, 128, 512), 0),         # single precision, more channels than fit, more threads than a launch takes
    ((1, 1, 272, 64, 128, 512), 0),
    ((1, 160000, 16, 64, 64, 16), 0),
])
def test_ffn_takes_the_faster_form(lib, shape, rows):
    f = lib._ZN4msla14ffn_block_rowsEiiiiii
    f.argtypes, f.restype = [ctypes.c_int] * 6, ctypes.c_int
    assert f(*shape) == rows


# (dtype, tokens, channels, heads, tokens an image): whether the projection reads a channel-planar x itself
@pytest.mark.parametrize("call,planar", [
    ((1, 8 * 9999, 128, 16, 9999), True), ((2, 8 * 8192, 256, 16, 8192), True), ((2, 2 * 4819, 160, 26, 4819), True), ((1, 9830, 160, 21, 9830), True),
    # many groups of output channels, each of which reads all of a large x
    ((1, 9831, 160, 21, 9831), False), ((1, 9831, 160, 20, 9831), True), ((2, 13 * 675, 256, 27, 675), False), ((2, 6 * 4611, 64, 32, 4611), False),
    # tiles of several images
    ((1, 256 * 49, 256, 16, 49), False), ((2, 131 * 81, 240, 15, 81), False), ((1, 16384, 256, 16, 64), True), ((1, 65 * 127, 256, 16, 127), False),
    ((1, 65 * 129, 256, 16, 129), True), ((1, 64 * 127, 256, 16, 127), True), ((2, 512 * 49, 128, 8, 49), True),
    ((0, 1600, 32, 4, 1600), True), ((0, 8192, 128, 8, 8192), True), ((0, 8193, 128, 8, 8193), False), ((0, 4096, 192, 12, 4096), False),
    ((1, 4096, 272, 16, 4096), False),
])
def test_projection_reads_a_planar_map_where_that_pays(lib, call, planar):
    f = lib._ZN4msla24qkv_project_takes_planarEiliii
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    assert f(*call) == planar


# (dtype, tokens, tokens an image, head-branches, channels): whether the output projection writes a channel-planar map itself
@pytest.mark.parametrize("call,planar", [
    ((1, 8 * 6144, 6144, 32, 256), True), ((2, 8 * 3551, 3551, 32, 256), True), ((1, 8 * 3551, 3551, 24, 256), True), ((1, 8 * 3551, 3551, 32, 128), True),
    ((1, 8 * 3551, 3551, 32, 256), False), ((1, 10 * 2303, 2303, 26, 320), False),      # fp16's widest form, rows that start anywhere
    ((1, 3 * 1539, 1539, 30, 208), True), ((1, 12288, 4095 + 1, 32, 256), True), ((1, 12289, 12289, 32, 256), False), ((1, 12290, 12290, 32, 256), True), ((1, 3 * 4095, 4095, 32, 256), True),
    ((1, 1 << 25, 1 << 25, 16, 128), False), ((0, 1600, 1600, 4, 32), True), ((2, 4 * 8515, 8515, 40, 512), False),
])
def test_output_projection_writes_a_planar_map_where_that_pays(lib, call, planar):
    f = lib._ZN4msla27apply_project_writes_planarEiliii
    f.argtypes, f.restype = [ctypes.c_int, ctypes.c_long, ctypes.c_int, ctypes.c_int, ctypes.c_int], ctypes.c_bool
    assert f(*call) == planar
