"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every function the
header declares, sizes layouts and scratch as documented, and rejects bad arguments before any
launch."""
import ctypes as C
import math
import os
import re
import threading

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1912_12607_amd", "csrc", "libint8t.so")
HDR = os.path.join(ROOT, "include", "int8t.h")


@pytest.fixture(scope="module")
def lib():
    if not os.path.exists(LIB):
        from paper_1912_12607_amd import build
        build.build(force=False)
    L = C.CDLL(LIB)
    L.int8t_code_bytes.restype = C.c_size_t
    L.int8t_workspace_bytes.restype = C.c_size_t
    L.int8t_quantize_workspace_bytes.restype = C.c_size_t
    L.int8t_status_string.restype = C.c_char_p
    L.int8t_dclr_scale.restype = C.c_double
    L.int8t_dclr_scale.argtypes = [C.c_double] * 3
    return L


class Desc(C.Structure):
    _fields_ = [(n, C.c_int) for n in
                ("N", "C", "H", "W", "K", "R", "S", "stride_h", "stride_w", "pad_h", "pad_w", "groups")]


def dims(*v):
    return (C.c_int * 4)(*v)


def test_every_declared_symbol_is_exported(lib):
    text = open(HDR).read()
    names = set(re.findall(r"\b(int8t_[a-z_0-9]+)\s*\(", text))
    assert {"int8t_quantize", "int8t_dsgc_clip", "int8t_conv_fwd", "int8t_conv_bwd_data",
            "int8t_conv_bwd_weight"} <= names
    for n in names:
        assert hasattr(lib, n), n


def test_binding_names_match_header():
    text = open(os.path.join(ROOT, "paper_1912_12607_amd", "binding.py")).read()
    hdr = set(re.findall(r"\b(int8t_[a-z_0-9]+)\s*\(", open(HDR).read()))
    for n in hdr:
        assert f"def {n}(" in text, n


# A stem in its space-to-depth form (C <= 4 under stride 2 x 2) may have the geometry of a plain layer on 4 C channels: the scratch
# of either, which follows from its plan, does not depend on what the thread planned before.
@pytest.mark.parametrize("stem,plain", [((3, 32, 32, 12, 5, 5, 2, 2), (12, 16, 16, 12, 3, 3, 1, 1)), ((3, 32, 32, 12, 6, 6, 2, 2), (12, 16, 16, 12, 3, 3, 1, 1)),
                                        ((4, 48, 47, 24, 9, 9, 4, 4), (16, 24, 24, 24, 5, 5, 2, 2)), ((2, 28, 28, 40, 13, 1, 6, 0), (8, 14, 14, 40, 7, 1, 3, 0))])
def test_plans_of_stems_and_plain_layers_of_one_geometry(lib, stem, plain):
    layers = []
    for (c, h, w, k, r, s, ph, pw), st in ((stem, 2), (plain, 1)):
        layers.append(Desc(2, c, h, w, k, r, s, st, st, ph, pw, 1))

    def sizes(*order):
        out = {}

        def plan():
            for i in order:
                out[i] = lib.int8t_workspace_bytes(4, C.byref(layers[i]), C.c_size_t(0), 0)
        t = threading.Thread(target=plan)        # (plans are kept per thread)
        t.start()
        t.join()
        return out
    alone = {**sizes(0), **sizes(1)}
    assert min(alone.values()) > 0
    assert sizes(0, 1) == alone and sizes(1, 0) == alone


# The kernels deal chunks to shares as chunk = chunks * share / shares in 32 bits: twice the shares are only taken where that stays below 2^31
# (2.6 million chunks of 32 lines, 512 shares by the library's own choice; an ordinary layer).
@pytest.mark.parametrize("shape,chunks", [((40, 16, 1 << 21, 1, 16, 1, 3, 1, 1, 0, 1, 1), 40 * (1 << 21) // 32), ((64, 256, 14, 14, 256, 3, 3, 1, 1, 1, 1, 1), 28)])
def test_twice_the_shares_stay_within_32_bits(lib, shape, chunks):
    d = Desc(*shape)
    share = 4 * d.K * d.C * d.R * d.S

    def shares():
        return lib.int8t_workspace_bytes(4, C.byref(d), C.c_size_t(0), 0) // share
    own = shares()
    assert lib.int8t_conv_select_variant(4, C.byref(d), 7) == 0
    try:
        more = shares()
    finally:
        assert lib.int8t_conv_select_variant(4, C.byref(d), 0) == 0
    assert more == (2 * own if chunks * 2 * own < 1 << 31 and 2 * own <= chunks and 2 * own <= 4096 else own)
    assert chunks * more < 1 << 31


# Bands and backward-weight share a launch up to 220 MB of codes and input gradient, which the last-level cache holds, and run apart above.
@pytest.mark.parametrize("ch,K,R,batch,form", [(64, 64, 3, 180, 11), (64, 64, 3, 190, 0), (64, 64, 1, 180, 11), (64, 64, 1, 241, 0), (64, 256, 1, 121, 11), (64, 256, 1, 160, 0)])
@pytest.mark.parametrize("parts", [192, 224])
def test_large_band_layers_run_apart(lib, ch, K, R, batch, form, parts):
    d = Desc(batch, ch, 56, 56, K, R, R, 1, 1, R // 2, R // 2, 1)
    assert (batch * 3136 * (5 * ch + K) <= 220e6) == (form == 11)
    assert lib.int8t_layer_step_form(C.byref(d), parts) == form


def test_code_bytes(lib):
    assert lib.int8t_code_bytes(dims(2, 16, 16, 16), 0) == 2 * 16 * 16 * 16
    assert lib.int8t_code_bytes(dims(64, 24, 56, 56), 0) == 64 * 56 * 56 * 32      # C padded to 32
    assert lib.int8t_code_bytes(dims(64, 24, 56, 56), 2) == 64 * 24 * 56 * 56      # planar
    k, c, r, s = 70, 33, 3, 3
    n1 = k * r * s * 48
    assert lib.int8t_code_bytes(dims(k, c, r, s), 1) == ((n1 + 255) // 256) * 256 + c * r * s * 80
    assert lib.int8t_code_bytes(dims(k, c, r, s), 3) == k * c * r * s
    assert lib.int8t_code_bytes(dims(0, 1, 1, 1), 0) == 0
    assert lib.int8t_code_bytes(dims(2, 2, 2, 2), 7) == 0


def test_workspace_sizes(lib):
    assert lib.int8t_quantize_workspace_bytes(dims(2, 16, 16, 16), 0) >= 4096 + 8 * 24
    assert lib.int8t_quantize_workspace_bytes(dims(2, 16, 16, -1), 0) == 0
    # clip search: absmax partials + 32 accumulator sets x 64 candidates x 3 words + sum-of-squares partials
    assert lib.int8t_workspace_bytes(1, None, C.c_size_t(1 << 20), 32) >= 1024 * 4 + 32 * 64 * 3 * 8 + 8 + 1024 * 8
    d = Desc(64, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1, 1)
    assert lib.int8t_workspace_bytes(4, C.byref(d), C.c_size_t(0), 0) >= 64 * 9 * 64 * 4
    assert lib.int8t_workspace_bytes(2, C.byref(d), C.c_size_t(0), 0) == 0
    # forward / backward-data of a layer with few output tiles: optional scratch for a split reduction,
    # a whole number of int32 result copies
    few = Desc(64, 768, 17, 17, 192, 3, 3, 2, 2, 0, 0, 1)
    nf = lib.int8t_workspace_bytes(2, C.byref(few), C.c_size_t(0), 0)
    assert nf >= 2 * 64 * 192 * 8 * 8 * 4 and nf % (64 * 192 * 8 * 8 * 4) == 0
    bad = Desc(64, 64, 56, 56, 64, 3, 3, 1, 1, 1, 1, 2)     # grouped but not depthwise
    assert lib.int8t_workspace_bytes(4, C.byref(bad), C.c_size_t(0), 0) == 0


def test_dclr_scale_golden_table(lib):
    # the library's host function against the fixture written from Eq.7 (tests/golden/dclr_eq7.txt)
    n = 0
    for line in open(os.path.join(ROOT, "tests", "golden", "dclr_eq7.txt")):
        if line.startswith("#"):
            continue
        alpha, beta, d, phi = (float(v) for v in line.split())
        assert lib.int8t_dclr_scale(d, alpha, beta) == pytest.approx(phi, rel=1e-15)
        n += 1
    assert n == 36


def test_dclr_scale_eq7(lib):
    assert lib.int8t_dclr_scale(0.0, 20.0, 0.1) == 1.0
    assert lib.int8t_dclr_scale(0.05, 20.0, 0.1) == pytest.approx(math.exp(-1.0), rel=1e-15)
    assert lib.int8t_dclr_scale(0.5, 20.0, 0.1) == 0.1


def test_argument_errors_before_any_launch(lib):
    vp = C.c_void_p
    fake = vp(0x1000)            # aligned, never dereferenced on these paths
    odd = vp(0x1004)
    q = lib.int8t_quantize
    q.restype = C.c_int
    q.argtypes = [vp, C.POINTER(C.c_int), C.c_int, vp, C.c_int, C.c_uint64, vp, vp, vp, vp, C.c_size_t, vp]
    assert q(None, dims(1, 1, 1, 1), 0, None, 0, 0, fake, fake, None, fake, 1 << 20, None) == 1
    assert q(fake, dims(1, 0, 1, 1), 0, None, 0, 0, fake, fake, None, fake, 1 << 20, None) == 2
    assert q(fake, dims(1, 1, 1, 1), 5, None, 0, 0, fake, fake, None, fake, 1 << 20, None) == 3
    assert q(fake, dims(1, 1, 1, 1), 0, None, 2, 0, fake, fake, None, fake, 1 << 20, None) == 3
    assert q(odd, dims(1, 1, 1, 1), 0, None, 0, 0, fake, fake, None, fake, 1 << 20, None) == 3
    assert q(fake, dims(1, 1, 1, 1), 0, None, 0, 0, fake, fake, None, fake, 16, None) == 4
    assert q(fake, dims(1, 1, 1, 1), 0, None, 0, 0, fake, fake, None, None, 0, None) == 1
    g = lib.int8t_dsgc_clip
    g.restype = C.c_int
    g.argtypes = [vp, C.c_size_t, vp, C.c_int, C.c_int, C.c_uint64, vp, vp, vp, vp, C.c_size_t, vp]
    assert g(fake, 100, fake, 0, 1, 0, fake, fake, None, fake, 1 << 24, None) == 3
    assert g(fake, 100, fake, 65, 1, 0, fake, fake, None, fake, 1 << 24, None) == 3
    assert g(fake, 0, fake, 4, 1, 0, fake, fake, None, fake, 1 << 24, None) == 2
    assert g(fake, 100, None, 4, 1, 0, fake, fake, None, fake, 1 << 24, None) == 1
    assert g(fake, 100, fake, 4, 1, 0, fake, fake, None, fake, 64, None) == 4
    for name in ("int8t_conv_fwd", "int8t_conv_bwd_data", "int8t_conv_bwd_weight"):
        f = getattr(lib, name)
        f.restype = C.c_int
        f.argtypes = [C.POINTER(Desc), vp, vp, vp, vp, vp, vp, vp, C.c_size_t, vp]
        good = Desc(1, 4, 5, 5, 4, 3, 3, 1, 1, 1, 1, 1)
        assert f(None, fake, fake, fake, fake, fake, None, fake, 1 << 20, None) == 1
        assert f(C.byref(Desc(1, 4, 5, 5, 4, 3, 3, 0, 1, 1, 1, 1)), fake, fake, fake, fake, fake, None, fake, 1 << 20, None) == 2
        assert f(C.byref(Desc(1, 4, 5, 5, 6, 3, 3, 1, 1, 1, 1, 2)), fake, fake, fake, fake, fake, None, fake, 1 << 20, None) == 2
        assert f(C.byref(Desc(1, 4, 2, 2, 4, 7, 7, 1, 1, 0, 0, 1)), fake, fake, fake, fake, fake, None, fake, 1 << 20, None) == 2
        assert f(C.byref(good), None, fake, fake, fake, fake, None, fake, 1 << 20, None) == 1
        assert f(C.byref(good), odd, fake, fake, fake, fake, None, fake, 1 << 20, None) == 3
    f = lib.int8t_conv_bwd_weight
    assert f(C.byref(Desc(1, 4, 5, 5, 4, 3, 3, 1, 1, 1, 1, 1)), fake, fake, fake, fake, fake, None, fake, 8, None) == 4
    assert lib.int8t_status_string(4) == b"workspace too small"


def test_profile_entry_points_without_launches(lib):
    class KT(C.Structure):
        _fields_ = [("name", C.c_char_p), ("launches", C.c_int), ("total_ms", C.c_double)]
    assert lib.int8t_profile_start(b"no_such_kernel") == 3          # INT8T_ERR_ARG, timing stays off
    assert lib.int8t_profile_start(b"dsgc_sweep_kernel") == 0
    n = C.c_int(-1)
    buf = (KT * 4)()
    assert lib.int8t_profile_stop(buf, 4, C.byref(n)) == 0 and n.value == 0
    assert lib.int8t_profile_start(None) == 0
    assert lib.int8t_profile_stop(None, 0, C.byref(n)) == 0 and n.value == 0
    assert lib.int8t_profile_stop(None, 4, C.byref(n)) == 3          # capacity without a buffer
    assert lib.int8t_profile_start_sampled(b"band_kernel", 0) == 3   # every >= 1
    assert lib.int8t_profile_start_sampled(b"igemm_reduce_kernel", 5) == 0
    assert lib.int8t_profile_stop(buf, 4, C.byref(n)) == 0 and n.value == 0


def test_quantize_batch_argument_errors(lib):
    class Item(C.Structure):
        _fields_ = [("x_dev", C.c_void_p), ("dims", C.c_int * 4), ("kind", C.c_int), ("clip_dev", C.c_void_p),
                    ("q_dev", C.c_void_p), ("scale_dev", C.c_void_p), ("mode", C.c_int), ("seed", C.c_uint64)]
    lib.int8t_quantize_batch_workspace_bytes.restype = C.c_size_t
    lib.int8t_quantize_batch_workspace_bytes.argtypes = [C.c_int, C.POINTER(Item)]
    f = lib.int8t_quantize_batch
    f.restype = C.c_int
    f.argtypes = [C.c_int, C.POINTER(Item), C.c_void_p, C.c_size_t, C.c_void_p]
    items = (Item * 2)()
    for it in items:
        it.x_dev, it.q_dev, it.scale_dev, it.kind = 0x1000, 0x2000, 0x3000, 0
        it.dims[:] = [1, 16, 4, 4]
    assert lib.int8t_quantize_batch_workspace_bytes(2, items) == 2 * 4096
    assert lib.int8t_quantize_batch_workspace_bytes(0, items) == 0
    assert lib.int8t_quantize_batch_workspace_bytes(9, items) == 0
    assert f(2, None, 0x4000, 1 << 20, None) == 1                  # INT8T_ERR_NULL
    assert f(0, items, 0x4000, 1 << 20, None) == 3                 # INT8T_ERR_ARG: count
    assert f(9, items, 0x4000, 1 << 20, None) == 3
    assert f(2, items, None, 0, None) == 1                         # absmax needs the scratch
    assert f(2, items, 0x4000, 4096, None) == 4                    # INT8T_ERR_WORKSPACE
    items[1].kind = 9
    assert f(2, items, 0x4000, 1 << 20, None) == 3
    items[1].kind = 0
    items[1].mode = 2                                              # neither nearest-even nor stochastic
    assert f(2, items, 0x4000, 1 << 20, None) == 3
    items[1].mode = 1
    items[1].dims[2] = 0
    assert f(2, items, 0x4000, 1 << 20, None) == 2                 # INT8T_ERR_SHAPE
    items[1].dims[2] = 4
    items[0].q_dev = 0x2004
    assert f(2, items, 0x4000, 1 << 20, None) == 3                 # alignment
    items[0].q_dev = 0x2000
    # ... with the first phase of a clip search in the same launch
    lib.int8t_workspace_bytes.restype = C.c_size_t
    lib.int8t_workspace_bytes.argtypes = [C.c_int, C.c_void_p, C.c_size_t, C.c_int]
    need = lib.int8t_workspace_bytes(1, None, 1000, 32)            # INT8T_OP_DSGC
    g = lib.int8t_quantize_batch_prepare
    g.restype = C.c_int
    g.argtypes = [C.c_int, C.POINTER(Item), C.c_void_p, C.c_size_t, C.c_void_p, C.c_size_t, C.c_void_p, C.c_size_t, C.c_void_p]
    assert g(2, items, 0x4000, 1 << 20, None, 1000, 0x100000, need, None) == 1       # g is required
    assert g(2, items, 0x4000, 1 << 20, 0x8000, 1000, None, 0, None) == 1            # ... and the search's scratch
    assert g(2, items, 0x4000, 1 << 20, 0x8000, 0, 0x100000, need, None) == 2        # n == 0
    assert g(2, items, 0x4000, 1 << 20, 0x8004, 1000, 0x100000, need, None) == 3     # alignment of g
    assert g(2, items, 0x4000, 1 << 20, 0x8000, 1000, 0x100000, need - 1, None) == 4
    assert g(0, items, 0x4000, 1 << 20, 0x8000, 1000, 0x100000, need, None) == 3     # the batch's own checks still apply


def test_dsgc_two_phase_argument_errors(lib):
    vp = C.c_void_p
    prep, search = lib.int8t_dsgc_prepare, lib.int8t_dsgc_search
    prep.restype = search.restype = C.c_int
    prep.argtypes = [vp, C.c_size_t, vp, C.c_size_t, vp]
    search.argtypes = [vp, C.c_size_t, vp, C.c_int, C.c_int, C.c_uint64, vp, vp, vp, vp, C.c_size_t, vp]
    need = lib.int8t_workspace_bytes(1, None, C.c_size_t(1000), 32)
    assert prep(None, 1000, 0x4000, need, None) == 1
    assert prep(0x1000, 0, 0x4000, need, None) == 2
    assert prep(0x1004, 1000, 0x4000, need, None) == 3
    assert prep(0x1000, 1000, 0x4000, need - 1, None) == 4
    assert search(0x1000, 1000, None, 32, 1, 0, 0x2000, 0x3000, None, 0x4000, need, None) == 1
    assert search(0x1000, 1000, 0x5000, 65, 1, 0, 0x2000, 0x3000, None, 0x4000, need, None) == 3
    assert search(0x1000, 1000, 0x5000, 32, 1, 0, 0x2000, 0x3000, None, 0x4000, need - 1, None) == 4


# int8t_layer_step with made-up addresses: every call below has to end in one of the argument checks, before a launch.
LAYER_STEP_ADDRESSES = {name: 0x100000 + 0x1000 * i for i, name in enumerate(
    ("x", "w", "dy", "xq", "wq", "dyq", "sx", "sw", "sdy", "ratios", "clip", "dev_search", "dev_all", "dev_final",
     "y", "dx", "dw", "y_acc", "dx_acc", "dw_acc"))}
LAYER_STEP_ADDRESSES.update({"ws_quant": 0x10000000, "ws_dy": 0x20000000, "ws_fwd": 0x30000000, "ws_bwd_data": 0x40000000,
                             "ws_bwd_weight": 0x50000000})


def layer_step_status(desc, parts, **fields):
    from paper_1912_12607_amd import binding as B
    b = B.LayerBuffers(n_cand=32, **LAYER_STEP_ADDRESSES)
    for name in ("ws_quant", "ws_dy", "ws_fwd", "ws_bwd_data", "ws_bwd_weight"):
        setattr(b, name + "_bytes", 1 << 24)
    for name, v in fields.items():
        setattr(b, name, v)
    return B.lib.int8t_layer_step(C.byref(desc), C.byref(b), parts, 0, None)


def test_layer_step_batch_limit_of_the_codes():
    """The channels-last quantizer takes 65535 images; planar codes (depthwise layers) have no such limit."""
    from paper_1912_12607_amd import binding as B
    dense, planar = B.make_desc(70000, 8, 5, 5, 8, 3, 3, (1, 1), (1, 1)), B.make_desc(70000, 8, 5, 5, 8, 3, 3, (1, 1), (1, 1), 8)
    parts = B.STEP_QUANT_G | B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    assert layer_step_status(dense, parts) == 2                            # INT8T_ERR_SHAPE, as int8t_quantize says
    assert layer_step_status(planar, parts, ws_dy_bytes=16) == 4           # past that check: INT8T_ERR_WORKSPACE

def test_layer_step_unused_pointers_may_be_null():
    """A pointer that no part of the call uses may be NULL; one that a part uses may not."""
    from paper_1912_12607_amd import binding as B
    d = B.make_desc(2, 16, 8, 8, 16, 3, 3, (1, 1), (1, 1))
    used = {B.STEP_ABSMAX: {"x", "w", "ws_quant"},
            B.STEP_ABSMAX | B.STEP_PREPARE: {"x", "w", "dy", "ws_quant", "ws_dy"},
            B.STEP_SEARCH: {"dy", "ratios", "clip", "dev_search", "ws_dy"},
            B.STEP_QUANT_XW: {"x", "w", "xq", "wq", "sx", "sw", "ws_quant"},
            B.STEP_QUANT_G: {"dy", "clip", "dyq", "sdy", "dev_final", "ws_dy"},
            B.STEP_BWD_WEIGHT: {"xq", "sx", "dyq", "sdy", "dw", "ws_bwd_weight"}}
    for parts, names in used.items():
        unused = {n: None for n in LAYER_STEP_ADDRESSES if n not in names}
        # with scratch too small for every part: the last check before the launches, so all others have passed
        small = {n + "_bytes": 16 for n in ("ws_quant", "ws_dy", "ws_bwd_weight")}
        assert layer_step_status(d, parts, **unused, **small) == 4
        for n in names - {"dev_final"}:
            assert layer_step_status(d, parts, **{**unused, n: None}) == 1, (parts, n)
    assert layer_step_status(d, B.STEP_FWD, xq=None) == 1 and layer_step_status(d, B.STEP_BWD_DATA, dx=None) == 1

def test_layer_step_checks_everything_before_the_first_launch():
    from paper_1912_12607_amd import binding as B
    d = B.make_desc(2, 16, 8, 8, 16, 3, 3, (1, 1), (1, 1))
    by = {"x": 4, "w": 4, "dy": 4, "xq": 4, "wq": 4, "dyq": 4, "sx": 2, "sw": 2, "sdy": 2, "ratios": 2, "clip": 2, "dev_search": 4, "dev_all": 4,
          "y": 4, "dx": 4, "dw": 4, "y_acc": 2, "dx_acc": 2, "dw_acc": 2, "ws_quant": 4, "ws_dy": 4, "ws_fwd": 4, "ws_bwd_data": 4,
          "ws_bwd_weight": 4}
    for dev_final in (LAYER_STEP_ADDRESSES["dev_final"], None):       # g_z quantized by itself, and in one launch with a and W
        for n, off in by.items():
            assert layer_step_status(d, B.STEP_ALL, **{"dev_final": dev_final, n: LAYER_STEP_ADDRESSES[n] + off}) == 3, n
        for ws, nbytes in (("ws_quant", 4096), ("ws_dy", 4096), ("ws_bwd_weight", 16)):
            assert layer_step_status(d, B.STEP_ALL, dev_final=dev_final, **{ws + "_bytes": nbytes}) == 4, ws
    convs = B.STEP_FWD | B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    for n in ("xq", "wq", "dyq", "y", "dx", "dw", "y_acc", "dx_acc", "dw_acc"):
        assert layer_step_status(d, convs, **{n: LAYER_STEP_ADDRESSES[n] + by[n]}) == 3, n
    assert layer_step_status(d, B.STEP_ALL, n_cand=0) == 3 and layer_step_status(d, B.STEP_ALL, n_cand=65) == 3
    assert layer_step_status(d, 0) == 3 and layer_step_status(d, 256) == 3 and layer_step_status(d, B.STEP_PREPARE) == 3
    assert B.lib.int8t_layer_step(C.byref(d), None, B.STEP_ALL, 0, None) == 1
    grouped = B.make_desc(2, 16, 8, 8, 16, 3, 3, (1, 1), (1, 1), 4)
    assert layer_step_status(grouped, B.STEP_ALL) == 2

def test_layer_step_scratch_of_the_search_and_of_the_maxima_overlap():
    from paper_1912_12607_amd import binding as B
    d = B.make_desc(2, 16, 8, 8, 16, 3, 3, (1, 1), (1, 1))
    need, q = B.int8t_workspace_bytes(B.OP_DSGC, None, 2 * 16 * 64, 32), LAYER_STEP_ADDRESSES["ws_quant"]
    for parts in (B.STEP_ALL, B.STEP_ABSMAX | B.STEP_PREPARE, B.STEP_ABSMAX | B.STEP_SEARCH, B.STEP_SEARCH | B.STEP_QUANT_XW):
        for ws_dy in (q, q + 8192 - 16, q - need + 16):
            assert layer_step_status(d, parts, ws_dy=ws_dy) == 3
        for ws_dy in (q + 8192, q - need):          # side by side: on to the next check
            assert layer_step_status(d, parts | B.STEP_BWD_DATA, ws_dy=ws_dy, dx=None) == 1


def test_unpack_codes_matches_the_documented_layouts():
    """int8t_unpack_codes against the layout formulas of include/int8t.h written out with numpy."""
    import numpy as np

    from paper_1912_12607_amd import binding as B
    r = np.random.RandomState(3)
    N, Cc, H, W = 3, 24, 5, 7
    q = r.randint(-127, 128, size=(N, Cc, H, W)).astype(np.int8)
    packed = np.zeros((N, H, W, 32), np.int8)
    packed[..., :Cc] = q.transpose(0, 2, 3, 1)
    out, bad = B.int8t_unpack_codes(packed.reshape(-1), (N, Cc, H, W), B.ACT)
    assert bad == 0 and np.array_equal(out, q)
    packed[1, 2, 3, 30] = 1
    assert B.int8t_unpack_codes(packed.reshape(-1), (N, Cc, H, W), B.ACT)[1] == 1
    K, Cg, R, S = 20, 40, 3, 2
    w = r.randint(-127, 128, size=(K, Cg, R, S)).astype(np.int8)
    n1 = K * R * S * 48
    buf = np.zeros(((n1 + 255) // 256) * 256 + Cg * R * S * 32, np.int8)
    a = np.zeros((K, R, S, 48), np.int8)
    a[..., :Cg] = w.transpose(0, 2, 3, 1)
    b = np.zeros((Cg, R, S, 32), np.int8)
    b[..., :K] = w.transpose(1, 2, 3, 0)
    buf[:n1] = a.reshape(-1)
    buf[((n1 + 255) // 256) * 256:] = b.reshape(-1)
    assert buf.size == B.int8t_code_bytes((K, Cg, R, S), B.WGT)
    for copy in (0, 1):
        out, bad = B.int8t_unpack_codes(buf, (K, Cg, R, S), B.WGT, copy)
        assert bad == 0 and np.array_equal(out, w)
    out, _ = B.int8t_unpack_codes(w.reshape(-1), (K, Cg, R, S), B.WGT_PLANAR)
    assert np.array_equal(out, w)
    with pytest.raises(B.Int8tError):
        B.int8t_unpack_codes(buf, (K, Cg, R, S), B.ACT_PLANAR, 1)


def test_layer_backward_arguments():
    from paper_1912_12607_amd import binding as B
    d, b = B.make_desc(2, 16, 8, 8, 32, 3, 3, (1, 1), (1, 1)), B.LayerBuffers()

    def call(parts, db=None):
        return B.lib.int8t_layer_backward(C.byref(d), C.byref(b), parts, 0, db, None)

    null, bad = 1, 3                               # INT8T_ERR_NULL, INT8T_ERR_ARG
    for parts in (0, 256, B.STEP_ABSMAX, B.STEP_QUANT_XW | B.STEP_QUANT_G, B.STEP_FWD, B.STEP_PREPARE, B.STEP_SEARCH, B.STEP_ALL):
        assert call(parts) == bad
    assert call(B.STEP_BWD_DATA, 4096) == bad      # a bias gradient of a layer with more than one output pixel
    assert call(B.STEP_PREPARE | B.STEP_SEARCH) == null and call(B.STEP_QUANT_G) == null and call(B.STEP_BWD_WEIGHT) == null


# The grid of the quantizer of N,H,W,Cp codes (internal functions of the library): every tile once.  Images beyond the batch may fill up
# the last eight that are walked side by side; the rows of 1 x 1 images are one grid over the whole batch.
@pytest.mark.parametrize("N,Cc,H,W", [(256, 1000, 1, 1), (64, 1000, 1, 1), (8192, 1000, 1, 1), (2100, 996, 1, 1), (128, 20, 1, 1), (16, 3, 1, 1),
                                     (8, 24, 17, 17), (31, 24, 17, 17), (15, 18, 17, 19), (64, 288, 35, 35), (8, 3, 33, 31), (64, 64, 56, 56)])
def test_quantizer_grid_runs_every_tile_once(lib, N, Cc, H, W):
    grid, count = getattr(lib, "_ZN5int8t10quant_gridEiPKiPiS2_S2_"), getattr(lib, "_ZN5int8t16quant_blocks_actEiii")
    g = [C.c_int() for _ in range(3)]
    grid(0, dims(N, Cc, H, W), *[C.byref(v) for v in g])
    gx, gy, gz = (v.value for v in g)
    tiles = count(N, (Cc + 15) // 16 * 16, H * W)
    assert tiles <= gx * gy * gz < tiles + (1 if H * W == 1 else 8 * gx * gy)
    if H * W > 1:
        assert tiles == gx * gy * N and gz in (N, (N + 7) // 8 * 8)
