"""GPU parity at the borders of the library's own choices: the sizes at which a kernel's launch shape or inner path
changes, against the CPU oracle.  Bars as in test_gpu_parity.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_1912_12607_amd import binding as B  # noqa: E402
from paper_1912_12607_amd import inputs  # noqa: E402
from paper_1912_12607_amd.autograd import Int8Conv2d  # noqa: E402
from paper_1912_12607_amd.step import LayerStep  # noqa: E402
from test_gpu_parity import DEV, REL_TOL, RTN, STO, check_dsgc, dev, gpu_dsgc, pack_act, pack_wgt  # noqa: E402


# The sweep runs blocks of 4 waves up to 1024 wave-iterations of 256 elements and blocks of 16 above, and leaves the clip
# at 127 out for eights of candidates that clip none of a wave's 256 elements: "flat" clips in every eight but the first
# candidate, "one" has a single large element (its wave clips, the others do not), "unsorted" mixes small and large
# candidates in every eight.
@pytest.mark.parametrize("n,kind", [(262144, "flat"), (262145, "one"), (262400, "tail"), (262401, "unsorted"), (1050627, "tail"),
                                    (1050624, "one"), (70001, "huge"), (70001, "tiny")])
def test_dsgc_block_sizes_and_clip_free_eights(n, kind):
    r = np.random.RandomState(n % 1000)
    g = (r.standard_t(3, size=n) * 1e-3).astype(np.float32)
    ratios = inputs.default_ratios(32)
    if kind == "flat":
        g = (np.sign(r.standard_normal(n)) * r.uniform(0.9, 1.0, size=n)).astype(np.float32)
    elif kind == "one":
        g[n // 2] = 2.0
    elif kind == "unsorted":
        ratios = r.permutation(ratios)
    elif kind == "huge":          # max|g| close to the largest fp32 number: a doubled element would be infinite
        g = (g / np.abs(g).max() * np.float32(3.3e38)).astype(np.float32)
    elif kind == "tiny":          # the quantizer scales by 127 * 2^24 / c: finite down to c = 7e-30, the smallest candidate is max / 216
        g = (g / np.abs(g).max() * np.float32(1e-26)).astype(np.float32)
    check_dsgc(g, ratios, STO, seed=n)
    check_dsgc(g, ratios, RTN, seed=n)


# An infinite gradient element makes every clip value infinite and every scale 0: all codes are 0, so the deviation is 1 by
# definition (a zero vector), whatever else the gradient holds.  The waves that hold the infinity work with clipped candidates,
# the others without; large finite elements stand beside it, and a NaN, whose code is 0 as well.
@pytest.mark.parametrize("n_cand", [32, 7])
@pytest.mark.parametrize("with_nan", [False, True])
def test_dsgc_infinite_element(n_cand, with_nan):
    n = 5003
    g = (np.random.RandomState(4).standard_t(3, size=n) * 1e-3).astype(np.float32)
    g[3] = np.inf
    g[5] = -3e38
    if with_nan:
        g[[6, 4000]] = np.nan
    clip, d, da = gpu_dsgc(g, inputs.default_ratios(n_cand), STO, 9)
    assert np.isinf(clip) and d == 1.0 and np.all(np.asarray(da) == 1.0)


def conv_pass_elementwise(op, desc, od, xq, wq, dyq, with_acc):
    """One pass of the library on codes against the oracle: fp32 result (and accumulators)."""
    s = [dev(np.array([v], np.float32)) for v in (0.013, 0.0021, 3.1e-5)]
    if op == B.OP_CONV_FWD:
        want64, call, args, s1, s2 = oracle.conv_fwd(od, xq, wq), B.int8t_conv_fwd, (dev(pack_act(xq)), s[0], dev(pack_wgt(wq)), s[1]), s[0], s[1]
    elif op == B.OP_CONV_BWD_DATA:
        want64, call, args, s1, s2 = (oracle.conv_bwd_data(od, dyq, wq), B.int8t_conv_bwd_data,
                                      (dev(pack_act(dyq)), s[2], dev(pack_wgt(wq)), s[1]), s[2], s[1])
    else:
        want64, call, args, s1, s2 = (oracle.conv_bwd_weight(od, xq, dyq), B.int8t_conv_bwd_weight,
                                      (dev(pack_act(xq)), s[0], dev(pack_act(dyq)), s[2]), s[0], s[2])
    want, ov = oracle.wrap32(want64)
    assert ov == 0
    out = torch.full(want.shape, 7.0, dtype=torch.float32, device=DEV)
    acc = torch.full(want.shape, 7, dtype=torch.int32, device=DEV) if with_acc else None
    ws = torch.empty(max(256, B.int8t_workspace_bytes(op, desc)), dtype=torch.uint8, device=DEV)
    call(desc, *args, out, acc, ws)
    torch.cuda.synchronize()
    if with_acc:
        assert np.array_equal(acc.cpu().numpy(), want)
    ref = oracle.dequant(want, np.float32(s1.item()), np.float32(s2.item()))
    assert np.all(np.abs(out.cpu().numpy() - ref) <= REL_TOL * np.abs(ref))


def random_layer(shape, seed):
    N, C, H, W, K, R, S, stride, pad = shape
    r = np.random.RandomState(seed)
    desc = B.make_desc(N, C, H, W, K, R, S, (stride, stride), pad)
    od = oracle.make_desc(N, C, H, W, K, R, S, (stride, stride), pad)
    P, Q = (H + 2 * pad[0] - R) // stride + 1, (W + 2 * pad[1] - S) // stride + 1
    codes = [r.randint(-127, 128, size=s).astype(np.int8) for s in ((N, C, H, W), (K, C, R, S), (N, K, P, Q))]
    return desc, od, codes


# Results staged through LDS (planes of whole 16-byte groups), tiles that end inside an image or beyond the last one, ragged
# rows, and the column tiles of an XCD in a run (rows of no whole lines, short reduction, at least 96 column tiles), forward
# and backward-data, plain and in 2 x 2 cells.
@pytest.mark.parametrize("shape", [(3, 40, 6, 6, 150, 1, 1, 1, (0, 0)), (5, 200, 10, 10, 72, 3, 3, 1, (1, 1)), (64, 24, 14, 14, 144, 1, 1, 1, (0, 0)),
                                   (66, 130, 14, 14, 80, 1, 1, 1, (0, 0)), (33, 70, 20, 20, 96, 1, 1, 2, (0, 0)), (64, 80, 15, 15, 70, 1, 1, 1, (0, 0))])
@pytest.mark.parametrize("with_acc", [False, True])
def test_staged_results_and_column_runs(shape, with_acc):
    desc, od, (xq, wq, dyq) = random_layer(shape, shape[1])
    for variant in (B.VARIANT_AUTO, B.VARIANT_WIDE_SQ128, B.VARIANT_WIDE_SQ128_DEEP, B.VARIANT_WIDE_128X64, B.VARIANT_WIDE128):
        for op in (B.OP_CONV_FWD, B.OP_CONV_BWD_DATA):
            B.int8t_conv_select_variant(op, desc, variant)
            try:
                conv_pass_elementwise(op, desc, od, xq, wq, dyq, with_acc)
            finally:
                B.int8t_conv_select_variant(op, desc, B.VARIANT_AUTO)


# Five taps along a line (a ring stage of 6 positions): lines shorter and longer than a stage, any padding, ragged channel tiles.
@pytest.mark.parametrize("shape", [(3, 20, 9, 9, 40, 5, 5, 1, (2, 2)), (2, 70, 8, 13, 130, 1, 5, 1, (0, 2)), (5, 33, 12, 7, 70, 5, 1, 1, (1, 0)),
                                   (40, 16, 5, 5, 24, 5, 5, 1, (0, 0)), (1, 100, 6, 20, 65, 5, 5, 1, (4, 4))])
def test_backward_weight_five_taps(shape):
    desc, od, (xq, wq, dyq) = random_layer(shape, 7)
    assert B.int8t_conv_variant_ok(B.OP_CONV_BWD_WEIGHT, desc, B.VARIANT_WGRAD_LINES)
    for variant in (B.VARIANT_AUTO, B.VARIANT_WGRAD_LINES, B.VARIANT_WGRAD_MORE):
        B.int8t_conv_select_variant(B.OP_CONV_BWD_WEIGHT, desc, variant)
        try:
            conv_pass_elementwise(B.OP_CONV_BWD_WEIGHT, desc, od, xq, wq, dyq, True)
        finally:
            B.int8t_conv_select_variant(B.OP_CONV_BWD_WEIGHT, desc, B.VARIANT_AUTO)


# The three passes of a step in one launch: both tile widths, 1, 3, 5 and 7 taps along either axis, planes of whole 16-byte
# groups and others, ragged rows and columns, backward-weight grids that are no multiple of the 8 XCDs.  Against the three
# calls one by one, which the other tests hold against the oracle, bit for bit -- and that the launch is the one under test.
TOGETHER_DENSE = [((2, 16, 16, 16, 32, 3, 3), True), ((64, 256, 14, 14, 256, 3, 3), True), ((32, 48, 35, 35, 64, 5, 5), True),
                  ((3, 130, 17, 17, 200, 1, 7), True), ((5, 70, 9, 11, 129, 7, 1), True), ((1, 300, 1, 1, 65, 1, 1), True),
                  ((64, 40, 28, 28, 500, 1, 3), True), ((64, 1000, 14, 14, 260, 1, 1), True), ((16, 64, 56, 56, 64, 3, 3), True),
                  ((48, 64, 56, 56, 64, 3, 3), False), ((64, 768, 17, 17, 768, 1, 7), False), ((2, 64, 9, 9, 64, 3, 5), True),
                  ((64, 96, 14, 14, 576, 1, 1), True), ((3, 50, 9, 11, 30, 1, 1), True), ((5, 33, 12, 8, 40, 5, 3), True),
                  ((64, 24, 56, 56, 144, 1, 1), False),
                  # backward-weight on image granules, one of several taps per block (and the narrow 1x1 layers above)
                  ((5, 33, 12, 8, 40, 4, 4), True), ((3, 40, 9, 11, 50, 2, 2), True), ((2, 24, 10, 19, 72, 1, 9), True)]
# planes alone and several to a block, rows of whole dwords and others, channel groups; planes that backward-weight does not prefetch
TOGETHER_DEPTHWISE = [((3, 5, 56, 56, 5, 3, 3), True), ((2, 6, 40, 64, 6, 3, 3), True), ((5, 32, 28, 28, 32, 3, 3), True),
                      ((3, 48, 14, 14, 48, 3, 3), True), ((9, 64, 7, 7, 64, 3, 3), True), ((1, 16, 16, 16, 16, 3, 3), True),
                      ((2, 3, 112, 112, 3, 3, 3), False), ((2, 5, 35, 35, 5, 3, 3), False)]


@pytest.mark.parametrize("shape,together,depthwise", [(*c, False) for c in TOGETHER_DENSE] + [(*c, True) for c in TOGETHER_DEPTHWISE])
def test_three_passes_in_one_launch(shape, together, depthwise):
    N, C, H, W, K, R, S = shape
    L = inputs.Layer("layer", N, C, H, W, K, R, S, stride=(1, 1), pad=(R // 2, S // 2), groups=C if depthwise else 1)
    st = LayerStep(L, keep_acc=True, requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(3)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    B.int8t_profile_start("dw_trio_kernel" if depthwise else "conv_trio_kernel")
    st.run(seed=5, overlap=0)
    torch.cuda.synchronize()
    assert bool(B.int8t_profile_stop()) == together
    outs = (st.y, st.dx, st.dw, st.y_acc, st.dx_acc, st.dw_acc)
    got = [t.clone() for t in outs]
    for t in outs[1:]:
        t.fill_(7)
    # the two backward passes without the forward one
    B.int8t_layer_step(st.desc, st._layer_buffers, B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT)
    torch.cuda.synchronize()
    for i in (1, 2, 4, 5):
        assert torch.equal(got[i], outs[i])
    for t in outs:
        t.fill_(7)
    st.fwd()
    st.bwd_data()
    st.bwd_weight()
    torch.cuda.synchronize()
    for a, b in zip(got, outs):
        assert torch.equal(a, b)


# Batches above 65535 images: the limit of the channels-last quantizer, not of planar codes.  Step and module against the calls
# one by one.
def test_depthwise_batch_above_65535():
    L = inputs.Layer("layer", 65537, 2, 5, 5, 2, 3, 3, stride=(1, 1), pad=(1, 1), groups=2)
    st = LayerStep(L)
    g = torch.Generator(device=DEV).manual_seed(2)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    got = [t.clone() for t in (st.y, st.dx, st.dw, st.clip, st.dev_final)]
    layer = Int8Conv2d(2, 2, 3, padding=1, groups=2, seed=4)          # (its first backward pass draws with seed 5)
    with torch.no_grad():
        layer.weight.copy_(st.w)
    x = st.x.clone().requires_grad_()
    y = layer(x)
    module = [y.detach()] + list(torch.autograd.grad(y, [x, layer.weight], st.dy)) + [layer.clip]
    for t in (st.y, st.dx, st.dw, st.clip, st.dev_final):
        t.fill_(7)
    st.quantize_xw()
    st.dsgc(5)
    st.quantize_dy(5)
    st.fwd()
    st.bwd_data()
    st.bwd_weight()
    torch.cuda.synchronize()
    for a, b in zip(got, (st.y, st.dx, st.dw, st.clip, st.dev_final)):
        assert torch.equal(a, b)
    for a, b in zip(module, got):
        assert torch.equal(a, b)


# Passes whose reduction is split when they run alone: the forward pass ahead of a shared launch of the backward ones, all three by
# themselves, or together in spite of it (5 to 88 stages of 128 bytes per tile); without the scratch of a split always together.
# Bit for bit the calls one by one.
@pytest.mark.parametrize("shape,reductions,together,reductions2,together2", [
    ((4, 1024, 8, 8, 96, 5, 5), 1, True, 0, True),              # forward 200 stages, backward-data 19
    ((1, 1024, 7, 7, 1024, 3, 3), 2, False, 1, False),          # 72 and 72
    ((1, 128, 10, 10, 440, 5, 5), 1, False, 1, False),          # 25 and 88
    ((2, 104, 8, 8, 200, 5, 5), 0, True, 1, False),             # 22 and 41
    ((1, 992, 10, 10, 832, 1, 7), 0, True, 0, True)])           # 55 and 46, backward-data not split
def test_split_reductions_and_the_shared_launch(shape, reductions, together, reductions2, together2):
    N, C, H, W, K, R, S = shape
    st = LayerStep(inputs.Layer("layer", N, C, H, W, K, R, S, stride=(1, 1), pad=(R // 2, S // 2)), keep_acc=True, requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(3)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    outs = (st.y, st.dx, st.dw, st.y_acc, st.dx_acc, st.dw_acc)
    for t in outs:
        t.fill_(7)
    st.fwd()
    st.bwd_data()
    st.bwd_weight()
    want = [t.clone() for t in outs]
    two = B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    no_scratch = B.LayerBuffers.from_buffer_copy(st._layer_buffers)
    no_scratch.ws_fwd = no_scratch.ws_bwd_data = None
    for buffers, parts, n_reduce, shared in ((st._layer_buffers, B.STEP_FWD | two, reductions, together), (st._layer_buffers, two, reductions2, together2),
                                             (no_scratch, B.STEP_FWD | two, 0, True), (no_scratch, two, 0, True)):
        for t in outs:
            t.fill_(7)
        B.int8t_profile_start(None)
        B.int8t_layer_step(st.desc, buffers, parts)
        torch.cuda.synchronize()
        launches = B.int8t_profile_stop()
        assert launches.get("igemm_reduce_kernel", (0,))[0] == n_reduce and ("conv_trio_kernel" in launches) == shared
        for i, t in enumerate(outs):
            assert torch.equal(t, want[i]) or (parts == two and i in (0, 3))


def small_step(depthwise, requantize_deviation=False):
    L = inputs.Layer("layer", 3, 32, 14, 14, 32, 3, 3, stride=(1, 1), pad=(1, 1), groups=32 if depthwise else 1)
    st = LayerStep(L, keep_acc=True, requantize_deviation=requantize_deviation)
    g = torch.Generator(device=DEV).manual_seed(6)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    torch.cuda.synchronize()
    return st


# A step dealt out over several calls, each with the pointers of its part alone: the tensors of the step in one call.
@pytest.mark.parametrize("requantize_deviation", [False, True])
@pytest.mark.parametrize("depthwise", [False, True])
def test_layer_step_parts_one_by_one(depthwise, requantize_deviation):
    st = small_step(depthwise, requantize_deviation)
    outs = ["xq", "wq", "dyq", "sx", "sw", "sdy", "clip", "dev_search", "dev_all", "y", "dx", "dw", "y_acc", "dx_acc", "dw_acc"]
    outs += ["dev_final"] if requantize_deviation else []
    want = [getattr(st, n).clone() for n in outs]
    for n in outs:
        getattr(st, n).fill_(7)
    parts = [(B.STEP_ABSMAX | B.STEP_PREPARE, "x w dy ws_quant ws_dy"), (B.STEP_SEARCH, "dy ratios clip dev_search dev_all ws_dy"),
             (B.STEP_QUANT_XW, "x w xq wq sx sw ws_quant"),
             (B.STEP_QUANT_G, "dy clip dyq sdy" + (" dev_final ws_dy" if requantize_deviation else "")),
             (B.STEP_FWD, "xq wq sx sw y y_acc"), (B.STEP_BWD_DATA, "dyq wq sdy sw dx dx_acc"),
             (B.STEP_BWD_WEIGHT, "xq dyq sx sdy dw dw_acc ws_bwd_weight")]
    tensors = {"ws_quant": st.ws_xw, "ws_bwd_weight": st.ws}
    for part, names in parts:
        buf = B.layer_buffers(n_cand=st.n_cand, **{n: tensors.get(n, getattr(st, n, None)) for n in names.split()})
        B.int8t_layer_step(st.desc, buf, part, 5)
    torch.cuda.synchronize()
    for n, w in zip(outs, want):
        assert torch.equal(getattr(st, n), w), n


# Results that overlap what another pass of the step writes: legal one after the other, so the passes do not share a launch.
@pytest.mark.parametrize("depthwise", [False, True])
@pytest.mark.parametrize("alias", ["dx over y", "dw over y", "scratch over y"])
def test_overlapping_results_run_one_by_one(depthwise, alias):
    st = small_step(depthwise)
    want = [st.dx.clone(), st.dw.clone()]
    st.y.fill_(7)
    buf = B.LayerBuffers.from_buffer_copy(st._layer_buffers)
    dx, dw = st.dx, st.dw
    if alias == "dx over y":
        buf.dx, dx = buf.y, st.y
    elif alias == "dw over y":
        buf.dw, dw = buf.y, st.y.view(-1)[:st.dw.numel()].view_as(st.dw)
    else:
        st.y_acc = torch.zeros(max(st.y_acc.numel(), st.ws.numel() // 4 + 4), dtype=torch.int32, device=DEV)
        buf.y_acc = buf.ws_bwd_weight = st.y_acc.data_ptr()
    for t in (st.dx, st.dw):
        t.fill_(7)
    B.int8t_profile_start("dw_trio_kernel" if depthwise else "conv_trio_kernel")
    B.int8t_layer_step(st.desc, buf, B.STEP_FWD | B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT)
    torch.cuda.synchronize()
    assert not B.int8t_profile_stop()
    assert torch.equal(dx, want[0]) and torch.equal(dw, want[1])


# Depthwise layers that form their codes in the launch of the passes, whole and in halves (a and W with the forward pass, g_z with
# the backward ones), against the calls one by one, bit for bit: one, two and four chunks of a plane per thread, channel groups with
# rows of whole dwords and others, elements that are no number.  What may not overlap in one launch does in the last form:
# the input gradient over the output gradient, which is legal one after the other.
@pytest.mark.parametrize("form", ["whole", "halves", "dx over dy"])
@pytest.mark.parametrize("shape", [(3, 5, 28, 28), (2, 3, 32, 32), (5, 2, 36, 32), (3, 4, 56, 56), (9, 2, 64, 64), (9, 64, 7, 7), (5, 32, 14, 14),
                                   (3, 16, 5, 7), (4, 32, 6, 4), (7, 8, 10, 6), (70, 16, 8, 8)])
def test_depthwise_codes_and_passes_in_one_launch(shape, form):
    N, C, H, W = shape
    L = inputs.Layer("layer", N, C, H, W, C, 3, 3, stride=(1, 1), pad=(1, 1), groups=C)
    st = LayerStep(L, keep_acc=True, requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(8)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.x.view(-1)[5] = st.dy.view(-1)[7] = float("nan")
    dy = st.dy.clone()
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    front = B.STEP_ABSMAX | B.STEP_PREPARE | B.STEP_SEARCH
    fwd, bwd = B.STEP_QUANT_XW | B.STEP_FWD, B.STEP_QUANT_G | B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    outs = ["xq", "wq", "dyq", "sx", "sw", "sdy", "clip", "y", "dx", "dw", "y_acc", "dx_acc", "dw_acc"]

    def result(calls, buf):
        for n in outs:
            getattr(st, n).fill_(7)
        st.dy.copy_(dy)
        for parts in calls:
            B.int8t_layer_step(st.desc, buf, parts, 5)
        torch.cuda.synchronize()
        return [getattr(st, n).clone() for n in outs]

    want = result([front] + [1 << i for i in range(3, 8)], st._layer_buffers)
    buf = B.LayerBuffers.from_buffer_copy(st._layer_buffers)
    if form == "dx over dy":
        buf.dx = buf.dy
    B.int8t_profile_start(None)
    got = result([front | fwd, bwd] if form == "halves" else [front | fwd | bwd], buf)
    launches = B.int8t_profile_stop()
    quantized = any(k.startswith("quantize") for k in launches)        # (a launch of its own for codes)
    if form == "dx over dy":
        got[outs.index("dx")] = st.dy.clone()
        assert quantized
    else:
        assert launches["dw_trio_kernel"][0] == (2 if form == "halves" else 1) and not quantized
        assert all(B.int8t_layer_step_form(st.desc, parts) == B.FORM_DW_CODES for parts in (front | fwd | bwd, fwd, bwd))
    for n, a, b in zip(outs, got, want):
        assert torch.equal(a, b), n


# Codes of 1 x 1 images whose channels need padding: rows of whole 16 bytes and others, one to four and many quads per thread, a
# single granule; both roundings, with and without a clip value and Eq.6, alone and in a batch.
@pytest.mark.parametrize("N,C", [(1, 1), (3, 7), (5, 18), (256, 1000), (17, 1001), (2, 4092), (300, 1785), (2100, 996)])
def test_codes_of_rows(N, C):
    r = np.random.RandomState(C)
    x = (r.standard_t(3, size=(N, C, 1, 1)) * 1e-3).astype(np.float32)
    x.reshape(-1)[0] = np.nan if C > 1 else 1.0
    xd, q, s = dev(x), torch.full((N * ((C + 15) // 16 * 16),), 7, dtype=torch.int8, device=DEV), torch.zeros(1, device=DEV)
    ws = torch.empty(B.int8t_quantize_workspace_bytes((N, C, 1, 1), B.ACT), dtype=torch.uint8, device=DEV)
    d = torch.zeros(1, dtype=torch.float64, device=DEV)
    finite = np.nan_to_num(x)
    for mode, om in ((RTN, oracle.ROUND_NEAREST_EVEN), (STO, oracle.ROUND_STOCHASTIC)):
        for clip in (None, np.float32(4e-3)):
            want, sc = oracle.quantize(finite, c=clip, mode=om, seed=11)
            cd = None if clip is None else dev(np.array([clip], np.float32))
            for batch in (False, True):
                q.fill_(7)
                if batch:
                    B.int8t_quantize_batch([(xd, (N, C, 1, 1), B.ACT, cd, q, s, mode, 11)], ws=torch.empty(1 << 14, dtype=torch.uint8, device=DEV))
                else:
                    B.int8t_quantize(xd, (N, C, 1, 1), B.ACT, cd, mode, 11, q, s, None if C > 1 else d, ws)
                torch.cuda.synchronize()
                got, pad = B.int8t_unpack_codes(q.cpu().numpy(), (N, C, 1, 1), B.ACT)
                assert np.array_equal(got, want) and pad == 0 and s.item() == sc
            if C > 1:
                xd0 = dev(finite)
                B.int8t_quantize(xd0, (N, C, 1, 1), B.ACT, cd, mode, 11, q, s, d, ws)
                torch.cuda.synchronize()
                ref = want.astype(np.float64).reshape(-1)
                g64 = finite.astype(np.float64).reshape(-1)
                dw = 1.0 - (g64 @ ref) / (np.sqrt(g64 @ g64) * np.sqrt(ref @ ref)) if ref.any() else 1.0
                assert abs(d.item() - dw) < 1e-9


# Passes of at most 64 rows on 64 x 128 tiles in the shared launch: all of them, the forward or the backward-data pass beside a wider
# one, the two backward passes alone, rows that end inside a fragment, planes of whole 16-byte groups and others, the last column tile
# ragged; and layers just below the rule's bounds, which stay on 128-row tiles.  The calls one by one are the other kernels.
@pytest.mark.parametrize("shape,three,two", [
    ((20, 40, 30, 30, 24, 3, 3), B.FORM_64X128, B.FORM_128X64), ((33, 40, 30, 30, 24, 3, 3), B.FORM_64X128, B.FORM_64X128),
    ((25, 33, 27, 27, 64, 3, 3), B.FORM_64X128, B.FORM_128X64), ((41, 33, 27, 27, 64, 3, 3), B.FORM_64X128, B.FORM_64X128),
    ((32, 5, 30, 31, 64, 5, 5), B.FORM_64X128, B.FORM_64X128), ((45, 64, 23, 29, 7, 1, 7), B.FORM_64X128, B.FORM_64X128),
    ((32, 200, 28, 28, 20, 3, 3), B.FORM_64X128_AND_128X128, B.FORM_128X64), ((42, 200, 28, 28, 20, 3, 3), B.FORM_64X128_AND_128X128, B.FORM_128X128),
    ((32, 20, 28, 28, 200, 3, 3), B.FORM_64X128_AND_128X128, B.FORM_128X64), ((33, 48, 27, 27, 130, 3, 1), B.FORM_64X128_AND_128X128, B.FORM_128X64),
    ((17, 40, 30, 30, 24, 3, 3), B.FORM_128X64, B.FORM_128X64), ((28, 200, 28, 28, 20, 3, 3), B.FORM_128X64, B.FORM_128X64),
    ((64, 40, 31, 31, 130, 1, 1), B.FORM_64X128_AND_128X128, B.FORM_64X128)])
@pytest.mark.parametrize("passes", [B.STEP_FWD | B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT, B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT])
def test_narrow_passes_in_one_launch(shape, three, two, passes):
    N, C, H, W, K, R, S = shape
    L = inputs.Layer("layer", N, C, H, W, K, R, S, stride=(1, 1), pad=(R // 2, S // 2), groups=1)
    st = LayerStep(L, keep_acc=True, requantize_deviation=False)
    assert B.int8t_layer_step_form(st.desc, passes) == (three if passes & B.STEP_FWD else two)
    g = torch.Generator(device=DEV).manual_seed(13)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    outs = [st.dx, st.dw, st.dx_acc, st.dw_acc] + ([st.y, st.y_acc] if passes & B.STEP_FWD else [])
    for t in outs:
        t.fill_(7)
    B.int8t_profile_start("conv_trio_kernel")
    B.int8t_layer_step(st.desc, st._layer_buffers, passes)
    torch.cuda.synchronize()
    assert B.int8t_profile_stop()
    got = [t.clone() for t in outs]
    for t in outs:
        t.fill_(7)
    st.fwd()
    st.bwd_data()
    st.bwd_weight()
    torch.cuda.synchronize()
    for a, b in zip(got, outs):
        assert torch.equal(a, b)


# Backward-weight of 1x1 filters with few channels on one side, either side of the bounds between its two kernels: 256 input
# channels, a batch of 32 on square and other images and under a stride, less than a hundred channels in all on large images.
@pytest.mark.parametrize("shape,lines", [
    ((2, 256, 5, 7, 8, 1, 1, 1, (0, 0)), True), ((2, 240, 5, 7, 8, 1, 1, 1, (0, 0)), False), ((31, 40, 6, 6, 20, 1, 1, 1, (0, 0)), False),
    ((32, 40, 6, 6, 20, 1, 1, 1, (0, 0)), True), ((9, 24, 28, 7, 130, 1, 1, 1, (0, 0)), True), ((33, 5, 9, 9, 250, 1, 1, 2, (0, 0)), True),
    ((32, 48, 32, 32, 33, 1, 1, 1, (0, 0)), False), ((32, 64, 32, 32, 33, 1, 1, 1, (0, 0)), True), ((64, 100, 1, 1, 70, 1, 1, 1, (0, 0)), True)])
def test_backward_weight_narrow_1x1(shape, lines):
    desc, od, (xq, wq, dyq) = random_layer(shape, 3)
    B.int8t_profile_start(None)
    conv_pass_elementwise(B.OP_CONV_BWD_WEIGHT, desc, od, xq, wq, dyq, True)
    launches = B.int8t_profile_stop()
    assert ("wgrad_lines_kernel" in launches, "wgrad_kernel" in launches) == (lines, not lines)


# Layers that run in space-to-depth form: backward-weight on what the forward pass made of the codes, in one call, in calls of their
# own and on two streams, against the pass that makes it itself; not where something may be written over it in between: one
# scratch for both passes, whose partial results then lie on the codes, and the schedule whose backward pass does not wait for the forward one.
@pytest.mark.parametrize("shape", [(3, 3, 33, 30, 24, 7, 7, 3), (2, 4, 16, 16, 40, 3, 3, 1), (5, 1, 11, 17, 130, 5, 5, 2)])
def test_backward_weight_on_the_forward_passes_codes(shape):
    N, C, H, W, K, R, S, pad = shape
    L = inputs.Layer("layer", N, C, H, W, K, R, S, stride=(2, 2), pad=(pad, pad), groups=1)
    st = LayerStep(L, keep_acc=True, requantize_deviation=False, input_grad=False)
    g = torch.Generator(device=DEV).manual_seed(14)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    st.dw.fill_(7)
    st.bwd_weight()
    torch.cuda.synchronize()
    want = [st.dw.clone(), st.dw_acc.clone()]

    def check(run, repacks):
        st.dw.fill_(7)
        st.dw_acc.fill_(7)
        B.int8t_profile_start("s2d_repack_kernel")
        run()
        torch.cuda.synchronize()
        assert B.int8t_profile_stop()["s2d_repack_kernel"][0] == repacks
        assert torch.equal(st.dw, want[0]) and torch.equal(st.dw_acc, want[1])

    def apart():
        st.fwd()
        B.int8t_conv_bwd_weight_fwd(st.desc, st.xq, st.sx, st.dyq, st.sdy, st.dw, st.dw_acc, st.ws, st.ws_fwd)

    check(lambda: st.run(seed=5, overlap=0), 1)
    check(lambda: st.run(seed=5, overlap=1), 1)
    check(lambda: st.run(seed=5, overlap=4), 2)
    check(apart, 1)
    check(lambda: (st.fwd(), B.int8t_conv_bwd_weight_fwd(st.desc, st.xq, st.sx, st.dyq, st.sdy, st.dw, st.dw_acc, st.ws, None)), 2)
    both = B.STEP_FWD | B.STEP_BWD_WEIGHT
    buf = B.LayerBuffers.from_buffer_copy(st._layer_buffers)
    shared = torch.empty(max(st.ws.numel(), st.ws_fwd.numel()), dtype=torch.uint8, device=DEV)
    buf.ws_fwd = buf.ws_bwd_weight = shared.data_ptr()
    check(lambda: B.int8t_layer_step(st.desc, buf, both), 2)
    B.int8t_conv_fwd(st.desc, st.xq, st.sx, st.wq, st.sw, st.y, None, shared)
    check(lambda: B.int8t_conv_bwd_weight_fwd(st.desc, st.xq, st.sx, st.dyq, st.sdy, st.dw, st.dw_acc, shared, shared), 1)


# Backward-weight with fewer shares beside other passes than by itself, one (no reduction) and several, for two passes and for three, stride 1 and 2:
# bit for bit the calls one by one, whatever the scratch held; the same layer again, another one in between.
@pytest.mark.parametrize("shape,reductions", [
    ((64, 512, 7, 7, 512, 3, 3, 1, 1), (0, 1)), ((6, 215, 15, 15, 197, 3, 3, 1, 1), (0, 0)), ((10, 677, 19, 19, 365, 3, 3, 2, 1), (0, 0)),
    ((32, 48, 35, 35, 64, 5, 5, 1, 2), (1, 1)), ((128, 1024, 14, 14, 256, 1, 1, 1, 0), (1, 1)), ((2, 16, 16, 16, 32, 3, 3, 1, 1), (0, 0))])
def test_fewer_shares_beside_other_passes(shape, reductions):
    N, C, H, W, K, R, S, stride, pad = shape
    L = inputs.Layer("layer", N, C, H, W, K, R, S, stride=(stride, stride), pad=(pad, pad), groups=1)
    st = LayerStep(L, keep_acc=True, requantize_deviation=False)
    small = LayerStep(inputs.Layer("layer", 2, 32, 9, 9, 40, 3, 3, stride=(1, 1), pad=(1, 1), groups=1), requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(16)
    for s in (st, small):
        for t in (s.x, s.w, s.dy):
            t.normal_(generator=g)
        s.clip.fill_(1.5)
        B.int8t_layer_step(s.desc, s._layer_buffers, B.STEP_ABSMAX | B.STEP_QUANT_XW | B.STEP_QUANT_G, 3)
    outs = [st.y, st.y_acc, st.dx, st.dx_acc, st.dw, st.dw_acc]
    for parts in (B.STEP_FWD, B.STEP_BWD_DATA, B.STEP_BWD_WEIGHT):
        B.int8t_layer_step(st.desc, st._layer_buffers, parts)
    want = [t.clone() for t in outs]
    two = B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    for parts, count in ((two, reductions[0]), (two | B.STEP_FWD, reductions[1]), (two, reductions[0])):
        for t in outs[2:] + [st.ws]:
            t.fill_(7)
        B.int8t_profile_start(None)
        B.int8t_layer_step(st.desc, st._layer_buffers, parts)
        torch.cuda.synchronize()
        launches = B.int8t_profile_stop()
        assert launches.pop("conv_trio_kernel")[0] == 1 and launches.pop("wgrad_reduce_kernel", (0,))[0] == count and not launches
        for a, b in zip(outs, want):
            assert torch.equal(a, b)
        B.int8t_layer_step(small.desc, small._layer_buffers, parts)


# Bands whose window takes six staged granules a thread and seven, nine, twelve, a row in one part and in more, one and two tiles of rows
# and of pixels, rows above and below the image, a last band that ends beyond it.
@pytest.mark.parametrize("op,shape", [
    (B.OP_CONV_FWD, (2, 16, 9, 130, 33, 6, 1, 1, (2, 0))), (B.OP_CONV_FWD, (2, 16, 9, 130, 24, 7, 1, 1, (3, 0))), (B.OP_CONV_FWD, (3, 40, 5, 120, 40, 3, 3, 1, (1, 1))),
    (B.OP_CONV_FWD, (2, 48, 6, 250, 20, 3, 3, 1, (1, 1))), (B.OP_CONV_FWD, (2, 48, 7, 128, 64, 6, 1, 1, (5, 0))), (B.OP_CONV_FWD, (3, 5, 11, 21, 7, 5, 3, 1, (4, 2))),
    (B.OP_CONV_BWD_DATA, (2, 33, 9, 130, 16, 6, 1, 1, (2, 0))), (B.OP_CONV_BWD_DATA, (2, 24, 9, 130, 16, 7, 1, 1, (3, 0))),
    (B.OP_CONV_BWD_DATA, (3, 64, 5, 120, 40, 3, 3, 1, (1, 1))), (B.OP_CONV_BWD_DATA, (2, 20, 6, 250, 48, 3, 3, 1, (1, 1)))])
@pytest.mark.parametrize("with_acc", [False, True])
def test_bands_of_few_and_many_staged_granules(op, shape, with_acc):
    desc, od, (xq, wq, dyq) = random_layer(shape, shape[3])
    B.int8t_conv_select_variant(op, desc, B.VARIANT_BAND)
    try:
        B.int8t_profile_start("band_kernel")
        conv_pass_elementwise(op, desc, od, xq, wq, dyq, with_acc)
        assert B.int8t_profile_stop()["band_kernel"][0] == 1
    finally:
        B.int8t_conv_select_variant(op, desc, B.VARIANT_AUTO)


# A stem's codes in both forms from one pass over the image: every count of channels, odd and even rows and columns, a last block of one
# pixel, with g_z's codes in the same launch and without, against the codes and the forward pass in calls of their own, bit for bit; and
# with the scratch of the forward pass over the partial maxima, which the codes' pass still reads.
@pytest.mark.parametrize("shape", [(3, 1, 1, 1, 8, 1, 1, 0), (2, 2, 16, 32, 24, 3, 3, 1), (1, 3, 33, 30, 8, 7, 7, 3), (257, 4, 2, 1, 130, 2, 3, 1),
                                   (5, 3, 30, 33, 16, 5, 5, 2), (4, 1, 15, 17, 40, 1, 1, 0)])
def test_stem_codes_in_both_forms(shape):
    N, C, H, W, K, R, S, pad = shape
    L = inputs.Layer("layer", N, C, H, W, K, R, S, stride=(2, 2), pad=(pad, pad), groups=1)
    st = LayerStep(L, keep_acc=True, requantize_deviation=False, input_grad=False)
    g = torch.Generator(device=DEV).manual_seed(15)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    outs = [st.xq, st.sx, st.wq, st.sw, st.y, st.y_acc, st.dyq, st.sdy]
    scratch = N * ((H + 1) // 2) * ((W + 1) // 2) * 16

    def result(*calls, buf=st._layer_buffers):
        for t in outs + [st.ws_fwd]:
            t.fill_(7)
        st.clip.fill_(1.5)
        for parts in calls:
            B.int8t_layer_step(st.desc, buf, parts, 3)
        torch.cuda.synchronize()
        return [t.clone() for t in outs + [st.ws_fwd[:scratch]]]

    codes = B.STEP_ABSMAX | B.STEP_QUANT_XW
    want = result(codes, B.STEP_QUANT_G, B.STEP_FWD)
    for a, b in zip(result(codes | B.STEP_QUANT_G | B.STEP_FWD), want):
        assert torch.equal(a, b)
    for a, b in zip(result(codes | B.STEP_FWD, B.STEP_QUANT_G), want):
        assert torch.equal(a, b)
    buf = B.LayerBuffers.from_buffer_copy(st._layer_buffers)
    shared = torch.empty(max(buf.ws_fwd_bytes, buf.ws_quant_bytes), dtype=torch.uint8, device=DEV)
    buf.ws_quant = buf.ws_fwd = shared.data_ptr()
    for a, b in list(zip(result(codes | B.STEP_QUANT_G | B.STEP_FWD, buf=buf), want))[:-1]:
        assert torch.equal(a, b)


# The forward pass without codes: one and two row tiles of filters, planes of whole 16-byte groups and others, ragged pixel tiles,
# more tiles than resident blocks, channels that end inside 64, elements that are no number; layers just outside the rule, and
# results over the input, which the calls one after the other allow.  Against the step's forward pass, bit for bit.
@pytest.mark.parametrize("shape,fused", [((3, 144, 20, 20, 24), True), ((2, 64, 9, 9, 32), True), ((5, 3, 16, 14, 33), True), ((1, 200, 8, 8, 40), True),
                                         ((31, 20, 57, 57, 7), True), ((40, 70, 48, 48, 40), True), ((2, 256, 10, 10, 32), True), ((260, 256, 16, 16, 64), True),
                                         ((2, 64, 7, 9, 24), False), ((2, 64, 10, 10, 65), False), ((2, 257, 10, 10, 24), False),
                                         ((2, 256, 10, 10, 33), False), ((2, 65, 9, 9, 8), False), ((2, 16, 9, 9, 33), False), ((42, 16, 57, 57, 8), False)])
def test_forward_without_codes(shape, fused):
    N, C, H, W, K = shape
    L = inputs.Layer("layer", N, C, H, W, K, 1, 1, stride=(1, 1), pad=(0, 0), groups=1)
    st = LayerStep(L, requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(15)
    for t in (st.x, st.w):
        t.normal_(generator=g)
    st.x.view(-1)[11] = float("nan")
    B.int8t_layer_step(st.desc, st._layer_buffers, B.STEP_ABSMAX | B.STEP_QUANT_XW | B.STEP_FWD)
    torch.cuda.synchronize()
    want = st.y.clone()
    st.y.fill_(7)
    B.int8t_profile_start("infer_1x1_kernel")
    B.int8t_layer_infer(st.desc, st._layer_buffers)
    torch.cuda.synchronize()
    assert bool(B.int8t_profile_stop()) == fused and torch.equal(st.y, want)
    if K <= C:
        buf = B.LayerBuffers.from_buffer_copy(st._layer_buffers)
        buf.y = buf.x
        B.int8t_layer_infer(st.desc, buf)
        torch.cuda.synchronize()
        assert torch.equal(st.x.view(-1)[:want.numel()], want.view(-1))


# The passes of a strided layer in one launch: 3x3 filters with the four pixel classes of a cell in a block, a class per tile, and plain
# (short runs of pixels); 1x1 filters in cells of even images, odd images, other strides; paddings, ragged rows and columns, results on
# planes of no whole 16-byte groups.  Against the calls one by one, bit for bit.
@pytest.mark.parametrize("shape,form", [
    ((3, 130, 28, 28, 40, 3, 2, 2, 1), B.FORM_STRIDED_CELLS), ((2, 150, 30, 32, 200, 3, 2, 2, 0), B.FORM_STRIDED_CELLS),
    ((5, 40, 24, 25, 70, 3, 2, 2, 1), B.FORM_STRIDED_CLASSES), ((2, 257, 33, 27, 30, 3, 2, 2, 2), B.FORM_STRIDED_CLASSES),
    ((9, 16, 11, 11, 33, 3, 2, 2, 1), B.FORM_STRIDED), ((34, 70, 14, 14, 50, 1, 2, 2, 0), B.FORM_STRIDED_CELL),
    ((3, 300, 15, 13, 140, 1, 2, 2, 0), B.FORM_STRIDED), ((3, 300, 14, 10, 20, 1, 3, 1, 0), B.FORM_STRIDED), ((2, 260, 9, 12, 33, 1, 1, 2, 0), B.FORM_STRIDED)])
@pytest.mark.parametrize("passes", [B.STEP_FWD | B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT, B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT])
def test_strided_passes_in_one_launch(shape, form, passes):
    N, C, H, W, K, R, sh, sw, pad = shape
    L = inputs.Layer("layer", N, C, H, W, K, R, R, stride=(sh, sw), pad=(pad, pad), groups=1)
    st = LayerStep(L, keep_acc=True, requantize_deviation=False)
    assert B.int8t_layer_step_form(st.desc, passes) == form
    g = torch.Generator(device=DEV).manual_seed(16)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    outs = [st.dx, st.dw, st.dx_acc, st.dw_acc] + ([st.y, st.y_acc] if passes & B.STEP_FWD else [])
    for t in outs:
        t.fill_(7)
    B.int8t_profile_start("conv_trio_kernel")
    B.int8t_layer_step(st.desc, st._layer_buffers, passes)
    torch.cuda.synchronize()
    assert B.int8t_profile_stop()
    got = [t.clone() for t in outs]
    for t in outs:
        t.fill_(7)
    st.fwd()
    st.bwd_data()
    st.bwd_weight()
    torch.cuda.synchronize()
    for a, b in zip(got, outs):
        assert torch.equal(a, b)


# Codes of planes of no whole 16-byte groups (a plane's last quad of one, two and three pixels, planes of two and three pixels, the
# tensor's end), and tiles dealt image by image or eight images side by side (with and without images beyond the batch, one and
# several channel groups, whole groups too; at most 16 channels, a pixel per thread); both roundings, with Eq.6 and in a batch with another tensor behind it.
@pytest.mark.parametrize("N,C,H,W", [(1, 17, 1, 2), (3, 20, 3, 1), (2, 100, 7, 7), (8, 33, 9, 9), (8, 65, 17, 17), (16, 20, 17, 18), (15, 18, 17, 19),
                                     (31, 24, 17, 17), (8, 130, 47, 45), (8, 40, 47, 45), (8, 70, 18, 18), (1, 18, 5, 13),
                                     (8, 3, 17, 17), (16, 16, 33, 31), (31, 9, 17, 17), (15, 3, 19, 17)])
def test_codes_of_ragged_planes(N, C, H, W):
    r = np.random.RandomState(C + W)
    x = (r.standard_t(3, size=(N, C, H, W)) * 1e-3).astype(np.float32)
    x2 = r.standard_normal((3, 24, 5, 5)).astype(np.float32)
    xd, x2d = dev(x), dev(x2)
    pad16 = lambda c: (c + 15) // 16 * 16
    q, s = torch.empty(N * H * W * pad16(C), dtype=torch.int8, device=DEV), torch.zeros(1, device=DEV)
    q2, s2 = torch.empty(3 * 25 * 32, dtype=torch.int8, device=DEV), torch.zeros(1, device=DEV)
    ws = torch.empty(B.int8t_quantize_workspace_bytes(x.shape, B.ACT), dtype=torch.uint8, device=DEV)
    d = torch.zeros(1, dtype=torch.float64, device=DEV)
    want2, _ = oracle.quantize(x2, c=None, mode=oracle.ROUND_NEAREST_EVEN, seed=0)
    for mode, om in ((RTN, oracle.ROUND_NEAREST_EVEN), (STO, oracle.ROUND_STOCHASTIC)):
        want, sc = oracle.quantize(x, c=None, mode=om, seed=11)
        ref, g64 = want.astype(np.float64).reshape(-1), x.astype(np.float64).reshape(-1)
        for form in ("plain", "eq6", "batch"):
            q.fill_(7)
            q2.fill_(7)
            if form == "batch":
                B.int8t_quantize_batch([(xd, x.shape, B.ACT, None, q, s, mode, 11), (x2d, x2.shape, B.ACT, None, q2, s2)],
                                       ws=torch.empty(1 << 14, dtype=torch.uint8, device=DEV))
            else:
                B.int8t_quantize(xd, x.shape, B.ACT, None, mode, 11, q, s, d if form == "eq6" else None, ws)
            torch.cuda.synchronize()
            got, pad = B.int8t_unpack_codes(q.cpu().numpy(), x.shape, B.ACT)
            assert np.array_equal(got, want) and pad == 0 and s.item() == sc, form
            if form == "batch":
                got2, pad2 = B.int8t_unpack_codes(q2.cpu().numpy(), x2.shape, B.ACT)
                assert np.array_equal(got2, want2) and pad2 == 0
            if form == "eq6":
                # sums of up to 1e6 fp64 products in another order: relative error below 1e6 * 2^-53 = 1.1e-10
                assert abs(d.item() - (1.0 - (g64 @ ref) / (np.sqrt(g64 @ g64) * np.sqrt(ref @ ref)))) < 1e-9


# Backward-weight's partial tiles: one share, whose tile is the result (no reduction launched), and the flat reduction with 64, 32, 16
# and 8 quads to a block, more shares than a thread has in flight, a last block that is not full, the space-to-depth stem.
@pytest.mark.parametrize("shape,one_share", [
    ((2, 16, 16, 16, 32, 3, 3, 1, (1, 1)), True), ((1, 300, 1, 1, 65, 1, 1, 1, (0, 0)), True), ((2, 70, 4, 9, 130, 7, 1, 1, (3, 0)), True),
    ((3, 33, 9, 9, 40, 3, 3, 2, (1, 1)), True), ((2, 130, 8, 8, 129, 1, 1, 2, (0, 0)), True), ((1, 40, 6, 7, 33, 5, 5, 1, (2, 2)), True),
    ((64, 500, 7, 7, 300, 1, 1, 1, (0, 0)), False), ((32, 250, 14, 14, 280, 1, 1, 1, (0, 0)), False), ((64, 64, 14, 14, 63, 3, 3, 1, (1, 1)), False),
    ((32, 33, 35, 35, 17, 3, 3, 1, (1, 1)), False), ((256, 60, 40, 40, 50, 1, 1, 1, (0, 0)), False), ((20, 3, 32, 32, 17, 7, 7, 2, (3, 3)), False)])
@pytest.mark.parametrize("with_acc", [False, True])
def test_backward_weight_shares(shape, one_share, with_acc):
    desc, od, (xq, wq, dyq) = random_layer(shape, 11)
    B.int8t_profile_start("wgrad_reduce_kernel")
    conv_pass_elementwise(B.OP_CONV_BWD_WEIGHT, desc, od, xq, wq, dyq, with_acc)
    assert bool(B.int8t_profile_stop()) != one_share


# The weight gradient over the codes it comes from: legal, the reduction runs after they have been read.
def test_backward_weight_over_its_codes():
    desc, od, (xq, wq, dyq) = random_layer((2, 70, 4, 9, 130, 7, 1, 1, (3, 0)), 12)
    want, _ = oracle.wrap32(oracle.conv_bwd_weight(od, xq, dyq))
    ws = torch.empty(B.int8t_workspace_bytes(B.OP_CONV_BWD_WEIGHT, desc), dtype=torch.uint8, device=DEV)
    one = torch.ones(1, device=DEV)
    for over_x in (True, False):
        codes = [dev(pack_act(xq)), dev(pack_act(dyq))]
        buf = torch.zeros(max(4 * want.size, codes[0].numel(), codes[1].numel()), dtype=torch.int8, device=DEV)
        i = 0 if over_x else 1
        buf[:codes[i].numel()].copy_(codes[i].view(-1))
        codes[i] = buf[:codes[i].numel()]
        dw = buf[:4 * want.size].view(torch.float32)
        B.int8t_profile_start("wgrad_reduce_kernel")
        B.int8t_conv_bwd_weight(desc, codes[0], one, codes[1], one, dw, None, ws)
        torch.cuda.synchronize()
        assert B.int8t_profile_stop() and np.array_equal(dw.cpu().numpy().reshape(want.shape), want.astype(np.float32))


# The reduction in blocks of 9, 7 and 3 taps x 64 and 16 channels, with few and with many shares, and the flat one; filters and channels
# that fill neither their last four nor their last sixteen.
@pytest.mark.parametrize("shape,variant", [
    ((8, 250, 7, 7, 515, 3, 3, 1, (1, 1)), B.VARIANT_WGRAD_MORE), ((8, 320, 7, 10, 410, 1, 7, 1, (0, 3)), 0), ((16, 254, 7, 7, 382, 1, 3, 1, (0, 1)), 0),
    ((16, 190, 7, 7, 190, 3, 3, 1, (1, 1)), 0), ((24, 100, 10, 10, 110, 1, 7, 1, (0, 3)), 0), ((64, 100, 6, 6, 110, 1, 3, 1, (0, 1)), 0),
    ((16, 40, 12, 14, 61, 5, 5, 1, (2, 2)), 0), ((64, 120, 14, 14, 519, 3, 1, 1, (1, 0)), 0), ((60, 30, 9, 9, 66, 3, 3, 1, (1, 1)), 0)])
def test_reductions_of_few_and_many_shares(shape, variant):
    desc, od, (xq, wq, dyq) = random_layer(shape, 29)
    B.int8t_conv_select_variant(B.OP_CONV_BWD_WEIGHT, desc, variant)
    try:
        B.int8t_profile_start("wgrad_reduce_kernel")
        conv_pass_elementwise(B.OP_CONV_BWD_WEIGHT, desc, od, xq, wq, dyq, True)
        assert B.int8t_profile_stop()
    finally:
        B.int8t_conv_select_variant(B.OP_CONV_BWD_WEIGHT, desc, B.VARIANT_AUTO)


# One share of a large filter: its tile is the result where the weights are few, or 5x5 and many; reduced otherwise.  Both alone and
# beside backward-data, whose launch may take fewer shares.
@pytest.mark.parametrize("shape,one_share", [
    ((1, 33, 8, 8, 33, 5, 5, 1, (2, 2)), True), ((1, 64, 8, 8, 64, 5, 5, 1, (2, 2)), False), ((1, 245, 6, 6, 245, 5, 5, 1, (2, 2)), True),
    ((2, 64, 8, 9, 61, 7, 7, 1, (3, 3)), False), ((1, 16, 9, 8, 48, 7, 7, 1, (3, 3)), True), ((1, 70, 8, 8, 130, 3, 3, 1, (1, 1)), True),
    ((1, 150, 7, 7, 130, 7, 7, 1, (3, 3)), False)])
def test_single_share_of_large_filters(shape, one_share):
    desc, od, (xq, wq, dyq) = random_layer(shape, 19)
    B.int8t_profile_start("wgrad_reduce_kernel")
    conv_pass_elementwise(B.OP_CONV_BWD_WEIGHT, desc, od, xq, wq, dyq, True)
    assert bool(B.int8t_profile_stop()) != one_share
    N, C, H, W, K, R, S, stride, pad = shape
    st = LayerStep(inputs.Layer("layer", N, C, H, W, K, R, S, stride=(stride, stride), pad=pad), keep_acc=True, requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(23)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.clip.fill_(1.5)
    B.int8t_layer_step(st.desc, st._layer_buffers, B.STEP_ABSMAX | B.STEP_QUANT_XW | B.STEP_QUANT_G, 3)
    st.bwd_data()
    st.bwd_weight()
    outs = [st.dx, st.dx_acc, st.dw, st.dw_acc]
    want = [t.clone() for t in outs]
    for t in outs:
        t.fill_(7)
    B.int8t_layer_step(st.desc, st._layer_buffers, B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT)
    torch.cuda.synchronize()
    for a, b in zip(outs, want):
        assert torch.equal(a, b)


# Passes with the filter bank on chip in one launch with backward-weight: every body (weights in registers, in LDS with one and two
# row tiles) with every form of backward-weight (image granules; 1, 3, 5, 7 taps along a line), all three passes or the
# forward pass ahead, bands that end below the image, planes of odd sizes.  Bit for bit the calls one by one.
@pytest.mark.parametrize("shape,ahead", [
    ((65, 24, 57, 55, 64, 1, 1), True), ((65, 64, 56, 56, 64, 1, 1), False), ((40, 16, 50, 100, 128, 1, 1), True), ((65, 16, 56, 56, 128, 1, 1), True),
    ((58, 32, 59, 60, 32, 3, 3), False), ((65, 64, 56, 56, 64, 3, 3), False), ((65, 24, 56, 56, 24, 1, 1), False), ((65, 16, 56, 56, 256, 1, 1), True),
    ((65, 16, 56, 57, 16, 3, 3), False), ((65, 8, 56, 56, 16, 5, 5), False), ((65, 24, 56, 56, 16, 1, 7), False), ((65, 40, 56, 56, 24, 1, 1), True),
    ((65, 56, 56, 56, 256, 1, 1), True), ((65, 40, 56, 56, 16, 3, 3), True), ((65, 48, 56, 56, 16, 1, 5), True), ((65, 56, 55, 56, 40, 7, 1), False)])
def test_bands_and_backward_weight_in_one_launch(shape, ahead):
    N, C, H, W, K, R, S = shape
    st = LayerStep(inputs.Layer("layer", N, C, H, W, K, R, S, stride=(1, 1), pad=(R // 2, S // 2)), keep_acc=True, requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(3)
    for t in (st.x, st.w, st.dy):
        t.normal_(generator=g)
    st.ratios.copy_(dev(inputs.default_ratios(32)))
    st.run(seed=5, overlap=0)
    outs = (st.y, st.dx, st.dw, st.y_acc, st.dx_acc, st.dw_acc)
    for t in outs:
        t.fill_(7)
    st.fwd()
    st.bwd_data()
    st.bwd_weight()
    want = [t.clone() for t in outs]
    two = B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    for parts in (two, B.STEP_FWD | two):
        assert B.int8t_layer_step_form(st.desc, parts) == B.FORM_BANDS
        for t in outs:
            t.fill_(7)
        B.int8t_profile_start(None)
        B.int8t_layer_step(st.desc, st._layer_buffers, parts)
        torch.cuda.synchronize()
        launches = B.int8t_profile_stop()
        assert launches.pop("conv_band_trio_kernel")[0] == 1 and launches.pop("wgrad_reduce_kernel")[0] == 1
        assert bool(launches) == (ahead and parts != two)
        for i, t in enumerate(outs):
            assert torch.equal(t, want[i]) or (parts == two and i in (0, 3))


# The wide tiles' position in the reduction: scalar where the channels are whole stages (of 128 or 64 bytes), per lane otherwise, down to
# several taps in a stage; taps that wrap rows, padding wider than the image border, strides with and without pixel classes, images of a
# single row or column, tiles that span images.
@pytest.mark.parametrize("shape", [(3, 128, 7, 9, 136, 3, 3, 1, (1, 1)), (2, 256, 5, 11, 64, 5, 3, 1, (4, 0)), (5, 64, 6, 6, 192, 3, 3, 1, (0, 2)),
                                   (3, 16, 9, 8, 130, 5, 5, 1, (2, 2)), (2, 48, 10, 7, 70, 1, 7, 1, (0, 3)), (4, 144, 1, 13, 128, 1, 3, 1, (0, 1)),
                                   (3, 128, 13, 1, 128, 3, 1, 1, (1, 0)), (3, 128, 11, 12, 128, 3, 3, 2, (1, 1)), (2, 128, 9, 10, 256, 1, 1, 2, (0, 0)),
                                   (2, 136, 12, 9, 72, 4, 3, 2, (1, 0)), (2, 128, 13, 11, 128, 5, 5, 3, (2, 2)), (9, 384, 1, 1, 130, 1, 1, 1, (0, 0))])
def test_reduction_positions_of_wide_tiles(shape):
    desc, od, (xq, wq, dyq) = random_layer(shape, 21)
    for op in (B.OP_CONV_FWD, B.OP_CONV_BWD_DATA):
        for variant in (B.VARIANT_WIDE128, B.VARIANT_WIDE256, B.VARIANT_WIDE_SQ128, B.VARIANT_WIDE_SQ128_DEEP, B.VARIANT_WIDE_128X64, B.VARIANT_WIDE_CELLS):
            if not B.int8t_conv_variant_ok(op, desc, variant):
                continue
            B.int8t_conv_select_variant(op, desc, variant)
            try:
                conv_pass_elementwise(op, desc, od, xq, wq, dyq, True)
            finally:
                B.int8t_conv_select_variant(op, desc, B.VARIANT_AUTO)


# Backward-weight of a stem, which runs in its space-to-depth form, and of a plain layer with that form's geometry, in turn on one thread,
# each with the scratch it asked for at the start: either pass has its own plan (one share, whose tile is the result, belongs to the plain
# layer), and nothing is written beyond dw.  5x5, 6x6 and 9x9 filters become 3x3 and 5x5, 2x2 ones 1x1.
@pytest.mark.parametrize("stem,plain", [((2, 3, 32, 32, 12, 5, 5, 2, (2, 2)), (2, 12, 16, 16, 12, 3, 3, 1, (1, 1))),
                                        ((2, 3, 32, 32, 12, 6, 6, 2, (2, 2)), (2, 12, 16, 16, 12, 3, 3, 1, (1, 1))),
                                        ((2, 4, 23, 24, 24, 9, 9, 2, (4, 4)), (2, 16, 12, 12, 24, 5, 5, 1, (2, 2))),
                                        ((2, 3, 32, 32, 12, 2, 2, 2, (0, 0)), (2, 12, 16, 16, 12, 1, 1, 1, (0, 0)))])
def test_stems_and_plain_layers_of_one_geometry(stem, plain):
    layers = []
    for shape in (stem, plain):
        desc, od, (xq, wq, dyq) = random_layer(shape, shape[5])
        want, ov = oracle.wrap32(oracle.conv_bwd_weight(od, xq, dyq))
        assert ov == 0
        ws = torch.empty(B.int8t_workspace_bytes(B.OP_CONV_BWD_WEIGHT, desc), dtype=torch.uint8, device=DEV)
        layers.append((desc, dev(pack_act(xq)), dev(pack_act(dyq)), want, ws))
    one, guard = torch.ones(1, device=DEV), 4096
    for i in (0, 1, 0, 1, 1, 0):
        desc, xq, dyq, want, ws = layers[i]
        dw = torch.full((want.size + guard,), 7.0, device=DEV)
        acc = torch.full((want.size + guard,), 7, dtype=torch.int32, device=DEV)
        B.int8t_conv_bwd_weight(desc, xq, one, dyq, one, dw[:want.size], acc[:want.size], ws)
        torch.cuda.synchronize()
        assert np.array_equal(acc[:want.size].cpu().numpy().reshape(want.shape), want) and bool((acc[want.size:] == 7).all())
        assert np.array_equal(dw[:want.size].cpu().numpy().reshape(want.shape), want.astype(np.float32)) and bool((dw[want.size:] == 7.0).all())


# A plain 1x1 layer whose shared launch takes one share of the two or four that the pass takes by itself, and in between a stem whose rewritten
# geometry is the same, planned for the other kernel with as many shares: nothing of either is taken over by the other, bit for bit the
# calls one by one.
@pytest.mark.parametrize("N,H,W", [(32, 2, 1), (64, 2, 2), (50, 2, 3)])
def test_shares_of_a_layer_after_a_stem_of_its_geometry(N, H, W):
    plain = LayerStep(inputs.Layer("layer", N, 12, H, W, 4, 1, 1, stride=(1, 1), pad=(0, 0)), keep_acc=True, requantize_deviation=False)
    stem = LayerStep(inputs.Layer("layer", N, 3, 2 * H, 2 * W, 4, 2, 2, stride=(2, 2), pad=(0, 0)), requantize_deviation=False)
    g = torch.Generator(device=DEV).manual_seed(17)
    for st in (plain, stem):
        for t in (st.x, st.w, st.dy):
            t.normal_(generator=g)
        st.clip.fill_(1.5)
        B.int8t_layer_step(st.desc, st._layer_buffers, B.STEP_ABSMAX | B.STEP_QUANT_XW | B.STEP_QUANT_G, 3)
    outs = [plain.y, plain.y_acc, plain.dx, plain.dx_acc, plain.dw, plain.dw_acc]
    plain.fwd()
    plain.bwd_data()
    plain.bwd_weight()
    stem.bwd_weight()
    want, stem_dw = [t.clone() for t in outs], stem.dw.clone()
    two = B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    for parts in (two, two | B.STEP_FWD, two):
        for t in outs[2:] + [stem.dw]:
            t.fill_(7)
        B.int8t_layer_step(plain.desc, plain._layer_buffers, parts)
        B.int8t_layer_step(stem.desc, stem._layer_buffers, B.STEP_BWD_WEIGHT)
        torch.cuda.synchronize()
        for a, b in zip(outs + [stem.dw], want + [stem_dw]):
            assert torch.equal(a, b)
