"""Host logic of LayerStep that needs no GPU: which kernel variants tune_kernels() selects, from made-up timings."""
import ctypes as C

import pytest

torch = pytest.importorskip("torch")

from paper_1912_12607_amd import binding as B  # noqa: E402
from paper_1912_12607_amd.inputs import Layer  # noqa: E402
from paper_1912_12607_amd.step import LayerStep  # noqa: E402

OPS = {"fwd": B.OP_CONV_FWD, "bwd_data": B.OP_CONV_BWD_DATA, "bwd_weight": B.OP_CONV_BWD_WEIGHT}


ALL = ("fwd", "bwd_data", "bwd_weight")


# The three passes, and the two backward ones, take 10 us with the library's own choice and t_all, t_two with variants selected.
@pytest.mark.parametrize("overlap,faster,t_all,t_two,kept", [
    (0, ALL, 9.0, 11.0, ALL),                    # (on one stream no step runs the two backward passes by themselves)
    (0, ALL, 11.0, 9.0, ()),
    (0, ("bwd_weight",), 11.0, 9.0, ()),         # one selection is enough to lose the shared launch
    (1, ALL, 9.0, 9.0, ALL),
    (1, ALL, 9.0, 11.0, ("fwd",)),
    (1, ("fwd",), 9.0, 11.0, ("fwd",)),
    (1, ("fwd",), 11.0, 9.0, ()),                # (a step that keeps its clip value runs on one stream)
    (0, (), 11.0, 11.0, ())])
def test_tune_kernels_against_the_shared_launch(monkeypatch, overlap, faster, t_all, t_two, kept):
    monkeypatch.setattr(B, "_ptr", lambda t: None if t is None else C.c_void_p(t.data_ptr()))
    st = LayerStep(Layer("layer", 2, 80, 8, 8, 96, 3, 3, stride=(1, 1), pad=(1, 1)), device="cpu")
    st._tuned_overlap = overlap
    calls = {id(st._k_fwd): "fwd", id(st._k_bwd_data): "bwd_data"}      # (backward-weight's call is bound anew with its scratch)

    def selected():
        return {name: B.lib.int8t_conv_selected_variant(op, C.byref(st.desc)) for name, op in OPS.items()}

    def time_us(call, reps):
        name = calls.get(id(call)) or ("bwd_weight" if call is st._k_bwd_weight else None)
        if name is None:          # the passes together
            two = call.args[0] == B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
            assert two or call.args[0] == B.STEP_FWD | B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
            return (t_two if two else t_all) if any(v for n, v in selected().items() if not two or n != "fwd") else 10.0
        return 5.0 if name in faster and selected()[name] != B.VARIANT_AUTO else 8.0

    monkeypatch.setattr(st, "_time_us", time_us, raising=False)
    monkeypatch.setattr(st, "refresh_scratch", lambda: None)
    try:
        out = st.tune_kernels()
        assert tuple(n for n, v in selected().items() if v != B.VARIANT_AUTO) == kept
        assert tuple(n for n, v in out.items() if v[0] != B.VARIANT_NAMES[B.VARIANT_AUTO]) == kept
    finally:
        for op in OPS.values():
            B.int8t_conv_select_variant(op, st.desc, B.VARIANT_AUTO)


# The two-stream step of a depthwise layer: in two halves, the second behind the first, only where the library takes the codes into the
# launch of the passes; elsewhere g_z is quantized beside the forward pass, before the main stream waits for it.
@pytest.mark.parametrize("shape,halves", [((2, 5, 56, 56), True), ((2, 5, 32, 36), True), ((2, 64, 7, 7), True), ((4, 32, 14, 14), True),
                                          ((2, 5, 57, 57), False), ((2, 5, 43, 43), False), ((2, 5, 55, 55), False), ((2, 5, 45, 45), False),
                                          ((2, 32, 65, 63), False), ((4, 16, 8, 3), False)])
def test_two_stream_order_of_depthwise_layers(monkeypatch, shape, halves):
    N, C_, H, W = shape
    monkeypatch.setattr(B, "_ptr", lambda t: None if t is None else C.c_void_p(t.data_ptr()))
    st = LayerStep(Layer("layer", N, C_, H, W, C_, 3, 3, stride=(1, 1), pad=(1, 1), groups=C_), device="cpu", requantize_deviation=False)
    seen = []

    class Stream:
        def __init__(self, name):
            self.name = name

        def wait_event(self, event):
            seen.append((self.name, "waits"))

    class Event:
        def record(self, stream):
            pass

    main = Stream("main")
    monkeypatch.setattr("paper_1912_12607_amd.step.side_stream", lambda dev: Stream("side"))
    monkeypatch.setattr(torch.cuda, "Event", Event)
    monkeypatch.setattr(B, "stream_pointer", lambda s: s.name)
    for name in ("prepare", "search", "qdy", "fwd"):
        monkeypatch.setattr(st, "_k_" + name, lambda *a, name=name: seen.append((a[-1], name)))
    monkeypatch.setattr(st, "_k_step", lambda parts, seed, sp: seen.append((sp, parts)))
    st.run(seed=1, stream=main, search=True, overlap=1)
    on_main = [what for name, what in seen if name == "main"]
    bwd = B.STEP_BWD_DATA | B.STEP_BWD_WEIGHT
    assert on_main == ["prepare", "search"] + (["waits", B.STEP_QUANT_G | bwd] if halves else ["qdy", "waits", bwd])
    assert [what for name, what in seen if name == "side"][1:] == (
        [B.STEP_ABSMAX | B.STEP_QUANT_XW | B.STEP_FWD] if halves else [B.STEP_ABSMAX | B.STEP_QUANT_XW, "fwd"])
