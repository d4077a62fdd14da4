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
