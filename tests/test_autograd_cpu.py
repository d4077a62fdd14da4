"""Host logic of the autograd modules that needs no GPU: what is refused before the library is called, and what the library is
asked for (its calls recorded, on host tensors)."""
import types

import pytest

torch = pytest.importorskip("torch")

from paper_1912_12607_amd import autograd as A  # noqa: E402
from paper_1912_12607_amd import binding as B  # noqa: E402
from paper_1912_12607_amd.autograd import Int8Conv2d, Int8Linear  # noqa: E402


@pytest.fixture
def calls(monkeypatch):
    """The library's calls, recorded as (name, arguments); results keep what their memory held."""
    seen = []

    def record(name):
        monkeypatch.setattr(B, name, lambda *args: seen.append((name, args)))

    for name in ("int8t_layer_step", "int8t_layer_infer", "int8t_layer_backward", "int8t_dsgc_clip", "int8t_quantize"):
        record(name)

    device = A._device

    def address(t):         # (a host tensor marked `foreign` stands for one the GPU cannot reach)
        return device(types.SimpleNamespace(is_cuda=not getattr(t, "foreign", False), is_contiguous=t.is_contiguous, data_ptr=t.data_ptr))

    monkeypatch.setattr(A, "_device", address)
    monkeypatch.setattr(B, "_ptr", lambda t: None if t is None else address(t))
    return seen


# The library takes the filters' channel count from the input's: one that is not the weights' would read and write past their end.
@pytest.mark.parametrize("grad", [True, False])
@pytest.mark.parametrize("C,K,kernel,groups", [(20, 32, 3, 1), (20, 8, 1, 1), (16, 16, 3, 16)])
def test_input_of_another_channel_count_is_refused(C, K, kernel, groups, grad):
    m = Int8Conv2d(C, K, kernel, padding=kernel // 2, groups=groups, device="cpu")
    with torch.set_grad_enabled(grad):
        for c in (C - 4, C + 4, 1, 2 * C):
            with pytest.raises(RuntimeError, match=f"{c} channels.*{C}"):
                m(torch.zeros(2, c, 9, 9))


# Tensors that a program may replace (a clip value out of a checkpoint, candidates of its own) are checked as the others are.
@pytest.mark.parametrize("name,period,strided", [("clip", 1, False), ("clip", 2, False), ("deviation", 1, False), ("deviation", 2, False),
                                                 ("ratios", 1, False), ("ratios", 1, True)])
def test_addresses_of_replaced_tensors_are_checked(calls, name, period, strided):
    m = Int8Conv2d(8, 8, 3, padding=1, dsgc_period=period, device="cpu")
    x = torch.zeros(2, 8, 5, 5, requires_grad=True)
    m(x).sum().backward()
    assert [c[0] for c in calls] == ["int8t_layer_step", "int8t_layer_backward"]
    t = getattr(m, name)
    t = t[::2] if strided else t.clone()
    t.foreign = not strided
    setattr(m, name, t)
    y = m(x)
    with pytest.raises(AssertionError, match="device-resident"):
        y.sum().backward()
    assert len(calls) == 3


# Whether a forward-mode level is open is asked of a private name of torch, which another release need not have.
def test_without_torchs_forward_mode_level(calls, monkeypatch):
    assert A._plain_eager()
    monkeypatch.delattr(torch.autograd.forward_ad, "_current_level")
    assert A._plain_eager()
    assert Int8Conv2d(8, 8, 3, device="cpu")(torch.zeros(1, 8, 5, 5)).shape == (1, 8, 3, 3)


# Sums over the rows in the library's call are one block per 64 columns: many rows (a batch of tokens) are summed by torch.
@pytest.mark.parametrize("rows,inside", [(1, True), (1024, True), (1025, False), (4096, False)])
def test_bias_gradient_of_many_rows(calls, rows, inside):
    m = Int8Linear(8, 6, device="cpu")
    x, g = torch.zeros(rows, 8, requires_grad=True), torch.randn(rows, 6)
    y = A._Int8ConvFn.apply(x, m.weight, m, True, m.bias, True)
    db = torch.autograd.grad(y, [m.bias, x], g)[0]
    name, args = calls[-1]
    assert name == "int8t_layer_backward" and db.shape == (6,)
    if inside:
        assert args[4].data_ptr() == db.data_ptr()
    else:
        assert args[4] is None and torch.equal(db, g.sum(0))
