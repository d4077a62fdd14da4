"""Host logic of the autograd modules that needs no GPU: what is refused before the library is called."""
import pytest

torch = pytest.importorskip("torch")

from paper_1912_12607_amd.autograd import Int8Conv2d  # noqa: E402


# The library takes the filters' channel count from the input's: one that is not the weights' would read and write past their end.
@pytest.mark.parametrize("grad", [True, False])
@pytest.mark.parametrize("C,K,kernel,groups", [(20, 32, 3, 1), (20, 8, 1, 1), (16, 16, 3, 16)])
def test_input_of_another_channel_count_is_refused(C, K, kernel, groups, grad):
    m = Int8Conv2d(C, K, kernel, padding=kernel // 2, groups=groups, device="cpu")
    with torch.set_grad_enabled(grad):
        for c in (C - 4, C + 4, 1, 2 * C):
            with pytest.raises(RuntimeError, match=f"{c} channels.*{C}"):
                m(torch.zeros(2, c, 9, 9))
