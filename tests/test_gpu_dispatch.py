"""GPU parity at the borders of the library's own choices: the sizes at which a kernel's launch shape or inner path
changes, against the CPU oracle.  Bars as in test_gpu_parity.py."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_1912_12607_amd import inputs  # noqa: E402
from test_gpu_parity import RTN, STO, check_dsgc  # noqa: E402


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
