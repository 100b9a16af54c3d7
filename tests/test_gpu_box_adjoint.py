"""A box filter (unfold, then a sum or avg fold) whose unfolded tensor has a second reader outside the fused chain: the gradient
that this reader sends back goes through the window as well.  Sums of at most 243 terms; the bounds are those of every parity
test (fp32 1e-5, bf16 2e-2 of the tensor's norms)."""
import math

import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("fold", ["sum", "avg"])
def test_unfolded_tensor_with_a_second_reader(oracle, fold, dtype):
    from paper_2304_07741_amd import harness

    body = f"%1 = unfold %0 kh=3 kw=3\n%2 = fc %1 groups=1 out=12\n%3 = fold %1 op={fold}\n%4 = binary %2 %3 op=mul\noutput %4\n"
    case = wl._case("box_second_reader", wl.HEADER + body, (3, 12, 9, 11), dtype, 91, [(1, 12, 108)], [1.0 / math.sqrt(108)])
    res, _, dy = harness.run_case(case)
    check_against_oracle(oracle, case, res, dy)
