"""Window loads of fp32 tensors and the hand-over of a window's gradients in fused chains, on planes small enough that most
windows leave the image: widths that allow one, two and four pixels per thread, windows with constant and with general
sizes, a displaced window, an fp32 tensor between two units of a bf16 DAG.  At most 25 terms a sum; the bounds are those of
every parity test (fp32 1e-5, bf16 2e-2 of the tensor's norms)."""
import math

import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

PLANES = [(2, 12, 7, 9), (3, 12, 5, 4), (1, 20, 6, 10), (2, 12, 8, 8)]
WINDOWS = [(3, 3), (5, 5), (1, 3), (5, 1), (3, 5)]
TAIL = "%{c} = softmax %{b} axis=T\n%{d} = binary %{b} %{c} op=mul\n%{e} = fold %{d} op=sum\noutput %{e}\n"


@pytest.mark.parametrize("shape", PLANES)
@pytest.mark.parametrize("kh,kw", WINDOWS)
@pytest.mark.parametrize("head", ["plain", "shift", "fc"])
def test_chain_windows(oracle, head, kh, kw, shape):
    from paper_2304_07741_amd import harness

    C = shape[1]
    lines, src, w = "", 0, []
    if head == "shift":
        lines, src = f"%1 = shift %0 dh=-1 dw=2 c0=0 c1={C // 2}\n", 1
    if head == "fc":
        lines, src, w = f"%1 = fc %0 groups=1 out={C}\n", 1, [(1, C, C)]
    body = lines + f"%{src + 1} = unfold %{src} kh={kh} kw={kw}\n" + TAIL.format(b=src + 1, c=src + 2, d=src + 3, e=src + 4)
    case = wl._case("chain_windows", wl.HEADER + body, shape, "bf16" if head == "fc" else "f32", 23, w, [1.0 / math.sqrt(C)] * len(w))
    res, r, dy = harness.run_case(case)
    assert "chain_fwd" in [d["name"] for d in r.launches(0)]
    check_against_oracle(oracle, case, res, dy)
    r.close()
