"""Backward of the element-wise middle  v = x (*|+) shift(act(z))  between two FCs: planes that are no multiple of 8 pixels,
shifts along both axes in both directions, up to and beyond the image's size, several slices, every activation and blend,
channel counts that fill no tile.  The bounds are those of every parity test (bf16: 2e-2 of the tensor's norms)."""
import math

import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (N, C, H, W), groups of the first FC, groups and outputs of the second, activation, blend, slices (c0, c1, dh, dw)
CASES = [
    ((1, 8, 1, 4), 1, 1, 8, "gelu", "mul", [(4, 8, 0, 1)]),                                     # one unit of 4 pixels
    ((3, 16, 7, 7), 2, 1, 16, "gelu", "mul", [(8, 16, 0, 1)]),                                  # planes of 49 pixels
    ((3, 16, 7, 7), 2, 1, 24, "relu", "mul", [(0, 5, 1, -1), (5, 9, -2, 0), (11, 16, 0, -3)]),  # three slices and a gap
    ((2, 24, 5, 9), 3, 3, 12, "abs", "add", [(0, 24, -1, 2)]),                                  # every channel shifted
    ((2, 24, 8, 8), 3, 1, 40, None, "mul", [(3, 20, 2, 1)]),                                    # aligned planes, no activation
    ((2, 16, 6, 10), 1, 1, 16, "gelu", "add", [(0, 4, 6, 0), (4, 8, 0, -10), (8, 12, -9, 3), (12, 16, 5, 9)]),  # out of the image
    ((2, 16, 6, 10), 1, 1, 16, "gelu", "mul", [(0, 4, 1, -10), (4, 8, 1, -9), (8, 12, -1, 9)]),  # flat offsets 0 and 1
    ((2, 16, 4, 6), 1, 1, 16, "relu", "mul", []),                                               # no shift
    ((40, 48, 14, 14), 8, 1, 80, "gelu", "mul", [(24, 48, 0, 1)]),
    ((9, 128, 7, 7), 8, 1, 130, "gelu", "mul", [(64, 128, -1, -1)]),                        
    ((2, 64, 9, 13), 8, 1, 512, "relu", "add", [(32, 64, 1, 0)]),                               # a shift by a row
    ((2, 16, 7, 9), 2, 1, 16, "sin", "mul", [(8, 16, 0, 1)]),                                   # the fourth activation
]


def _blob(C, g1, g2, out, act, blend, slices):
    lines, k = [f"%1 = unfold %0 kh=3 kw=3", f"%2 = fc %1 groups={g1} out={C}"], 2
    if act:
        lines.append(f"%{k + 1} = unary %{k} op={act}")
        k += 1
    for c0, c1, dh, dw in slices:
        lines.append(f"%{k + 1} = shift %{k} dh={dh} dw={dw} c0={c0} c1={c1}")
        k += 1
    lines += [f"%{k + 1} = binary %0 %{k} op={blend}", f"%{k + 2} = fc %{k + 1} groups={g2} out={out}", f"output %{k + 2}"]
    return wl.HEADER + "\n".join(lines) + "\n"


@pytest.mark.parametrize("shape,g1,g2,out,act,blend,slices", CASES)
def test_mid_adjoint(oracle, shape, g1, g2, out, act, blend, slices):
    from paper_2304_07741_amd import harness

    C = shape[1]
    k1 = C // g1 * 9
    case = wl._case("mid_adjoint", _blob(C, g1, g2, out, act, blend, slices), shape, "bf16", 17,
                    [(g1, C // g1, k1), (g2, out // g2, C // g2)], [math.sqrt(2.0 / k1), math.sqrt(2.0 / (C // g2))])
    res, r, dy = harness.run_case(case)
    names = [d["name"] for d in r.launches(1)]
    assert "ufc_mid_bwd" in names, names
    check_against_oracle(oracle, case, res, dy)
    r.close()
