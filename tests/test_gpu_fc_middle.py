"""The middle  v = x (*|+) shift(act(z))  in the launch of the FC before it, and its adjoint in that of the FC whose data gradient it takes: several
images per tile, row tiles, merged groups, outputs that end inside a tile, shifts in both directions, past an image's ends and by the
whole image, channels in several slices; and the same middle in launches of its own, where the tensors are larger or the activation is the sine."""
import math

import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

# shape, groups of the first FC, outputs of the second, activation, blend, slices (c0, c1, dh, dw), whether the launches are joined
CASES = [
    ((5, 64, 7, 7), 8, 64, "gelu", "mul", [(32, 64, 0, 1)], True),                       # merged groups, several images per tile
    ((2, 128, 21, 13), 8, 72, "relu", "mul", [(0, 50, -1, 2), (70, 128, 2, -3)], True),  # row tiles
    ((3, 256, 14, 14), 8, 256, "abs", "add", [(0, 256, 1, 0)], True),                    # every channel shifted by a row
    ((2, 512, 7, 7), 8, 300, "gelu", "add", [(0, 100, 7, 0), (100, 200, 0, -6), (200, 300, -9, 2)], True),  # out of the image
    ((1, 80, 27, 29), 8, 80, None, "mul", [(40, 80, -2, -1)], True),                     # ten rows in 16, no activation
    ((2, 96, 8, 8), 1, 160, "gelu", "mul", [(13, 77, 3, 3)], True),                      # one group, whole units
    ((1, 256, 14, 14), 8, 256, "gelu", "mul", [], True),                                 # no shift
    ((2, 64, 9, 10), 4, 64, "sin", "mul", [(32, 64, 0, 1)], False),
    ((30, 256, 16, 16), 8, 64, "gelu", "mul", [(128, 256, 0, 1)], False),
    ((35, 144, 19, 17), 8, 100, "relu", "add", [(72, 144, -1, 1)], None),                # backward joined, forward not
]


@pytest.mark.parametrize("shape,g1,out,act,blend,slices,joined", CASES)
def test_middle(oracle, shape, g1, out, act, blend, slices, joined):
    from paper_2304_07741_amd import harness

    C, k = shape[1], 2
    lines = ["%1 = unfold %0 kh=3 kw=3", f"%2 = fc %1 groups={g1} out={C}"]
    if act:
        lines.append(f"%{k + 1} = unary %{k} op={act}")
        k += 1
    for c0, c1, dh, dw in slices:
        lines.append(f"%{k + 1} = shift %{k} dh={dh} dw={dw} c0={c0} c1={c1}")
        k += 1
    lines += [f"%{k + 1} = binary %0 %{k} op={blend}", f"%{k + 2} = fc %{k + 1} groups=1 out={out}", f"output %{k + 2}"]
    k1 = C // g1 * 9
    case = wl._case("middle", wl.HEADER + "\n".join(lines) + "\n", shape, "bf16", 23, [(g1, C // g1, k1), (1, out, C)], [math.sqrt(2.0 / k1), math.sqrt(2.0 / C)])
    res, r, dy = harness.run_case(case)
    fwd, bwd = [[d["name"] for d in r.launches(k)] for k in (0, 1)]
    assert ("ufc_mid_fwd" in fwd) == (joined is not True) and ("ufc_fc2_dgrad" in bwd) == (joined is False), (fwd, bwd)
    check_against_oracle(oracle, case, res, dy)
    r.close()
