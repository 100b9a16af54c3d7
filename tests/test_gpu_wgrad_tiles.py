"""Weight gradient of bf16 FCs without a window (64 x 64 and 128 x 64 tiles, steps of eight 8-pixel units counted through the images):
planes of one unit, a unit and a pixel, seven units, ragged rows of units; outputs and rows that end inside a tile; groups; more steps
than slices and fewer.  And of FCs behind a 3x3 window by image rows through LDS: several images per step, the last step with fewer; row
tiles with their halo; rows of one and two units, ragged and whole; rows and outputs of a group that fill no tile."""
import math

import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

# (groups, channels, outputs, batch, plane)
CASES = [
    (1, 64, 64, 3, (2, 4)),        # planes of one unit: eight images per step
    (1, 64, 130, 5, (3, 3)),       # a unit and a pixel
    (1, 100, 72, 21, (7, 7)),      # seven units: a step ends inside an image
    (2, 160, 192, 2, (5, 13)),     # two groups of 80 rows and 96 outputs; nine units
    (1, 512, 384, 2, (7, 9)),      # 128 x 64 tiles, one step per slice
    (4, 256, 512, 3, (10, 11)),    # 128 x 64 tiles in groups
    (1, 64, 64, 50, (28, 29)),     # many steps per slice, the last one short
    (1, 64, 64, 1, (1, 8)),        # a single unit
    (1, 160, 144, 9, (9, 7)),      # three tiles of outputs: 64 x 64, a slice more than fits for its four steps
    (1, 132, 136, 500, (7, 7)),    # the same in 128 x 64 tiles from 420 steps on
]


@pytest.mark.parametrize("idx", range(len(CASES)))
def test_weight_gradient(oracle, idx):
    from paper_2304_07741_amd import harness

    g, c, o, n, (h, w) = CASES[idx]
    body = f"%1 = fc %0 groups={g} out={o}\noutput %1\n"
    case = wl._case(f"wgrad{idx}", wl.HEADER + body, (n, c, h, w), "bf16", 60 + idx, [(g, o // g, c // g)], [1.0 / math.sqrt(c // g)])
    res, r, dy = harness.run_case(case)
    check_against_oracle(oracle, case, res, dy)
    r.close()


WINDOWS = [
    (8, 256, (9, 14, 14)),     # one image per step; two units, the second with six pixels
    (8, 512, (33, 7, 7)),      # four images per step, the last with one; tiles of 32 of 64 rows
    (4, 128, (40, 9, 6)),      # three images per step, rows of six pixels
    (8, 480, (33, 8, 8)),      # whole units, 60 rows in 64
    (1, 32, (3, 40, 13)),      # row tiles, the last one shorter
    (2, 64, (8, 16, 16)),      # two row tiles of whole units
    (8, 144, (10, 12, 12)),    # 18 rows in 32, sums of partials four wide
    (2, 96, (70, 4, 8)),       # six images per step
]


@pytest.mark.parametrize("idx", range(len(WINDOWS)))
def test_weight_gradient_of_a_window(oracle, idx):
    from paper_2304_07741_amd import harness

    g, c, (n, h, w) = WINDOWS[idx]
    body = f"%1 = unfold %0 kh=3 kw=3\n%2 = fc %1 groups={g} out={c}\n%3 = unary %2 op=gelu\n%4 = binary %0 %3 op=mul\n%5 = fc %4 groups=1 out=64\noutput %5\n"
    k1 = c // g * 9
    case = wl._case(f"wgrad_window{idx}", wl.HEADER + body, (n, c, h, w), "bf16", 70 + idx, [(g, c // g, k1), (1, 64, c)], [math.sqrt(2.0 / k1), math.sqrt(2.0 / c)])
    res, r, dy = harness.run_case(case)
    assert r.info.fused == 1
    check_against_oracle(oracle, case, res, dy)
    r.close()
