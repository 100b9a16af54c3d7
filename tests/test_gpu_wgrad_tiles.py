"""Weight gradient of bf16 FCs without a window (64 x 64 and 128 x 64 tiles, steps of eight 8-pixel units counted through the images):
planes of one unit, a unit and a pixel, seven units, ragged rows of units; outputs and rows that end inside a tile; groups; more steps
than slices and fewer."""
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
