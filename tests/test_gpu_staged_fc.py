"""bf16 FC kernels whose source tile goes through LDS: one and several images per tile, row tiles with and without whole 8-pixel units,
planes whose last unit ends behind the tensor, padded rows and outputs, taps in pairs and alone, one to four pieces per thread,
results that are added to, fp32 results, the softmax over the outputs."""
import math

import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

SAMPLED = "%1 = unfold %0 kh=3 kw=3\n%2 = fc %1 groups={g1} out={c}\n%3 = unary %2 op=gelu\n%4 = binary %0 %3 op=mul\n%5 = fc %4 groups={g2} out={o}\noutput %5\n"
# (groups of the windowed FC, groups of the other, channels, outputs, batch and plane)
CASES = [
    (8, 1, 64, 64, (9, 7, 7)),          # merged groups, taps in pairs, several images per tile, the last tile with fewer
    (8, 1, 128, 96, (5, 9, 7)),         # 16 rows, outputs that end inside a workgroup's
    (8, 1, 256, 256, (3, 14, 14)),      # 32 rows: all weights in registers; a plane that ends inside a unit
    (8, 1, 256, 300, (40, 8, 8)),       # several images of 32 rows
    (8, 1, 512, 512, (3, 7, 7)),        # 64 rows: weights streamed
    (2, 1, 80, 80, (6, 13, 11)),        # 40 rows padded to 64
    (8, 2, 160, 160, (2, 27, 29)),      # 20 rows; rows of 29 pixels in tiles of rows that are no whole units
    (4, 1, 100, 72, (1, 50, 33)),       # 25 rows, outputs of a group that fill no tile
    (1, 1, 64, 384, (2, 20, 56)),       # one group, tiles of one and two rows, three quarters of a workgroup's outputs
    (1, 1, 128, 128, (1, 9, 10)),       # four pieces per thread
]


@pytest.mark.parametrize("idx", range(len(CASES)))
def test_staged(oracle, idx):
    from paper_2304_07741_amd import harness

    g1, g2, c, o, (n, h, w) = CASES[idx]
    k1 = c // g1 * 9
    case = wl._case(f"staged{idx}", wl.HEADER + SAMPLED.format(g1=g1, g2=g2, c=c, o=o), (n, c, h, w), "bf16", 90 + idx,
                    [(g1, c // g1, k1), (g2, o // g2, c // g2)], [math.sqrt(2.0 / k1), math.sqrt(2.0 / (c // g2))])
    res, r, dy = harness.run_case(case)
    assert r.info.fused == 1
    check_against_oracle(oracle, case, res, dy)
    r.close()


@pytest.mark.parametrize("c,shape", [(72, (3, 7, 7)), (128, (2, 9, 13)), (130, (1, 28, 28))])
def test_softmax_and_fp32_results(oracle, c, shape):
    from paper_2304_07741_amd import harness

    case = wl._case("staged_softmax", wl.HEADER + wl.blob_involution(c).split("\n", 1)[1], (shape[0], c, *shape[1:]), "bf16", 7,
                    [(1, 9, c), (1, c, c)], [0.5, 1.0 / math.sqrt(c)])
    res, r, dy = harness.run_case(case)
    check_against_oracle(oracle, case, res, dy)
    r.close()
    body = "%1 = unfold %0 kh=3 kw=3\n%2 = fc %1 groups=2 out=64\n%3 = unary %2 op=gelu\noutput %3\n"   # fp32 between the units
    case = wl._case("staged_f32", wl.HEADER + body, (3, 64, *shape[1:]), "bf16", 8, [(2, 32, 288)], [1.0 / 17.0])
    res, r, dy = harness.run_case(case)
    check_against_oracle(oracle, case, res, dy)
    r.close()
