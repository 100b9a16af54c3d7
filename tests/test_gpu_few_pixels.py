"""bf16 FC kernels where the launch is small and a tile takes 16 or 32 outputs instead of 64 (32 under a window): output counts
at the edges of those tiles, one to many row chunks, split and unsplit, planes that are no multiple of 8 pixels."""
import math

import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

SAMPLED = "%1 = unfold %0 kh={k} kw={k}\n%2 = fc %1 groups={g1} out={c}\n%3 = unary %2 op=gelu\n%4 = binary %0 %3 op=mul\n%5 = fc %4 groups={g2} out={o}\noutput %5\n"
CASES = [
    (3, 8, 1, 256, 256, (1, 256, 14, 14)), (3, 8, 1, 512, 512, (2, 512, 7, 7)), (3, 2, 1, 80, 65, (3, 80, 9, 13)), (3, 1, 1, 24, 33, (1, 24, 5, 4)),
    (3, 1, 2, 40, 34, (2, 40, 6, 7)), (1, 1, 1, 96, 17, (5, 96, 11, 5)), (1, 3, 1, 48, 48, (2, 48, 8, 8)), (5, 2, 1, 66, 129, (1, 66, 7, 7)),
    (3, 8, 1, 128, 128, (8, 128, 28, 28)), (3, 8, 1, 256, 256, (16, 256, 14, 14)), (1, 1, 1, 16, 320, (9, 16, 13, 15))]


@pytest.mark.parametrize("k,g1,g2,c,o,shape", CASES)
def test_small_launches(oracle, k, g1, g2, c, o, shape):
    from paper_2304_07741_amd import harness

    C = shape[1]
    body = SAMPLED.format(k=k, g1=g1, g2=g2, c=c, o=o)
    if k == 1:
        body = body.replace("%1 = unfold %0 kh=1 kw=1\n%2 = fc %1", "%2 = fc %0")
        for n in range(2, 6):
            body = body.replace(f"%{n}", f"%{n - 1}")
    K1 = C // g1 * k * k
    case = wl._case("few_pixels", wl.HEADER + body, shape, "bf16", 41, [(g1, c // g1, K1), (g2, o // g2, c // g2)],
                    [math.sqrt(2.0 / K1), math.sqrt(2.0 / (c // g2))])
    res, r, dy = harness.run_case(case)
    assert r.info.fused == 1
    check_against_oracle(oracle, case, res, dy)
    r.close()
