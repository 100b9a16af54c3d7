"""Where the planner cuts chains: planes that a workgroup holds whole (no halo) neither split a plan that is faster in fewer pieces nor make it outgrow the library's
static workspace, and where more pieces are faster it gets them."""
import os
import subprocess
import sys

import pytest

from paper_2304_07741_amd import binding as B
from paper_2304_07741_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

TAP_SOFTMAX = ("%1 = unary %0 op=relu\n%2 = unfold %1 kh=3 kw=3\n%3 = softmax %2 axis=T\n%4 = binary %3 %2 op=mul\n%5 = unary %4 op=gelu\n"
               "%6 = fold %5 op=sum\noutput %6\n")
SHIFTED = ("%1 = unfold %0 kh=3 kw=3\n%2 = shift %1 dh=2 dw=0 c0=48 c1=96\n%3 = binary %0 %2 op=mul\n%4 = fold %3 op=avg\n%5 = binary %4 %0 op=add\noutput %5\n")
AVG5 = ("%1 = unary %0 op=abs\n%2 = unfold %1 kh=5 kw=5\n%3 = binary %0 %2 op=mul\n%4 = fold %3 op=avg\n%5 = unary %4 op=expclip lo=-4 hi=4\n"
        "%6 = shift %5 dh=-2 dw=0 c0=0 c1=48\n%7 = softmax %6 axis=C\n%8 = unary %7 op=gelu\noutput %8\n")
GATED_MAX = ("%1 = softmax %0 axis=C\n%2 = unary %1 op=relu\n%3 = unfold %2 kh=5 kw=5\n%4 = fold %3 op=max\n%5 = binary %2 %4 op=mul\n"
             "%6 = shift %5 dh=0 dw=1 c0=0 c1=48\n%7 = shift %6 dh=1 dw=0 c0=24 c1=48\noutput %7\n")


def _plan(body, shape, flags=0, dtype=B.CANVAS_BF16):
    h = B.canvas_dag_compile(wl.HEADER + body, shape, dtype, flags)
    i = B.canvas_dag_query(h)
    refused = B.load().canvas_dag_forward_static(h, None, None, None, None) == -5
    B.canvas_dag_destroy(h)
    return i.n_launches_fwd, i.n_launches_bwd, refused


@pytest.mark.parametrize("body,shape,want", [
    (TAP_SOFTMAX, (6, 96, 16, 16), (1, 1)),     # 26 us, 36 in two pieces
    (SHIFTED, (9, 96, 32, 32), (1, 1)),         # 72 us, 93 in two pieces
    (AVG5, (16, 96, 27, 15), (4, 4)),           # 214, 239 in five
    (GATED_MAX, (7, 96, 19, 25), (4, 4)),       # 143, 212 in three
])
def test_pieces(body, shape, want):
    assert _plan(body, shape)[:2] == want


@pytest.mark.parametrize("flags", [0, B.CANVAS_OPT_INFERENCE])
@pytest.mark.parametrize("body,shape", [(TAP_SOFTMAX, (512, 96, 14, 14)), (SHIFTED, (64, 96, 32, 32)), (SHIFTED, (512, 96, 32, 32)), (AVG5, (512, 48, 12, 12)),
                                        (GATED_MAX, (512, 48, 12, 12))])
def test_static_workspace(body, shape, flags):
    for dtype in (B.CANVAS_BF16, B.CANVAS_F32):
        assert not _plan(body, shape, flags, dtype)[2]


GATE = "%1 = fc %0 groups=1 out=48\n%2 = unary %1 op=expclip lo=-4 hi=4\n%3 = unary %2 op=relu\n%4 = binary %1 %3 op=add\n%5 = softmax %4 axis=C\noutput %5\n"


@pytest.mark.parametrize("shape", [(5, 48, 14, 14), (32, 48, 8, 8), (3, 48, 12, 8)])
def test_values_kept_across_the_passes_of_a_softmax(shape):
    """Backward of the softmax over channels keeps what its first pass computes: the later passes load nothing but the gradient (5x48x14x14: 34.5 us, 42.9 with
    everything computed three times over)."""
    code = (f"from paper_2304_07741_amd import binding as B, workloads as wl\n"
            f"B.canvas_dag_destroy(B.canvas_dag_compile(wl.HEADER + {GATE!r}, {shape!r}, B.CANVAS_BF16))\n")
    p = subprocess.run([sys.executable, "-c", code], cwd=ROOT, env=dict(os.environ, CANVAS_LOG="1"), capture_output=True, text=True, check=True)
    backward = p.stderr.rsplit("program:", 1)[1].split(" pass ")
    assert len(backward) == 4 and sum(" LD " in line for part in backward[2:] for line in part.splitlines()) == 1
