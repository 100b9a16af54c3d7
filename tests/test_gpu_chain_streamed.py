"""Windows that are folded as they are loaded: every fold, blend and side, a unary on the taps, two windows against each other, values that a fold's
adjoint spreads over the taps; windows of three and five columns; bf16 tensors and fp32 ones between two units; rows of whole vectors and
tensors large enough for these programs, and forms beside them that must keep their lanes."""
import pytest

from test_gpu_parity import _mk, check_against_oracle

pytestmark = pytest.mark.gpu

BODIES = [
    "%1 = unfold %0 kh=3 kw=3\n%2 = fold %1 op=sum\noutput %2\n",
    "%1 = unary %0 op=gelu\n%2 = unfold %1 kh=3 kw=5\n%3 = fold %2 op=avg\noutput %3\n",
    "%1 = unary %0 op=abs\n%2 = unfold %1 kh=5 kw=3\n%3 = fold %2 op=max\noutput %3\n",
    "%1 = unfold %0 kh=5 kw=5\n%2 = binary %0 %1 op=mul\n%3 = fold %2 op=avg\noutput %3\n",
    "%1 = unfold %0 kh=3 kw=3\n%2 = binary %0 %1 op=sub\n%3 = fold %2 op=sum\noutput %3\n",
    "%1 = unary %0 op=relu\n%2 = unfold %0 kh=1 kw=3\n%3 = binary %1 %2 op=add\n%4 = fold %3 op=max\noutput %4\n",
    # (an unfolded tensor that a unit of its own writes: lanes)
    "%1 = unary %0 op=sin\n%2 = unfold %0 kh=3 kw=3\n%3 = unfold %1 kh=3 kw=3\n%4 = binary %2 %3 op=mul\n%5 = fold %4 op=sum\noutput %5\n",
    # a window over another chain's result (fp32), in turn folded
    "%1 = unfold %0 kh=3 kw=3\n%2 = fold %1 op=sum\n%3 = unfold %2 kh=5 kw=5\n%4 = binary %2 %3 op=mul\n%5 = fold %4 op=avg\noutput %5\n",
    "%1 = unfold %0 kh=3 kw=3\n%2 = fold %1 op=avg\n%3 = unary %2 op=gelu\n%4 = unfold %3 kh=3 kw=3\n%5 = fold %4 op=max\n%6 = binary %0 %5 op=mul\noutput %6\n",
    # these keep their lanes
    "%1 = unfold %0 kh=3 kw=3\n%2 = binary %0 %1 op=min\n%3 = fold %2 op=sum\noutput %3\n",
    "%1 = shift %0 dh=1 dw=-1 c0=0 c1=5\n%2 = unfold %1 kh=3 kw=3\n%3 = fold %2 op=sum\noutput %3\n",
    "%1 = unfold %0 kh=3 kw=3\n%2 = softmax %1 axis=T\n%3 = binary %0 %2 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
]
SHAPES = [(2, 100, 40, 56), (10, 53, 28, 60), (4, 101, 32, 32)]   # 8, 4 and 8 pixels per thread (test_chain_paths_host.py looks at the programs)


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("idx", range(len(BODIES)))
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_folded_windows(oracle, idx, shape, dtype):
    from paper_2304_07741_amd import harness

    case = _mk(BODIES[idx], shape, dtype, 980 + idx, [], f"streamed{idx}")
    res, r, dy = harness.run_case(case)
    assert "chain_fwd" in [d["name"] for d in r.launches(0)]
    check_against_oracle(oracle, case, res, dy)
    r.close()
