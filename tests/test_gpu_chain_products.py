"""Fused chains over windows, backward: sums with a product of two registers as one instruction, the softmax over taps with its gradient in
the accumulator, planes that one workgroup holds whole (no halo), and the planes just beside that."""
import pytest

from test_gpu_parity import _mk, check_against_oracle

pytestmark = pytest.mark.gpu

BODIES = [
    # the softmax's values used twice on: its gradient is a sum with a product
    "%1 = unfold %0 kh=3 kw=3\n%2 = softmax %1 axis=T\n%3 = binary %2 %1 op=mul\n%4 = unary %3 op=gelu\n%5 = fold %4 op=sum\noutput %5\n",
    "%1 = unary %0 op=relu\n%2 = unfold %1 kh=3 kw=3\n%3 = softmax %2 axis=T\n%4 = binary %3 %2 op=mul\n%5 = fold %4 op=avg\noutput %5\n",
    # not kept: the gradient goes to a register
    "%1 = unfold %0 kh=3 kw=3\n%2 = softmax %1 axis=T\n%3 = fold %2 op=max\noutput %3\n",
    # two softmaxes, one of the other's result
    "%1 = unfold %0 kh=3 kw=3\n%2 = softmax %1 axis=T\n%3 = binary %2 %1 op=mul\n%4 = softmax %3 axis=T\n%5 = binary %4 %2 op=mul\n%6 = fold %5 op=sum\noutput %6\n",
    "%1 = unfold %0 kh=5 kw=5\n%2 = softmax %1 axis=T\n%3 = binary %2 %1 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
]
# 32 x 32 is one tile of two pixels per thread; 33 x 32 and 64 x 17 are not; 5 x 3 and 7 x 9 are smaller than a wavefront
SHAPES = [(2, 10, 32, 32), (1, 3, 33, 32), (2, 5, 64, 17), (3, 4, 5, 3), (2, 33, 7, 9), (1, 4, 16, 64)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("idx", range(len(BODIES)))
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_products_and_whole_planes(oracle, idx, shape, dtype):
    from paper_2304_07741_amd import harness

    case = _mk(BODIES[idx], shape, dtype, 970 + idx, [], f"products{idx}")
    res, r, dy = harness.run_case(case)
    assert "chain_bwd" in [d["name"] for d in r.launches(1)]
    check_against_oracle(oracle, case, res, dy)
    r.close()
