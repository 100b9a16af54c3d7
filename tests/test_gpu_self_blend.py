"""y = x (*|+) shift(act(x)) of one bf16 tensor, which has kernels of its own: shifts in every direction, by rows, past the image's ends and by the whole
image, in several slices; the activation before, between and behind the shifts; planes that are no multiple of eight pixels, rows shorter than a
vector; and neighbours of the form that stay programs of the fused-chain kernels."""
import pytest

from test_gpu_parity import _mk, check_against_oracle

pytestmark = pytest.mark.gpu

BODIES = [
    "%1 = unary %0 op=gelu\n%2 = shift %1 dh=0 dw=1 c0=7 c1=14\n%3 = binary %0 %2 op=mul\noutput %3\n",
    "%1 = shift %0 dh=1 dw=0 c0=0 c1=7\n%2 = shift %1 dh=0 dw=-1 c0=7 c1=14\n%3 = unary %2 op=relu\n%4 = binary %0 %3 op=add\noutput %4\n",
    "%1 = shift %0 dh=-2 dw=3 c0=0 c1=5\n%2 = unary %1 op=abs\n%3 = shift %2 dh=2 dw=-4 c0=6 c1=14\n%4 = binary %3 %0 op=mul\noutput %4\n",
    "%1 = shift %0 dh=-1 dw=-1 c0=0 c1=14\n%2 = binary %0 %1 op=mul\noutput %2\n",
    "%1 = unary %0 op=relu\n%2 = binary %1 %0 op=add\noutput %2\n",
    "%1 = unary %0 op=gelu\n%2 = shift %1 dh=40 dw=0 c0=0 c1=4\n%3 = shift %2 dh=0 dw=-40 c0=4 c1=8\n%4 = shift %3 dh=-3 dw=2 c0=8 c1=12\n%5 = binary %0 %4 op=add\noutput %5\n",
    # programs of the chain kernels: two shifts of one channel, two activations, a third use, another activation, another blend
    "%1 = shift %0 dh=1 dw=0 c0=0 c1=9\n%2 = shift %1 dh=0 dw=1 c0=5 c1=14\n%3 = binary %0 %2 op=mul\noutput %3\n",
    "%1 = unary %0 op=gelu\n%2 = unary %1 op=abs\n%3 = shift %2 dh=1 dw=1 c0=0 c1=9\n%4 = binary %0 %3 op=mul\noutput %4\n",
    "%1 = unary %0 op=gelu\n%2 = shift %1 dh=0 dw=1 c0=0 c1=9\n%3 = binary %1 %2 op=mul\n%4 = binary %0 %3 op=add\noutput %4\n",
    "%1 = unary %0 op=sin\n%2 = shift %1 dh=0 dw=1 c0=0 c1=9\n%3 = binary %0 %2 op=mul\noutput %3\n",
    "%1 = unary %0 op=relu\n%2 = shift %1 dh=0 dw=1 c0=0 c1=9\n%3 = binary %0 %2 op=max\noutput %3\n",
]
SHAPES = [(2, 14, 16, 24), (3, 14, 9, 11), (2, 14, 13, 5), (5, 14, 1, 8), (1, 14, 56, 56), (2, 14, 7, 1)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("idx", range(len(BODIES)))
def test_blend_with_itself(oracle, idx, shape):
    from paper_2304_07741_amd import harness

    case = _mk(BODIES[idx], shape, "bf16", 1040 + idx, [], f"self{idx}")
    res, r, dy = harness.run_case(case)
    assert [d["name"] for d in r.launches(0)] == ["chain_fwd"] and [d["name"] for d in r.launches(1)] == ["chain_bwd"]
    check_against_oracle(oracle, case, res, dy)
    r.close()


@pytest.mark.parametrize("blend,shift", [("mul", ""), ("add", ""), ("mul", "%2 = shift %1 dh=0 dw=1 c0=0 c1=14\n"), ("add", "%2 = shift %1 dh=1 dw=0 c0=0 c1=14\n")])
def test_relu_stops_infinite_gradients(blend, shift):
    """Where the input is not positive, relu's adjoint is zero whatever arrives: an infinite gradient, and one that overflows in the product."""
    import math

    import torch

    from paper_2304_07741_amd import harness
    from paper_2304_07741_amd import workloads as wl

    k = 2 if shift else 1
    r = harness.DagRunner(wl.HEADER + f"%1 = unary %0 op=relu\n{shift}%{k + 1} = binary %0 %{k} op={blend}\noutput %{k + 1}\n", (2, 14, 16, 24), "bf16")
    x = torch.full(r.x.shape, -1.0, device="cuda")
    x[0, :, 3, 5], x[1, :, 7, 20] = -3e38, 2.0
    dy = torch.full((2, 14, 16, 24), 2.0, device="cuda")
    dy[:, :, 9, 9] = math.inf
    r.x.copy_(x)
    r.dy.copy_(dy.view(r.dy.shape))
    r.forward()
    r.backward()
    xr = r.x.float().requires_grad_(True)
    t = torch.relu(xr)
    if "dw=1" in shift:
        t = torch.nn.functional.pad(t, (0, 1))[..., 1:]
    elif shift:
        t = torch.nn.functional.pad(t, (0, 0, 0, 1))[:, :, 1:]
    (xr * t if blend == "mul" else xr + t).backward(dy)
    got, want = r.dx.float().view(xr.shape), xr.grad
    assert torch.equal(got.isnan(), want.isnan()) and torch.equal(got.isinf(), want.isinf())
    ok = want.isfinite()
    assert (got[ok] - want[ok]).abs().max().item() <= 2.0 ** -8 * want[ok].abs().max().item()   # (one rounding to bf16)
    r.close()
