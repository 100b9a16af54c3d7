"""Softmax over channels in kernels of its own: one and many wavefronts per pixel tile, a last one with fewer channels, 8 and 16 channels per thread, one to
four pixels, planes that end inside a tile; between other units in fp32, its gradient added to another one's; more channels than the
kernels take; infinities and the type's lowest values."""
import math

import pytest

from helpers import check_against_oracle
from test_gpu_parity import _mk
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

SOFTMAX = "%1 = softmax %0 axis=C\noutput %1\n"


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("shape", [(1, 1, 5, 7), (2, 8, 4, 4), (3, 9, 9, 7), (2, 100, 13, 11), (2, 129, 6, 10), (1, 256, 7, 7), (1, 257, 6, 6), (130, 12, 32, 32), (520, 17, 9, 10)],
                         ids=lambda s: "x".join(map(str, s)))
def test_alone(oracle, shape, dtype):
    from paper_2304_07741_amd import harness

    case = _mk(SOFTMAX, shape, dtype, 1100, [], "softmax_c")
    res, r, dy = harness.run_case(case)
    check_against_oracle(oracle, case, res, dy)
    r.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("body", [
    "%1 = fc %0 groups=1 out=40\n%2 = softmax %1 axis=C\n%3 = fc %2 groups=1 out=24\noutput %3\n",
    "%1 = fc %0 groups=1 out=24\n%2 = softmax %1 axis=C\n%3 = unfold %2 kh=3 kw=3\n%4 = fold %3 op=sum\n%5 = binary %1 %4 op=mul\noutput %5\n",
    "%1 = softmax %0 axis=C\n%2 = fc %1 groups=2 out=24\n%3 = binary %1 %2 op=add\noutput %3\n",
])
def test_between_units(oracle, body, dtype):
    from paper_2304_07741_amd import harness

    shape = (3, 24, 12, 10)
    ws = [(1, 40, 24), (1, 24, 40)] if "out=40" in body else [(2, 12, 12)] if "groups=2" in body else [(1, 24, 24)]
    case = wl._case("softmax_mid", wl.HEADER + body, shape, dtype, 1110, ws, [1.0 / math.sqrt(w[2]) for w in ws])
    res, r, dy = harness.run_case(case)
    check_against_oracle(oracle, case, res, dy)
    r.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("ops", [["relu"], ["gelu"], ["abs", "gelu"], ["gelu", "relu"], ["sin"], ["abs", "abs", "gelu"]], ids="_".join)
def test_behind_unaries(oracle, ops, dtype):
    from paper_2304_07741_amd import harness

    body = "".join(f"%{k + 1} = unary %{k} op={op}\n" for k, op in enumerate(ops)) + f"%{len(ops) + 1} = softmax %{len(ops)} axis=C\noutput %{len(ops) + 1}\n"
    for shape in [(2, 37, 12, 10), (130, 12, 16, 33), (1, 140, 5, 6)]:
        case = _mk(body, shape, dtype, 1120, [], "softmax_unary")
        res, r, dy = harness.run_case(case)
        check_against_oracle(oracle, case, res, dy)
        r.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_infinities(dtype):
    import torch

    from paper_2304_07741_amd import harness

    r = harness.DagRunner(wl.HEADER + SOFTMAX, (2, 40, 6, 8), dtype)
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    x = torch.randn(r.x.shape, generator=g, device="cuda") * 4
    x[:, :16] = -math.inf                        # whole threads without a finite value
    x[0, :, 0] = torch.finfo(r.tdtype).min       # every channel the lowest value
    x[1, 39, 2] = torch.finfo(r.tdtype).max / 2
    x[1, :, 4] = -math.inf                       # no finite channel: not a number
    r.x.copy_(x)
    r.dy.copy_(torch.randn(r.dy.shape, generator=g, device="cuda"))
    r.forward()
    r.backward()
    xr = r.x.double().requires_grad_(True)
    y = torch.softmax(xr, dim=1).view(r.y.shape)
    y.backward(r.dy.double())
    tol = 1e-5 if dtype == "f32" else 1e-2       # (a rounding to the type is 6e-8 or 4e-3 of a value that is 1 at most)
    for got, want in ((r.y.double(), y.detach()), (r.dx.double().view(xr.shape), xr.grad)):
        assert torch.equal(got.isnan(), want.isnan())
        assert (got - want).nan_to_num().abs().max().item() <= tol * max(1.0, want.nan_to_num().abs().max().item())
    r.close()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_relu_in_front_stops_infinite_gradients(dtype):
    """An infinite gradient leaves no number behind the softmax of its pixel, and zero behind relu where the input is negative."""
    import torch

    from paper_2304_07741_amd import harness

    r = harness.DagRunner(wl.HEADER + "%1 = unary %0 op=relu\n%2 = softmax %1 axis=C\noutput %2\n", (2, 40, 6, 8), dtype)
    g = torch.Generator(device="cuda").manual_seed(7)
    r.x.copy_(torch.randn(r.x.shape, generator=g, device="cuda"))
    r.dy.copy_(torch.randn(r.dy.shape, generator=g, device="cuda"))
    r.dy.view(2, 40, 6, 8)[1, 17, 2, 3] = math.inf
    r.forward()
    r.backward()
    xr = r.x.double().requires_grad_(True)
    torch.softmax(torch.relu(xr), dim=1).backward(r.dy.double().view(xr.shape))
    got, want = r.dx.double().view(xr.shape), xr.grad
    assert torch.equal(got.isfinite(), want.isfinite())
    assert (got - want)[want.isfinite()].abs().max().item() <= (1e-6 if dtype == "f32" else 1e-2) * want[want.isfinite()].abs().max().item()
    r.close()
