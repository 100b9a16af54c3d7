"""One fp32 FC, alone or behind an unfold, with y in the place of x and dx in the place of dy: the same bits as with separate
buffers (the launch reads the one and writes the other).  Tensors of many workgroups, buffers that coincide and buffers that
are shifted against each other."""
import pytest

pytestmark = pytest.mark.gpu

FC = "canvas-dag 1\n%1 = fc %0 groups={g} out={o}\noutput %1\n"
WIN = "canvas-dag 1\n%1 = unfold %0 kh={k} kw={k}\n%2 = fc %1 groups={g} out={o}\noutput %2\n"
CASES = [
    (FC.format(g=1, o=64), (32, 64, 28, 28)),
    (FC.format(g=64, o=64), (32, 64, 28, 28)),
    (FC.format(g=4, o=24), (16, 40, 27, 29)),
    (WIN.format(k=3, g=1, o=64), (32, 64, 28, 28)),
    (WIN.format(k=3, g=32, o=32), (32, 32, 28, 28)),
    (WIN.format(k=5, g=2, o=24), (16, 16, 27, 29)),
]


@pytest.mark.parametrize("shift", [0, 4, 1024, -4096])
@pytest.mark.parametrize("blob,shape", CASES)
def test_in_place(blob, shape, shift):
    import torch

    from paper_2304_07741_amd import harness

    r = harness.DagRunner(blob, shape, "f32")
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    for t in [r.x, r.dy, *r.w]:
        t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    r.poison_outputs()
    r.forward()
    r.backward()
    y, dx, dw = r.y.clone(), r.dx.clone(), r.dw[0].clone()
    x0, dy0 = r.x.clone(), r.dy.clone()

    def pair(a, b):  # two tensors of these shapes in one buffer, the second `shift` elements behind the first
        lo = max(0, -shift)
        buf = torch.empty(2 * abs(shift) + max(a.numel(), b.numel()) + 16, device="cuda")
        return buf[lo:lo + a.numel()].view(a.shape), buf[lo + shift:lo + shift + b.numel()].view(b.shape)

    for _ in range(3):
        r.x, r.y = pair(x0, y)
        r.x.copy_(x0)
        r.forward()
        assert torch.equal(r.y, y)
        r.x = x0
        r.dy, r.dx = pair(dy0, dx)
        r.dy.copy_(dy0)
        r.backward()
        assert torch.equal(r.dx, dx) and torch.equal(r.dw[0], dw)
    r.close()


def test_static_workspace_with_and_without_an_overlap():
    """68 MB tensors: with room for an overlap the plan would not fit the 64 MB of the static workspace; only a call that has
    one is refused, and nothing of it is launched."""
    import torch

    from paper_2304_07741_amd import binding as B
    from paper_2304_07741_amd import harness

    r = harness.DagRunner(FC.format(g=1, o=16), (340, 16, 56, 56), "f32")
    assert int(r.info.workspace_bytes) > B.CANVAS_STATIC_WORKSPACE_BYTES
    r.x.normal_()
    r.w[0].normal_()
    r.forward()
    want = r.y.clone()
    r.y.zero_()
    B.canvas_dag_forward_static(r.handle, r.x, r.w, r.y)
    assert torch.equal(r.y, want)
    x0 = r.x.clone()
    with pytest.raises(B.CanvasError):
        B.canvas_dag_forward_static(r.handle, r.x, r.w, r.x)
    torch.cuda.synchronize()
    assert torch.equal(r.x, x0)
    r.close()
