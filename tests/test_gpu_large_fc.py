"""fp32 FC on tensors of more than 2^31 elements (8 GB) and of more than 2^32, where a launch with one row of workgroups would
pass 2^32 threads: a thread takes one element where the plane is no multiple of four pixels.  One product per element, so y
and dx are exact; dW is a sum of products of +-1, +-0.5 (exact in fp64, and in fp32 as long as no partial sum needs more than
24 bits; sums of 2^32 random signs stay below 2^19)."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("images,side,gigabytes", [(65, 5760, 48), (131, 5727, 96)], ids=["2_31_elements", "2_32_elements"])
def test_one_output_per_group(images, side, gigabytes):
    import torch

    from paper_2304_07741_amd import binding as B
    from paper_2304_07741_amd import harness

    blob = "canvas-dag 1\n%1 = fc %0 groups=1 out=1\noutput %1\n"
    shape = (images, 1, side, side)   # 2 156 544 000 and 4 296 607 299 elements
    assert images * side * side > (2**31 if side % 2 == 0 else 2**32)
    if torch.cuda.mem_get_info()[0] < gigabytes << 30:
        pytest.skip(f"needs {gigabytes} GB of free device memory")
    r = harness.DagRunner(blob, shape, "f32")
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    signs = torch.randint(0, 2, (2, side * side), generator=g, device="cuda", dtype=torch.int8)
    for n in range(shape[0]):  # (image n: the random signs turned by n pixels)
        r.x[n].copy_((signs[0].roll(n) * 2 - 1).reshape(1, side, side))
        r.dy[n].copy_((signs[1].roll(3 * n) - 0.5).reshape(1, side, side))
    r.w[0].fill_(1.5)
    r.y.zero_()
    r.dx.zero_()
    r.forward()
    r.backward()
    dw = 0.0
    for n in range(shape[0]):
        assert torch.equal(r.y[n].reshape(-1), r.x[n].reshape(-1) * 1.5), n
        assert torch.equal(r.dx[n].reshape(-1), r.dy[n].reshape(-1) * 1.5), n
        dw += float((r.x[n].double() * r.dy[n].reshape(r.x[n].shape).double()).sum())
    assert abs(float(r.dw[0].reshape(-1)[0]) - dw) <= 1e-6 * max(abs(dw), 1.0) + 1.0, (float(r.dw[0].reshape(-1)[0]), dw)
    r.close()
    del r
    torch.cuda.empty_cache()
