"""fp32 FC on tensors of more than 2^31 elements (8 GB): with one output per group a launch with one row of workgroups would
pass 2^32 threads there.  One product per element, so y and dx are exact; dW is a sum of 2^31 products of +-1, +-0.5 (exact
in fp64, and in fp32 as long as no partial sum needs more than 24 bits; sums of 2^31 random signs stay below 2^18)."""
import pytest

pytestmark = pytest.mark.gpu


def test_one_output_per_group_beyond_2_31_elements():
    import torch

    from paper_2304_07741_amd import binding as B
    from paper_2304_07741_amd import harness

    blob = "canvas-dag 1\n%1 = fc %0 groups=1 out=1\noutput %1\n"
    shape = (65, 1, 5760, 5760)   # 2 156 544 000 elements
    assert shape[0] * shape[2] * shape[3] > 2**31
    if torch.cuda.mem_get_info()[0] < 48 << 30:
        pytest.skip("needs 48 GB of free device memory")
    r = harness.DagRunner(blob, shape, "f32")
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    signs = torch.randint(0, 2, (2, 5760 * 5760), generator=g, device="cuda", dtype=torch.int8)
    for n in range(shape[0]):  # (image n: the random signs turned by n pixels)
        r.x[n].copy_((signs[0].roll(n) * 2 - 1).reshape(1, 5760, 5760))
        r.dy[n].copy_((signs[1].roll(3 * n) - 0.5).reshape(1, 5760, 5760))
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
