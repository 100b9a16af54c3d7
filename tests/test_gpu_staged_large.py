"""FC kernels that stage their source through LDS on batches of more than 2^16 pixel tiles, where the product of a workgroup's number and the tile count
passes 2^32: every image against the same images in batches of a few hundred, the first and the last ones against the oracle."""
import math

import pytest

from helpers import TOL, assert_close
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("images", [1405, 2364])   # the FC without a window; the windowed one (8 groups of 8) too
def test_many_pixel_tiles(oracle, images):
    import torch

    from paper_2304_07741_amd import harness

    if torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 24 GB of free device memory")
    blob = wl.blob_sampled(64)
    r = harness.DagRunner(blob, (images, 64, 56, 56), "bf16")
    assert r.info.fused == 1
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    for n in range(0, images, 64):
        for t in (r.x, r.dy):
            t[n:n + 64].copy_(torch.randn(t[n:n + 64].shape, generator=g, device="cuda"))
    for w in r.w:
        w.copy_(torch.randn(w.shape, generator=g, device="cuda") * math.sqrt(2.0 / w.shape[2]))
    r.poison_outputs()
    r.forward()
    r.backward()

    step = 300
    for n in range(0, images, step):
        part = harness.DagRunner(blob, (min(step, images - n), 64, 56, 56), "bf16")
        part.x.copy_(r.x[n:n + step])
        part.dy.copy_(r.dy[n:n + step])
        for a, b in zip(part.w, r.w):
            a.copy_(b)
        part.forward()
        part.backward()
        for whole, small in ((r.y, part.y), (r.dx, part.dx)):
            d = (whole[n:n + step].float() - small.float()).abs().max().item()
            assert d <= TOL["bf16"] * small.float().abs().max().item(), (n, d)   # (NaN, where nothing was stored, fails too)
        part.close()
    for n in (0, images - 2):
        ref = oracle.run(blob, r.x[n:n + 2].float().cpu().numpy(), [w.float().cpu().numpy() for w in r.w], r.dy[n:n + 2, :, 0].float().cpu().numpy())
        assert_close(r.y[n:n + 2, :, 0].float().cpu().numpy(), ref["y"], TOL["bf16"], f"y of images {n}..")
        assert_close(r.dx[n:n + 2].float().cpu().numpy(), ref["dx"], TOL["bf16"], f"dx of images {n}..")
    r.close()
    torch.cuda.empty_cache()
