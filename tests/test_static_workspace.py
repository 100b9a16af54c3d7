"""Plans of the whole-DAG families whose workspace is the larger for the partial sums of their weight gradients: a forward call has no use for those, so
they do not keep a plan from the library's static workspace."""
import pytest

from paper_2304_07741_amd import binding as B
from paper_2304_07741_amd import workloads as wl

# (64 to 66 MB without the partial sums' last slices, 64 to 70 MB with them)
PLANS = [
    ("sampled", (36, 256, 21, 34)), ("sampled", (32, 504, 28, 14)), ("sampled", (100, 256, 16, 16)), ("sampled", (46, 504, 16, 16)),
    ("sampled", (512, 248, 7, 7)), ("sampled", (10, 368, 40, 40)), ("sampled", (55, 440, 44, 6)), ("involution", (172, 384, 14, 14)),
]


def _blob(family, C):
    return wl.blob_sampled(C) if family == "sampled" else wl.blob_involution(C, 3)


@pytest.mark.parametrize("flags", [0, B.CANVAS_OPT_INFERENCE])
@pytest.mark.parametrize("family,shape", PLANS)
def test_partial_sums_do_not_count(family, shape, flags):
    B.load()
    h = B.canvas_dag_compile(_blob(family, shape[1]), shape, B.CANVAS_BF16, flags)
    assert B.canvas_dag_query(h).workspace_bytes > B.CANVAS_STATIC_WORKSPACE_BYTES
    # (null pointers: BAD_ARG on a GPU, HIP_ERROR without one; the size is looked at first)
    assert B.load().canvas_dag_forward_static(h, None, None, None, None) in (-4, -7)
    B.canvas_dag_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("family,shape", [PLANS[0], PLANS[4], PLANS[7]])
def test_forward_beside_the_partial_sums(family, shape):
    import torch

    from paper_2304_07741_amd import harness

    r = harness.DagRunner(_blob(family, shape[1]), shape, "bf16")
    r.x.normal_(generator=torch.Generator(device="cuda").manual_seed(3))
    for w in r.w:
        w.normal_(std=0.1)
    r.forward()
    want = r.y.clone()
    r.poison_outputs()
    B.canvas_dag_forward_static(r.handle, r.x, r.w, r.y)
    assert torch.isfinite(want.float()).all() and torch.equal(r.y, want)
    r.close()
