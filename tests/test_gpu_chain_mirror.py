"""Fused chains, backward: gradients through a window that the source pixel fetches itself (lanes and positions change places),
and softmaxes over channels whose values stay in registers from pass to pass; on planes that most windows leave, with images
smaller than a window, every blend on either side of the window, and neighbours of those forms that must keep the hand-over."""
import pytest

from test_gpu_parity import _mk, check_against_oracle

pytestmark = pytest.mark.gpu

BODIES = [
    # product with the pixel's own value on either side of it, sum and avg
    "%1 = unfold %0 kh=5 kw=5\n%2 = binary %0 %1 op=mul\n%3 = fold %2 op=avg\noutput %3\n",
    "%1 = unary %0 op=gelu\n%2 = unfold %1 kh=3 kw=3\n%3 = binary %0 %2 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
    # add and sub, a unary on the window's lanes, one behind the blend
    "%1 = unfold %0 kh=3 kw=3\n%2 = binary %0 %1 op=sub\n%3 = unary %2 op=gelu\n%4 = fold %3 op=sum\noutput %4\n",
    "%1 = unary %0 op=abs\n%2 = unfold %1 kh=1 kw=3\n%3 = binary %0 %2 op=add\n%4 = unary %3 op=sin\n%5 = fold %4 op=avg\noutput %5\n",
    "%1 = unfold %0 kh=3 kw=1\n%2 = unary %1 op=expclip lo=-1 hi=1\n%3 = binary %0 %2 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
    # min and max with the pixel's own value
    "%1 = unfold %0 kh=3 kw=3\n%2 = binary %0 %1 op=max\n%3 = fold %2 op=sum\noutput %3\n",
    "%1 = unary %0 op=sin\n%2 = unfold %1 kh=3 kw=3\n%3 = binary %0 %2 op=min\n%4 = fold %3 op=avg\noutput %4\n",
    # lanes of the window against each other
    "%1 = unfold %0 kh=3 kw=3\n%2 = unary %1 op=gelu\n%3 = binary %1 %2 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
    # values of all taps (softmax, first maximum, a fold's result used on): the hand-over stays
    "%1 = unfold %0 kh=3 kw=3\n%2 = softmax %1 axis=T\n%3 = binary %0 %2 op=mul\n%4 = fold %3 op=max\noutput %4\n",
    "%1 = unfold %0 kh=3 kw=3\n%2 = fold %1 op=avg\n%3 = binary %0 %2 op=mul\noutput %3\n",
    "%1 = unfold %0 kh=3 kw=3\n%2 = binary %0 %1 op=mul\n%3 = fold %2 op=sum\n%4 = unary %3 op=gelu\noutput %4\n",
    # shifted before the window
    "%1 = shift %0 dh=1 dw=-1 c0=0 c1=5\n%2 = unfold %1 kh=3 kw=3\n%3 = binary %0 %2 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
]
SHAPES = [(2, 10, 9, 7), (3, 16, 8, 16), (1, 33, 3, 2), (5, 8, 32, 32)]


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("idx", range(len(BODIES)))
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_gradients_through_windows(oracle, idx, shape, dtype):
    from paper_2304_07741_amd import harness

    case = _mk(BODIES[idx], shape, dtype, 900 + idx, [], f"mirror{idx}")
    res, r, dy = harness.run_case(case)
    assert "chain_bwd" in [d["name"] for d in r.launches(1)]
    check_against_oracle(oracle, case, res, dy)
    r.close()


SOFTMAX = ["%1 = softmax %0 axis=C\noutput %1\n",
           "%1 = unary %0 op=abs\n%2 = softmax %1 axis=C\n%3 = binary %0 %2 op=mul\noutput %3\n",
           "%1 = softmax %0 axis=C\n%2 = unary %1 op=gelu\n%3 = softmax %2 axis=C\noutput %3\n",
           "%1 = shift %0 dh=0 dw=1 c0=0 c1=9\n%2 = softmax %1 axis=C\noutput %2\n"]


@pytest.mark.parametrize("shape", [(2, 96, 32, 32), (3, 16, 9, 7), (2, 17, 8, 8), (1, 128, 5, 13), (2, 200, 4, 4), (2, 64, 16, 32)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("idx", range(len(SOFTMAX)))
def test_softmax_over_channels(oracle, idx, shape):
    from paper_2304_07741_amd import harness

    case = _mk(SOFTMAX[idx], shape, "bf16", 950 + idx, [], f"one_trip{idx}")
    res, r, dy = harness.run_case(case)
    check_against_oracle(oracle, case, res, dy)
    r.close()


PRODUCTS = ["%1 = unfold %0 kh=3 kw=3\n%2 = unary %1 op=abs\n%3 = binary %1 %2 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
            "%1 = unfold %0 kh=5 kw=5\n%2 = binary %1 %1 op=mul\n%3 = fold %2 op=avg\noutput %3\n",
            "%1 = unfold %0 kh=3 kw=3\n%2 = binary %0 %1 op=mul\n%3 = binary %1 %2 op=mul\n%4 = fold %3 op=sum\noutput %4\n",
            "%1 = unfold %0 kh=5 kw=5\n%2 = binary %0 %1 op=mul\n%3 = binary %1 %2 op=mul\n%4 = fold %3 op=avg\noutput %4\n"]


@pytest.mark.parametrize("shape", [(2, 10, 9, 7), (3, 16, 8, 16), (1, 33, 3, 2)], ids=lambda s: "x".join(map(str, s)))
@pytest.mark.parametrize("idx", range(len(PRODUCTS)))
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_infinities_at_the_border(oracle, idx, shape, dtype):
    """Consumers outside the image do not exist: an infinite pixel at the border gets what those inside hand back, and no 0 * infinity
    from the others.  All values positive: nothing cancels."""
    import numpy as np

    from paper_2304_07741_amd import harness, workloads as wl

    case = _mk(PRODUCTS[idx], shape, dtype, 930 + idx, [], f"mirror_inf{idx}")
    x = np.abs(case["x"]) + np.float32(0.5)
    x[0, 0, 0, 0], x[-1, 1, -1, -1], x[0, 3, shape[2] // 2, 0] = np.inf, np.inf, np.inf
    case["x"] = x
    dy = np.abs(wl.make_dy(case, shape)) + np.float32(0.5)
    res, r, _ = harness.run_case(case, dy=dy)
    assert "chain_bwd" in [d["name"] for d in r.launches(1)]
    r.close()
    ref = oracle.run(case["blob"], x, [], dy)
    assert not np.isnan(ref["dx"]).any() and np.isinf(ref["dx"]).any()
    for k in ("y", "dx"):
        got, want = res[k], ref[k].reshape(res[k].shape)
        assert np.array_equal(np.isposinf(got), np.isposinf(want)) and np.array_equal(np.isnan(got), np.isnan(want)), k
        ok = np.isfinite(want)
        assert np.abs(got[ok] - want[ok]).max() <= (1e-5 if dtype == "f32" else 2e-2) * np.abs(want[ok]).max(), k
