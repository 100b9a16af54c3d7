"""The fp32 FC kernels at the edges of their tiles: remainders in channels, outputs, pixels and images, windows of every
kind they take, accumulated gradients, one image row wider than the implicit window takes."""
import numpy as np
import pytest

from oracle import canvas_oracle
from paper_2304_07741_amd import harness
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

FC = "canvas-dag 1\n%1 = fc %0 groups={g} out={o}\noutput %1\n"
WIN = "canvas-dag 1\n%1 = unfold %0 kh={kh} kw={kw}\n%2 = fc %1 groups={g} out={o}\noutput %2\n"
# two FCs read the same unfolded tensor, and x directly: three data gradients add into dx
FAN = ("canvas-dag 1\n%1 = unfold %0 kh=3 kw=3\n%2 = fc %1 groups=1 out={o}\n%3 = fc %1 groups={g} out={o}\n%4 = fc %0 groups=1 out={o}\n"
       "%5 = binary %2 %3 op=mul\n%6 = binary %4 %5 op=add\noutput %6\n")

CASES = [
    ("one_element", FC.format(g=1, o=1), (1, 1, 1, 1)),
    ("pooled_size", FC.format(g=2, o=6), (70, 10, 1, 1)),
    ("1x1_remainders", FC.format(g=1, o=70), (3, 37, 5, 13)),
    ("1x1_groups", FC.format(g=5, o=85), (2, 15, 9, 11)),
    ("1x1_long_k", FC.format(g=1, o=33), (2, 300, 7, 7)),
    ("1x1_big_tiles", FC.format(g=1, o=64), (64, 64, 33, 31)),
    ("3x3_tiny", WIN.format(kh=3, kw=3, g=1, o=1), (1, 1, 1, 1)),
    ("3x3_few_pixels", WIN.format(kh=3, kw=3, g=1, o=17), (5, 9, 2, 3)),
    ("3x3_images_per_tile", WIN.format(kh=3, kw=3, g=3, o=39), (7, 15, 7, 7)),
    ("3x3_many_blocks", WIN.format(kh=3, kw=3, g=1, o=65), (40, 20, 28, 29)),
    ("3x3_wide_tile", WIN.format(kh=3, kw=3, g=1, o=20), (2, 6, 5, 200)),
    ("3x3_too_wide", WIN.format(kh=3, kw=3, g=1, o=4), (1, 3, 3, 700)),
    ("5x5", WIN.format(kh=5, kw=5, g=2, o=40), (3, 12, 11, 9)),
    ("7x7_wide", WIN.format(kh=7, kw=7, g=1, o=50), (2, 5, 6, 90)),
    ("1x3", WIN.format(kh=1, kw=3, g=1, o=24), (4, 21, 6, 17)),
    ("3x1", WIN.format(kh=3, kw=1, g=1, o=24), (4, 21, 17, 6)),
    ("9x1_materialised", WIN.format(kh=9, kw=1, g=1, o=9), (3, 7, 8, 9)),
    ("fan_out", FAN.format(g=2, o=10), (3, 10, 9, 14)),
]


@pytest.mark.parametrize("name,blob,shape", CASES, ids=[c[0] for c in CASES])
def test_fp32_fc(name, blob, shape):
    from paper_2304_07741_amd import binding as B

    h = B.canvas_dag_compile(blob, shape, B.CANVAS_F32)
    info = B.canvas_dag_query(h)
    wsh = [tuple(int(v) for v in info.weight_shape[k]) for k in range(info.n_weights)]
    B.canvas_dag_destroy(h)
    rng = np.random.default_rng(len(name))
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    case = {"blob": blob, "shape": shape, "dtype": "f32", "x": f(*shape), "weights": [f(*s) / np.sqrt(s[2]) for s in wsh], "seed": 1}
    res, r, dy = harness.run_case(case)
    assert any(d["name"].startswith("sfc_") for d in r.launches(0))
    ref = canvas_oracle.run(blob, case["x"], case["weights"], dy)
    # A sum of K fp32 terms in any order is off by at most about K * 2^-24 of the sum of their magnitudes, in practice by
    # sqrt(K) * 2^-24: below 1e-5 of the largest element up to K = 2.8e4 (the longest here, 6.6e4 pixels, in slices).
    for n, a, b in [("y", res["y"], ref["y"]), ("dx", res["dx"], ref["dx"])] + [(f"dw{k}", a, b) for k, (a, b) in enumerate(zip(res["dw"], ref["dw"]))]:
        err = np.abs(a.reshape(b.shape) - b).max() / max(np.abs(b).max(), 1e-30)
        assert np.isfinite(a).all() and err <= 1e-5, (n, err)
    r.close()


def test_rows_of_the_last_channels_do_not_leak():
    """An infinity in one pixel reaches only the outputs whose window holds it, in ragged tiles too."""
    shape = (2, 5, 7, 9)
    blob = WIN.format(kh=3, kw=3, g=1, o=6)
    rng = np.random.default_rng(5)
    x = rng.standard_normal(shape).astype(np.float32)
    x[1, 4, 6, 8] = np.inf
    w = rng.standard_normal((1, 6, 45)).astype(np.float32)
    case = {"blob": blob, "shape": shape, "dtype": "f32", "x": x, "weights": [w], "seed": 1}
    res, r, dy = harness.run_case(case)
    ok = np.ones(shape[2:], bool)
    ok[5:, 7:] = False
    assert np.isfinite(res["y"][0]).all() and np.isfinite(res["y"][1][:, ok]).all() and not np.isfinite(res["y"][1][:, ~ok]).any()
    assert np.isfinite(res["dx"]).all()
    assert np.isfinite(res["dw"][0][..., :36]).all()  # channels 0-3
    r.close()
