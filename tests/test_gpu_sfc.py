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

# Path of the unfold: "-" there is none, "in_lds" the FC reads the window from its operand tile, "stored" the unfolded
# tensor is materialised.  An operand tile holds at most 1024 positions for 64 pixels, margin included, and is a wide one
# (an instance of its own) beyond 512: 5 rows of 200 columns under a 3 x 3 window need (2 + 2*2) * 202 = 1212.
CASES = [
    ("one_element", "-", FC.format(g=1, o=1), (1, 1, 1, 1)),
    ("pooled_size", "-", FC.format(g=2, o=6), (70, 10, 1, 1)),
    ("1x1_remainders", "-", FC.format(g=1, o=70), (3, 37, 5, 13)),
    ("1x1_groups", "-", FC.format(g=5, o=85), (2, 15, 9, 11)),
    ("1x1_long_k", "-", FC.format(g=1, o=33), (2, 300, 7, 7)),
    ("1x1_big_tiles", "-", FC.format(g=1, o=64), (64, 64, 33, 31)),
    ("3x3_tiny", "in_lds", WIN.format(kh=3, kw=3, g=1, o=1), (1, 1, 1, 1)),
    ("3x3_few_pixels", "in_lds", WIN.format(kh=3, kw=3, g=1, o=17), (5, 9, 2, 3)),
    ("3x3_images_per_tile", "in_lds", WIN.format(kh=3, kw=3, g=3, o=39), (7, 15, 7, 7)),
    ("3x3_many_blocks", "in_lds", WIN.format(kh=3, kw=3, g=1, o=65), (40, 20, 28, 29)),
    ("3x3_200_columns", "stored", WIN.format(kh=3, kw=3, g=1, o=20), (2, 6, 5, 200)),
    ("3x3_too_wide", "stored", WIN.format(kh=3, kw=3, g=1, o=4), (1, 3, 3, 700)),
    ("5x5", "in_lds", WIN.format(kh=5, kw=5, g=2, o=40), (3, 12, 11, 9)),
    ("7x7_90_columns", "stored", WIN.format(kh=7, kw=7, g=1, o=50), (2, 5, 6, 90)),
    ("1x3", "in_lds", WIN.format(kh=1, kw=3, g=1, o=24), (4, 21, 6, 17)),
    ("3x1", "in_lds", WIN.format(kh=3, kw=1, g=1, o=24), (4, 21, 17, 6)),
    ("9x1_materialised", "stored", WIN.format(kh=9, kw=1, g=1, o=9), (3, 7, 8, 9)),
    ("fan_out", "in_lds", FAN.format(g=2, o=10), (3, 10, 9, 14)),
    # wide operand tiles, several chunks of four channels, each number of wavefronts across the outputs (Og to 16, to 32, beyond)
    ("3x3_wide_o7", "in_lds", WIN.format(kh=3, kw=3, g=1, o=7), (3, 9, 5, 120)),
    ("3x3_wide_o20", "in_lds", WIN.format(kh=3, kw=3, g=1, o=20), (2, 6, 5, 120)),
    ("3x3_wide_o40", "in_lds", WIN.format(kh=3, kw=3, g=1, o=40), (3, 9, 5, 120)),
    ("3x3_widest", "in_lds", WIN.format(kh=3, kw=3, g=1, o=20), (2, 9, 5, 168)),
    ("3x3_just_too_wide", "stored", WIN.format(kh=3, kw=3, g=1, o=20), (2, 9, 5, 169)),
    ("5x5_wide_o10", "in_lds", WIN.format(kh=5, kw=5, g=1, o=10), (2, 5, 56, 56)),
    ("7x7_wide_o20", "in_lds", WIN.format(kh=7, kw=7, g=1, o=20), (2, 9, 20, 56)),
    ("7x7_wide_o50", "in_lds", WIN.format(kh=7, kw=7, g=1, o=50), (2, 5, 20, 56)),
    # at least 512 tiles of 128 pixels (65536 pixels and groups), the tile of ordinary training: Og to 16 and to 32, ragged
    # channels and pixels, planes below, just above and well above 128 pixels
    ("1x1_128_pixels_o9", "-", FC.format(g=8, o=72), (9, 280, 31, 33)),
    ("1x1_128_pixels_o20_small_planes", "-", FC.format(g=8, o=160), (100, 280, 9, 11)),
    ("1x1_128_pixels_o12_planes_of_130", "-", FC.format(g=8, o=96), (70, 280, 10, 13)),
    ("3x3_128_pixels_o16", "in_lds", WIN.format(kh=3, kw=3, g=8, o=128), (8, 40, 33, 32)),
    ("3x3_128_pixels_o24", "in_lds", WIN.format(kh=3, kw=3, g=8, o=192), (9, 24, 31, 33)),
    ("3x3_128_pixels_o16_small_planes", "in_lds", WIN.format(kh=3, kw=3, g=8, o=128), (100, 40, 9, 11)),
    ("3x3_128_pixels_o20_planes_of_130", "in_lds", WIN.format(kh=3, kw=3, g=8, o=160), (70, 40, 10, 13)),
    ("5x5_128_pixels_o3", "in_lds", WIN.format(kh=5, kw=5, g=8, o=24), (9, 16, 31, 33)),
    # few rows and outputs per group: one thread per pixel (four where the plane is a multiple of four pixels); groups that end
    # inside a workgroup, planes below and above a workgroup's pixels, one to four outputs per thread and a remainder
    ("narrow_1x1_1_1", "-", FC.format(g=7, o=7), (5, 7, 6, 9)),
    ("narrow_1x1_1_1_one_pixel", "-", FC.format(g=300, o=300), (3, 300, 1, 1)),
    ("narrow_1x1_2_5", "-", FC.format(g=9, o=45), (3, 18, 7, 7)),
    ("narrow_1x1_8_16", "-", FC.format(g=3, o=48), (2, 24, 20, 60)),
    ("narrow_1x1_16_2", "-", FC.format(g=2, o=4), (3, 32, 33, 31)),
    ("narrow_1x1_17_1_beside_tiles", "-", FC.format(g=2, o=2), (3, 34, 9, 8)),
    ("narrow_3x3_1_1", "in_lds", WIN.format(kh=3, kw=3, g=70, o=70), (10, 70, 7, 7)),
    ("narrow_3x3_1_8", "in_lds", WIN.format(kh=3, kw=3, g=9, o=72), (4, 9, 31, 33)),
    ("narrow_3x3_2_3", "in_lds", WIN.format(kh=3, kw=3, g=21, o=63), (4, 42, 20, 22)),
    ("narrow_3x3_one_column", "in_lds", WIN.format(kh=3, kw=3, g=64, o=64), (70, 64, 9, 1)),
    ("narrow_5x5_1_3", "in_lds", WIN.format(kh=5, kw=5, g=33, o=99), (2, 33, 24, 22)),
    ("narrow_7x7_1_1", "in_lds", WIN.format(kh=7, kw=7, g=37, o=37), (3, 37, 17, 19)),
    ("narrow_1x3_1_1", "in_lds", WIN.format(kh=1, kw=3, g=64, o=64), (5, 64, 11, 10)),
    ("narrow_3x1_1_4", "in_lds", WIN.format(kh=3, kw=1, g=32, o=128), (5, 32, 15, 16)),
    ("narrow_9x1_stored", "stored", WIN.format(kh=9, kw=1, g=12, o=12), (3, 12, 18, 9)),
    ("narrow_fan_out", "in_lds", FAN.format(g=8, o=8), (70, 8, 21, 24)),
]
# cases whose launches (forward, weight gradient, data gradient) are expected on the vector unit; one letter each
NARROW = {"one_element": "fwd", "pooled_size": "fwd", "1x1_groups": "w", "5x5_128_pixels_o3": "w",
          "narrow_1x1_1_1": "fwd", "narrow_1x1_1_1_one_pixel": "fwd", "narrow_1x1_2_5": "fwd",
          "narrow_1x1_8_16": "f", "narrow_1x1_16_2": "fwd", "narrow_1x1_17_1_beside_tiles": "w", "narrow_3x3_1_1": "fwd",
          "narrow_3x3_1_8": "fw", "narrow_3x3_2_3": "fw", "narrow_3x3_one_column": "fwd", "narrow_5x5_1_3": "fw",
          "narrow_7x7_1_1": "fwd", "narrow_1x3_1_1": "fwd", "narrow_3x1_1_4": "fw", "narrow_9x1_stored": "fwd", "narrow_fan_out": None}


def check_path(name, path, blob, shape, fwd, bwd):
    """The launch lists (names) fit the path that a case is written for."""
    if NARROW.get(name, "") is not None:
        narrow = "".join(l for l, names, what in [("f", fwd, "sfc_fwd"), ("w", bwd, "sfc_wgrad"), ("d", bwd, "sfc_dgrad")]
                         if any(n.startswith(what) and n.endswith("_narrow") for n in names))
        assert narrow == NARROW.get(name, ""), narrow
    slices_wanted = shape[0] * shape[2] * shape[3] > (1024 if any("wgrad" in n and "narrow" in n for n in bwd) else 64)
    fwd, bwd = ([n.replace("_narrow", "") for n in names] for names in (fwd, bwd))
    fans = blob.count("= fc ")
    sfc = lambda names, what: [n for n in names if n.startswith("sfc_" + what)]
    if path == "in_lds":
        direct = blob.count("= fc %0")  # (FCs that read x itself, beside those behind the window)
        for names, what in [(fwd, "fwd"), (bwd, "wgrad"), (bwd, "dgrad")]:
            got = sfc(names, what)
            assert got.count(f"sfc_{what}_unfold") == fans - direct and got.count(f"sfc_{what}") == direct, (names, what)
        assert not any("node_unfold" in n for n in fwd + bwd), (fwd, bwd)
    else:
        assert sfc(fwd, "") == ["sfc_fwd"] * fans and sorted(sfc(bwd, "")) == ["sfc_dgrad"] * fans + ["sfc_wgrad"] * fans, (fwd, bwd)
        assert any("node_unfold" in n or n.startswith("chain") for n in fwd) == (path == "stored"), fwd
    # the weight gradient of more than one step (64 pixels, on the vector unit 1024) is split into slices, as long as they fit
    # the partials' budget
    assert ("wgrad_reduce" in bwd) == slices_wanted, bwd


@pytest.mark.parametrize("name,path,blob,shape", CASES, ids=[c[0] for c in CASES])
def test_fp32_fc(name, path, blob, shape):
    from paper_2304_07741_amd import binding as B

    h = B.canvas_dag_compile(blob, shape, B.CANVAS_F32)
    info = B.canvas_dag_query(h)
    wsh = [tuple(int(v) for v in info.weight_shape[k]) for k in range(info.n_weights)]
    B.canvas_dag_destroy(h)
    rng = np.random.default_rng(len(name))
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    case = {"blob": blob, "shape": shape, "dtype": "f32", "x": f(*shape), "weights": [f(*s) / np.sqrt(s[2]) for s in wsh], "seed": 1}
    res, r, dy = harness.run_case(case)
    check_path(name, path, blob, shape, *[[d["name"] for d in r.launches(b)] for b in (0, 1)])
    ref = canvas_oracle.run(blob, case["x"], case["weights"], dy)
    # A sum of K fp32 terms in any order is off by at most about K * 2^-24 of the sum of their magnitudes, in practice by
    # sqrt(K) * 2^-24: below 1e-5 of the largest element up to K = 2.8e4 (the longest here, 7e4 pixels, in slices).
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
