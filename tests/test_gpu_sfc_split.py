"""fp32 FCs on the bf16 matrix units (operands cut into three parts) at the edges of their tiles: remainders in channels,
outputs, pixels and images, groups, wide images, accumulated gradients, results that overlap an input, and values that the
parts cannot hold."""
import numpy as np
import pytest

from oracle import canvas_oracle
from paper_2304_07741_amd import binding as B
from paper_2304_07741_amd import harness

pytestmark = pytest.mark.gpu

FC = "canvas-dag 1\n%1 = fc %0 groups={g} out={o}\noutput %1\n"
WIN = "canvas-dag 1\n%1 = unfold %0 kh=3 kw=3\n%2 = fc %1 groups={g} out={o}\noutput %2\n"
FAN = ("canvas-dag 1\n%1 = unfold %0 kh=3 kw=3\n%2 = fc %1 groups=1 out={o}\n%3 = fc %1 groups=1 out={o}\n"
       "%4 = binary %2 %3 op=mul\noutput %4\n")

CASES = [
    ("3x3_four_pixels", WIN.format(g=1, o=64), (1, 64, 2, 2)),
    ("3x3_few_pixels", WIN.format(g=1, o=65), (3, 64, 2, 3)),
    ("3x3_ragged_channels", WIN.format(g=1, o=71), (2, 69, 9, 7)),
    ("3x3_images_per_tile", WIN.format(g=1, o=64), (23, 66, 3, 5)),
    ("3x3_groups_of_32", WIN.format(g=4, o=128), (9, 128, 28, 25)),
    ("3x3_two_rows_of_outputs", WIN.format(g=1, o=129), (2, 65, 11, 13)),
    ("3x3_three_items", WIN.format(g=1, o=64), (2, 64, 10, 50)),
    ("3x3_four_items", WIN.format(g=1, o=64), (2, 64, 10, 60)),
    ("3x3_one_column", WIN.format(g=1, o=64), (2, 64, 70, 1)),
    ("1x1_ragged", FC.format(g=1, o=131), (70, 133, 11, 13)),
    ("1x1_groups", FC.format(g=2, o=260), (35, 256, 14, 15)),
    ("fan_out", FAN.format(o=64), (3, 64, 9, 14)),
]


def _case(name, blob, shape):
    h = B.canvas_dag_compile(blob, shape, B.CANVAS_F32)
    info = B.canvas_dag_query(h)
    names = [B.canvas_dag_launch_desc(h, 0, i)["name"] for i in range(info.n_launches_fwd)]
    wsh = [tuple(int(v) for v in info.weight_shape[k]) for k in range(info.n_weights)]
    B.canvas_dag_destroy(h)
    assert names[0] == "weight_prep", names
    rng = np.random.default_rng(len(name))
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    return {"blob": blob, "shape": shape, "dtype": "f32", "x": f(*shape), "weights": [f(*s) / np.sqrt(s[2]) for s in wsh], "seed": 1}


def _check(case, res, dy):
    # (K terms in any order: about sqrt(K) * 2^-24 of the largest element, K up to 2.8e4 here)
    ref = canvas_oracle.run(case["blob"], case["x"], case["weights"], dy)
    for n, a, b in [("y", res["y"], ref["y"]), ("dx", res["dx"], ref["dx"])] + [(f"dw{k}", a, b) for k, (a, b) in enumerate(zip(res["dw"], ref["dw"]))]:
        err = np.abs(a.reshape(b.shape) - b).max() / max(np.abs(b).max(), 1e-30)
        assert np.isfinite(a).all() and err <= 1e-5, (n, err)
        # In norm the parts' products are as good as fp32 sums, 5e-8 to 1.3e-7; without the products of a third part it is 4e-6.
        norm = np.linalg.norm(a.reshape(b.shape) - b) / np.linalg.norm(b)
        print(f"[{n}] {norm:.1e}")
        assert norm <= 5e-7, (n, norm)


@pytest.mark.parametrize("name,blob,shape", CASES, ids=[c[0] for c in CASES])
def test_split_fc(name, blob, shape):
    case = _case(name, blob, shape)
    res, r, dy = harness.run_case(case)
    r.ws.fill_(0xFF)  # (a second pass on a workspace of NaN: nothing is read before it is written)
    r.poison_outputs()
    r.forward()
    r.backward()
    again = r.results()
    r.close()
    for a, b in zip([res["y"], res["dx"], *res["dw"]], [again["y"], again["dx"], *again["dw"]]):
        assert np.array_equal(a, b)
    _check(case, res, dy)


def test_values_that_the_parts_cannot_hold():
    """Infinities, NaN and magnitudes that round to an infinity in bf16 give what fp32 gives, in their windows and nowhere else."""
    case = _case("3x3_values", WIN.format(g=1, o=64), (2, 64, 9, 11))
    x, w = case["x"], case["weights"][0]
    x[0, 3, 4, 5], x[0, 9, 0, 0], x[1, 63, 8, 10], x[1, 7, 4, 1] = np.inf, -np.inf, np.nan, 3.4e38
    x[1, 30, 4, 6] = -3.39e38
    w.reshape(64, 64, 9)[:, 7] *= 1e-3
    w.reshape(64, 64, 9)[:, 30] *= 1e-3
    res, r, dy = harness.run_case(case)
    r.close()
    xp = np.pad(x.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
    with np.errstate(invalid="ignore"):
        ref = sum(np.einsum("oc,nchw->nohw", w.reshape(64, 64, 3, 3)[:, :, i, j].astype(np.float64), xp[:, :, i:i + 9, j:j + 11], optimize=False)
                  for i in range(3) for j in range(3))
    got = res["y"].reshape(ref.shape)
    # (einsum multiplies an infinity into every output of its pixel; elsewhere in a window it meets real weights too)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isposinf(got), np.isposinf(ref)) and np.array_equal(np.isneginf(got), np.isneginf(ref))
    ok = np.isfinite(ref)
    small = ok & (np.abs(ref) < 1e6)
    assert small.sum() > 0.5 * ref.size and np.abs(got[small] - ref[small]).max() <= 1e-5 * np.abs(ref[small]).max()
    big = ok & (np.abs(ref) > 1e30)
    assert big.any() and (np.abs(got[big] - ref[big]) <= 1e-5 * np.abs(ref[big])).all()


@pytest.mark.parametrize("what", ["x", "w"])
def test_result_on_top_of_an_input(what):
    import torch

    case = _case("3x3_overlap", WIN.format(g=1, o=64), (2, 64, 12, 12))
    r = harness.DagRunner(case["blob"], case["shape"], "f32")
    dy = np.random.default_rng(3).standard_normal(r.out_shape).astype(np.float32)
    r.load(case["x"], case["weights"], dy)
    n = r.y.numel()
    if what == "x":
        y = r.x.view(-1).view(r.y.shape)
        B.canvas_dag_forward(r.handle, r.x, r.w, y, r.ws)
    else:
        buf = torch.empty(max(n, r.w[0].numel()), dtype=torch.float32, device="cuda")
        w = buf[:r.w[0].numel()].view(r.w[0].shape)
        w.copy_(r.w[0])
        y = buf[:n].view(r.y.shape)
        B.canvas_dag_forward(r.handle, r.x, [w], y, r.ws)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    r.close()
    ref = canvas_oracle.run(case["blob"], case["x"], case["weights"], dy.reshape(2, 64, 12, 12))["y"]
    assert np.abs(got.reshape(ref.shape) - ref).max() <= 1e-5 * np.abs(ref).max()


@pytest.mark.parametrize("shape,o,groups", [((1, 32, 1, 9), 33, 1), ((3, 40, 7, 7), 32, 1), ((40, 64, 13, 17), 97, 1), ((9, 192, 11, 6), 192, 4)])
def test_weight_gradient(shape, o, groups):
    """Weight gradients of one slice and of many, ragged tiles of outputs and channels; an infinity, a NaN and a value whose bf16 is
    infinite reach exactly the weights whose products meet them."""
    import torch

    N, C, H, W = shape
    r = harness.DagRunner(WIN.format(g=groups, o=o), shape, "f32")
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    for t in [r.x, r.dy, *r.w]:
        t.copy_(torch.randn(t.shape, generator=g, device="cuda"))
    for extreme in [False, True]:
        if extreme:
            r.x[0, 3, 0, 0], r.x[N - 1, C - 1, H - 1, W - 1], r.x[0, 20, 0, W // 2] = float("inf"), float("nan"), 3.4e38
            r.dy.view(N, o, H, W)[0, 1, 0, 1] = -float("inf")
            r.dy.mul_(0.25)  # (3.4e38 times dy is finite)
        r.poison_outputs()
        r.ws.fill_(0xFF)
        r.forward()
        r.backward()
        got = r.dw[0].cpu().double().reshape(o, C // groups, 3, 3)
        xp = torch.nn.functional.pad(r.x.cpu().double(), (1, 1, 1, 1))
        dy = r.dy.cpu().double().view(N, o, H, W)
        og, cg = o // groups, C // groups
        ref = torch.empty_like(got)
        for k in range(groups):
            d = dy[:, k * og:(k + 1) * og].transpose(0, 1).reshape(og, -1)
            for i in range(3):
                for j in range(3):
                    v = xp[:, k * cg:(k + 1) * cg, i:i + H, j:j + W]
                    ref[k * og:(k + 1) * og, :, i, j] = d @ v.transpose(0, 1).reshape(cg, -1).T  # (the margin's zeros are multiplied)
        if not extreme:
            # (N*H*W terms of unit variance: some 2^-24 of the sum's root mean square per hundred of them, in any order)
            assert (got - ref).norm() <= 1e-6 * ref.norm()
            continue
        finite = torch.isfinite(ref) & (ref.abs() < 3e38)
        assert torch.equal(torch.isnan(got), torch.isnan(ref)) and not torch.isfinite(got[torch.isinf(ref)]).any()
        err = (got - ref).abs()[finite]
        assert (err <= 1e-5 * ref.abs()[finite].clamp_min(float(N * H * W) ** 0.5)).all()
        assert torch.isfinite(got).any() and not torch.isfinite(got).all()
    r.close()


@pytest.mark.parametrize("shape,o,groups", [((2, 64, 7, 9), 96, 1), ((3, 128, 5, 6), 128, 2)])
def test_infinite_weights_and_gradients_at_the_border(shape, o, groups):
    """The margin's zeros are multiplied, as in every fp32 FC kernel here: an infinite weight makes NaN of the pixels whose tap lies
    there and infinities of the others (forward; and, on dy, the data gradient), an infinite dy NaN of the taps that leave the image."""
    case = _case("3x3_border", WIN.format(g=groups, o=o), shape)
    N, C, H, W = shape
    og, cg = o // groups, C // groups
    w = case["weights"][0].reshape(o, cg, 3, 3)
    w[5, 2, 0, 0] = np.inf
    dy = np.random.default_rng(11).standard_normal((N, o, H, W)).astype(np.float32)
    dy[0, 1, 0, 1], dy[N - 1, o - 1, H - 1, W - 1] = np.inf, -np.inf
    res, r, _ = harness.run_case(case, dy=dy)
    r.close()

    def windows(t):  # [N, channels, 9, H, W]
        p = np.pad(t.astype(np.float64), ((0, 0), (0, 0), (1, 1), (1, 1)))
        return np.stack([p[:, :, i:i + H, j:j + W] for i in range(3) for j in range(3)], 2)

    ref = {"y": np.empty((N, o, H, W)), "dx": np.empty(shape), "dw": np.empty((o, cg, 3, 3))}
    with np.errstate(invalid="ignore"):
        for k in range(groups):
            so, sc = slice(k * og, (k + 1) * og), slice(k * cg, (k + 1) * cg)
            xw, dw, wk = windows(case["x"][:, sc]), windows(dy[:, so]), w[so].astype(np.float64).reshape(og, cg, 9)
            for n in range(N):
                ref["y"][n, so] = (wk.reshape(og, -1) @ xw[n].reshape(cg * 9, -1)).reshape(og, H, W)
                ref["dx"][n, sc] = (wk[:, :, ::-1].transpose(1, 0, 2).reshape(cg, -1) @ dw[n].reshape(og * 9, -1)).reshape(cg, H, W)
            d = dy[:, so].astype(np.float64).transpose(1, 0, 2, 3).reshape(og, -1)
            ref["dw"][so] = (d @ xw.transpose(0, 3, 4, 1, 2).reshape(-1, cg * 9)).reshape(og, cg, 3, 3)
    for name, got in [("y", res["y"]), ("dx", res["dx"]), ("dw", res["dw"][0])]:
        want = ref[name]
        got = got.reshape(want.shape)
        assert np.array_equal(np.isnan(got), np.isnan(want)) and np.isnan(want).any(), name
        inf, ok = np.isinf(want), np.isfinite(want)
        assert np.array_equal(got[inf], want[inf]) and inf.any(), name
        assert np.abs(got[ok] - want[ok]).max() <= 1e-5 * np.abs(want[ok]).max(), name


def test_a_step_of_nan_is_no_slower_than_a_few_steps():
    """Results computed again go through the fp32 matrix units as tiles: a step in which every result does takes about three times as
    long as one of finite values (two passes, the second at the fp32 rate), and not a time that grows with each result's terms."""
    import torch

    r = harness.DagRunner(WIN.format(g=1, o=64), (16, 64, 28, 28), "f32")
    times = []
    for nan in [False, True]:
        for t in [r.x, r.dy, *r.w]:
            t.normal_()
        if nan:
            r.w[0].fill_(float("nan"))
            r.dy.fill_(float("nan"))
        best = float("inf")
        for _ in range(5):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            for _ in range(3):
                r.forward()
                r.backward()
            ev[1].record()
            torch.cuda.synchronize()
            best = min(best, ev[0].elapsed_time(ev[1]) / 3)
        times.append(best)
        if nan:
            assert torch.isnan(r.y).all() and torch.isnan(r.dx).all() and torch.isnan(r.dw[0]).all()
    r.close()
    print(f"[nan step] finite {times[0] * 1e3:.1f} us, NaN {times[1] * 1e3:.1f} us")
    assert times[1] <= 10 * times[0]


# magnitudes of x, of the weights and of dy: each as small as fp32 goes, against ones and against the inverse; products that are
# subnormal; operands and results beyond what the scaled parts hold
SCALES = [(1e-30, 1, 1), (1e-36, 1, 1), (1e-38, 1, 1e30), (1, 1e-37, 1e-36), (1e-41, 1e38, 1e-30), (1e-20, 1e-20, 1e-10), (1e31, 1e-30, 1e-25), (1e33, 1e-36, 1e-35), (1e20, 1e10, 1e-3)]


@pytest.mark.parametrize("body,shape", [(WIN.format(g=1, o=64), (2, 64, 9, 11)), (FC.format(g=1, o=256), (140, 192, 14, 15))], ids=["3x3", "1x1"])
@pytest.mark.parametrize("scales", SCALES, ids=lambda s: "_".join(f"{v:g}" for v in s))
def test_operands_of_any_magnitude(body, shape, scales):
    """Three bf16 parts hold an fp32 value of any magnitude, subnormal ones among them: the error of fp32 sums (2.5e-7 in norm; K and
    N*H*W terms) plus the rounding of subnormal results, not that of the parts that would be lost."""
    case = _case("magnitudes", body, shape)
    case["x"] *= np.float32(scales[0])
    case["weights"][0] *= np.float32(scales[1])
    N, C, H, W = shape
    o = case["weights"][0].shape[1]
    dy = np.random.default_rng(17).standard_normal((N, o, H, W)).astype(np.float32) * np.float32(scales[2])
    res, r, _ = harness.run_case(case, dy=dy)
    r.close()
    w = case["weights"][0].astype(np.float64).reshape(o, C, -1)
    k = w.shape[2]

    def rows(t):  # [channels * taps, N * H * W]
        t = t.astype(np.float64)
        if k == 9:
            p = np.pad(t, ((0, 0), (0, 0), (1, 1), (1, 1)))
            t = np.stack([p[:, :, i:i + H, j:j + W] for i in range(3) for j in range(3)], 2)
        else:
            t = t[:, :, None]
        return t.transpose(1, 2, 0, 3, 4).reshape(t.shape[1] * k, -1)

    planes = lambda m: m.reshape(-1, N, H, W).transpose(1, 0, 2, 3)
    xr = rows(case["x"])
    ref = {"y": planes(w.reshape(o, -1) @ xr), "dx": planes(w[:, :, ::-1].transpose(1, 0, 2).reshape(C, -1) @ rows(dy)),
           "dw": dy.astype(np.float64).transpose(1, 0, 2, 3).reshape(o, -1) @ xr.T}
    for name, got in [("y", res["y"]), ("dx", res["dx"]), ("dw", res["dw"][0])]:
        want = ref[name]
        got = got.astype(np.float64).reshape(want.shape)
        err, size = np.linalg.norm(got - want), np.linalg.norm(want)
        print(f"[magnitudes {scales} {name}] {err / size:.2e} of {size / want.size ** 0.5:.1e}")
        assert err <= 2.5e-7 * size + 2.0 ** -149 * want.size ** 0.5, name
