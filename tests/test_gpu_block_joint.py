"""Blocks whose instances run in one launch (shift / grouped FC / unary / residual, groups of 16 channels): sizes at the edges
of a tile (128 pixels, 512 per workgroup, two tiles per wavefront), every activation, one to nine instances (nine run one
after the other), and outputs that overlap an input, which the launch must not take."""
import numpy as np
import pytest

from helpers import TOL, assert_close, has_kinks
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _blob(C, act, res):
    lines = ["%1 = shift %0 dh=1 dw=-1 c0=0 c1=16", f"%2 = fc %1 groups={C // 16} out={C}"]
    if act:
        lines.append(f"%3 = unary %2 op={act}")
    if res:
        lines.append(f"%{len(lines) + 1} = binary %{len(lines)} %0 op=add")
    return wl.HEADER + "\n".join(lines) + f"\noutput %{len(lines)}\n"


# (c_in, c_out, N, H, W, activation, residual)
CASES = [(32, 64, 1, 8, 9, "relu", True), (64, 32, 1, 8, 9, "relu", True), (32, 64, 5, 16, 8, "gelu", True), (64, 32, 5, 16, 8, "gelu", False),
         (16, 128, 3, 24, 24, "abs", True), (128, 16, 3, 24, 24, "abs", True), (16, 48, 9, 8, 17, "expclip lo=-1 hi=1", True),
         (48, 16, 9, 8, 17, "expclip lo=-1 hi=1", False), (32, 64, 2, 8, 65, None, True), (64, 32, 2, 8, 65, None, False),
         (16, 144, 2, 8, 16, "relu", True), (144, 16, 2, 8, 16, "relu", True)]


def _runner(idx):
    from paper_2304_07741_amd import harness

    c_in, c_out, N, H, W, act, res = CASES[idx]
    C = min(c_in, c_out)
    blob = _blob(C, act, res)
    case = wl.block_case(f"joint{idx}", blob, (N, c_in, H, W), c_out, "bf16", 700 + idx, [(C // 16, 16, 16)], [0.25])
    r = harness.BlockRunner(blob, (N, c_in, H, W), c_out, "bf16")
    r.load(case["x"], case["weights"], case["dy"])
    return blob, case, r


def _check(oracle, blob, case, c_out, got):
    bracketed = {}

    def alt(mg, v):
        if (mg, v) not in bracketed:
            bracketed[(mg, v)] = oracle.run_block(blob, case["x"], case["weights"], c_out, case["dy"], tie_margin=v[0] * mg, tie_rule=v[1])
        return bracketed[(mg, v)]

    ref = oracle.run_block(blob, case["x"], case["weights"], c_out, case["dy"])
    kinks = has_kinks(blob)
    floor = 1e-5 * float(np.abs(case["dy"]).max())
    if "y" in got:
        assert_close(got["y"], ref["y"], TOL["bf16"], "y")
    if "dx" in got:
        assert_close(got["dx"], ref["dx"], TOL["bf16"], "dx", (lambda mg, v: alt(mg, v)["dx"]) if kinks else None, floor)
    for j, d in enumerate(got.get("dw", [])):
        assert_close(d[0], ref["dw"][j][0], TOL["bf16"], f"dw{j}", (lambda mg, v, j=j: alt(mg, v)["dw"][j][0]) if kinks else None, floor)


@pytest.mark.parametrize("idx", range(len(CASES)))
def test_instances_in_one_launch(idx):
    from oracle import block_oracle

    blob, case, r = _runner(idx)
    try:
        got, again = r.run(), r.run()
    finally:
        r.close()
    assert np.array_equal(got["y"], again["y"]) and np.array_equal(got["dx"], again["dx"])
    _check(block_oracle, blob, case, CASES[idx][1], got)


@pytest.mark.parametrize("idx", [0, 1])
def test_outputs_that_overlap_an_input(idx):
    """The narrow output on top of the wide input (expand: dx on dy, reduce: y on x): every input is read before the first
    element of the output is written."""
    import torch

    from oracle import block_oracle
    from paper_2304_07741_amd import binding as B

    blob, case, r = _runner(idx)
    try:
        if idx == 0:
            B.canvas_block_forward(r.handle, r.x, r.w, r.y, r.ws)
            over = r.dy.view(-1)[:r.dx.numel()].view(r.dx.shape)
            B.canvas_block_backward(r.handle, r.x, r.w, r.dy, over, r.dw, r.ws)
            torch.cuda.synchronize()
            got = {"dx": over.float().cpu().numpy(), "dw": [[d.cpu().numpy()] for d in r.dw]}
        else:
            over = r.x.view(-1)[:r.y.numel()].view(r.y.shape)
            B.canvas_block_forward(r.handle, r.x, r.w, over, r.ws)
            torch.cuda.synchronize()
            got = {"y": over.float().cpu().numpy()}
    finally:
        r.close()
    _check(block_oracle, blob, case, CASES[idx][1], got)
