"""Which kernels take a chain, as the planner reports it (CANVAS_LOG): the cases of the GPU tests of the streamed windows, of tensors blended with
themselves and of the softmax over channels reach the programs and kernels that they are there for, and their neighbours do not."""
import json
import os
import re
import subprocess
import sys

import pytest

import test_gpu_chain_streamed as streamed
import test_gpu_self_blend as blend
import test_gpu_softmax_c as softmax
from paper_2304_07741_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
BLEND, SOFTMAX = "the kernels of a tensor blended with itself", "the kernels of a softmax over channels"
CODE = """
import json, os, sys
from paper_2304_07741_amd import binding as B
for body, shape, dtype in json.load(sys.stdin):
    os.write(2, b"\\n=== plan\\n")
    B.canvas_dag_destroy(B.canvas_dag_compile(body, shape, B.CANVAS_F32 if dtype == "f32" else B.CANVAS_BF16))
"""


def reports(cases):
    """What the planner says of each (body, shape, dtype)."""
    p = subprocess.run([sys.executable, "-c", CODE], input=json.dumps([(wl.HEADER + b, s, d) for b, s, d in cases]), cwd=ROOT, env=dict(os.environ, CANVAS_LOG="1"),
                       capture_output=True, text=True, check=True)
    out = p.stderr.split("\n=== plan\n")[1:]
    assert len(out) == len(cases)
    return out


def test_streamed_windows():
    """Bodies 0-5, 7 and 8 fold their windows as they load them, with as many pixels per thread as the row allows, 3 and 7 two windows against each other in
    the backward pass; of the others only what a cut leaves of the shifted one."""
    cases = [(b, s, d) for b in streamed.BODIES for s in streamed.SHAPES for d in ("bf16", "f32")]
    for (body, shape, dtype), text in zip(cases, reports(cases)):
        idx = streamed.BODIES.index(body)
        programs = [t for t in text.split("program:")[1:] if " LDFOLD " in t]
        kinds = [int(k) for k in re.findall(r" LDFOLD T=\d+ kind=(\d+)", text)]
        if idx not in (6, 9, 10, 11):
            assert programs, (body, shape, dtype)
        elif idx != 10:
            assert not programs, (body, shape, dtype)
        assert any(k & 0x80 for k in kinds) == (idx in (3, 7)), (body, shape, dtype)
        assert all(f" vec={8 if shape[3] % 8 == 0 else 4} " in t for t in programs), (body, shape, dtype)


def test_blend_with_itself():
    """The first six bodies, whatever the plane; in fp32 none."""
    cases = [(b, s, "bf16") for b in blend.BODIES for s in blend.SHAPES]
    for (body, shape, _), text in zip(cases, reports(cases)):
        assert (BLEND in text) == (blend.BODIES.index(body) < 6), (body, shape)
    assert not any(BLEND in t for t in reports([(b, (2, 14, 16, 24), "f32") for b in blend.BODIES]))


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_softmax_over_channels(dtype):
    """Up to 256 channels; behind up to two of relu, abs and gelu."""
    cases = [(softmax.SOFTMAX, (2, C, 6, 6), dtype) for C in (1, 8, 100, 129, 256, 257)]
    assert [SOFTMAX in t for t in reports(cases)] == [True] * 5 + [False]

    def behind(*ops):
        body = "".join(f"%{k + 1} = unary %{k} op={op}\n" for k, op in enumerate(ops))
        return (body + f"%{len(ops) + 1} = softmax %{len(ops)} axis=C\noutput %{len(ops) + 1}\n", (2, 37, 12, 10), dtype)

    cases = [behind("relu"), behind("abs", "gelu"), behind("gelu", "relu"), behind("sin"), behind("abs", "abs", "gelu")]
    assert [SOFTMAX in t for t in reports(cases)] == [True, True, True, False, False]
