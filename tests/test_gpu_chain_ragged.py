"""Fused chains on planes that no thread's pixels divide (the last thread of a plane has fewer): the FC-free bodies and random
micro-DAGs against the oracle, widths around 2, 4, 8 and 16 pixels, a plane of one row, one pixel more or less than a tile."""
import math
import re

import numpy as np
import pytest

from helpers import check_against_oracle
from paper_2304_07741_amd import workloads as wl

pytestmark = pytest.mark.gpu

PLANES = [(1, 37), (7, 3), (5, 9), (13, 17), (23, 29), (9, 57), (33, 31), (11, 18)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("H,W", PLANES)
@pytest.mark.parametrize("body", sorted(wl.CHAIN_BODIES))
def test_chain_bodies(oracle, body, H, W, dtype):
    from paper_2304_07741_amd import harness

    case = wl._case(f"ragged_{body}", wl.HEADER + wl.CHAIN_BODIES[body].format(C=24, half=12), (3, 24, H, W), dtype, 31, [], [])
    res, r, dy = harness.run_case(case)
    assert [d["name"] for d in r.launches(0)] == ["chain_fwd"]
    check_against_oracle(oracle, case, res, dy)
    r.close()


@pytest.mark.parametrize("H,W", PLANES)
def test_random_dags(oracle, H, W):
    from paper_2304_07741_amd import harness

    for seed in range(100 + 40 * (H % 5), 100 + 40 * (H % 5) + 16):
        blob, wshapes = wl.fuzz_dag(seed, 0, 16)
        # (a tap softmax that is summed again is a constant: its gradient is rounding noise on both sides)
        if any(f"fold %{k} op={op}" in blob for k in re.findall(r"%(\d+) = softmax %\d+ axis=T", blob) for op in ("sum", "avg")):
            continue
        case = wl._case(f"ragged_seed{seed}", blob, (2, 16, H, W), "bf16", seed, wshapes, [1.0 / math.sqrt(s[2]) for s in wshapes])
        ref = oracle.run(case["blob"], case["x"], case["weights"])
        if not np.isfinite(ref["y"]).all():
            continue
        res, r, dy = harness.run_case(case)
        try:
            check_against_oracle(oracle, case, res, dy, what=f"seed {seed} {H}x{W}\n{blob}")
        finally:
            r.close()
