"""Block edges of the column quantizer (8 unit rows x 64 columns per block) and
of the dequantizer (1024 quads per block), bit-exact against the oracle."""
from __future__ import annotations

import numpy as np
import pytest
import torch

import oracle
import paper_2110_15456_amd as fb
from paper_2110_15456_amd import synth
from gpu_util import announce, check_quantize, THREADS

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("g", [4, 8, 16, 32, 64])
@pytest.mark.parametrize("units", [1, 7, 8, 9, 17])
def test_column_blocks(g, units):
    unit = max(g, 16)
    for cols in (1, 63, 65):
        for m in (2, 4, 6, 8):
            announce("column blocks g=%d %d units x %d columns m=%d" % (g, units, cols, m))
            x = synth.draw("grads", (units * unit, cols), 800 + units + cols)
            t, q, E = check_quantize(x, 0, g, m, "stochastic" if m == 4 else "nearest", seed=3)
            y = fb.dequantize(t).cpu().numpy()
            assert np.array_equal(y, oracle.dequantize(q, E, g, m))


@pytest.mark.parametrize("g", [4, 16, 64])
def test_dequantize_blocks(g):
    """64 and 65 units of 64 values: one block's quads, and one unit more."""
    for rows in (1, 64, 65, 129):
        for m in (2, 4, 6, 8):
            announce("dequantize blocks g=%d rows=%d m=%d" % (g, rows, m))
            x = synth.draw("normal", (rows, 64), 900 + rows)
            t = fb.quantize(torch.from_numpy(x).cuda(), g=g, m=m)
            q, E, _ = oracle.quantize(x, g=g, m=m, threads=THREADS)
            out = torch.full((rows, 64), float("nan"), device="cuda")
            assert np.array_equal(fb.dequantize(t, out=out).cpu().numpy(), oracle.dequantize(q, E, g, m))
