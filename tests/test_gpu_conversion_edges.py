"""Block edges of the column quantizer (8 unit rows x 64 columns per block) and
of the dequantizer (256 or 1024 quads per block), bit-exact against the oracle."""
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
    """64 and 65 units of 64 values: whole blocks' quads, and one unit more."""
    for rows in (1, 64, 65, 129):
        for m in (2, 4, 6, 8):
            announce("dequantize blocks g=%d rows=%d m=%d" % (g, rows, m))
            x = synth.draw("normal", (rows, 64), 900 + rows)
            t = fb.quantize(torch.from_numpy(x).cuda(), g=g, m=m)
            q, E, _ = oracle.quantize(x, g=g, m=m, threads=THREADS)
            out = torch.full((rows, 64), float("nan"), device="cuda")
            assert np.array_equal(fb.dequantize(t, out=out).cpu().numpy(), oracle.dequantize(q, E, g, m))


def test_dequantize_many():
    """2^20 quads and a few more: four per lane, the last block not whole."""
    rows = 65537
    x = synth.draw("grads", (rows, 64), 950)
    xt = torch.from_numpy(x).cuda()
    for m in (2, 4, 6, 8):
        announce("dequantize %d x 64 m=%d" % (rows, m))
        t = fb.quantize(xt, g=16, m=m)
        q, E, _ = oracle.quantize(x, g=16, m=m, threads=THREADS)
        assert np.array_equal(fb.dequantize(t).cpu().numpy(), oracle.dequantize(q, E, 16, m))
        p = fb.quantize_packed(xt, m=m)
        assert torch.equal(fb.dequantize_packed(p), fb.dequantize(fb.repack(p)))


@pytest.mark.parametrize("m", range(1, 9))
@pytest.mark.parametrize("g", [4, 8, 16, 64])
def test_whole_word_repacks(g, m):
    """The repacks that move whole words of codes (packed storage at g = 16,
    groups of 4 and 8; groups of 64 in bfp_gemm_ws) at every width: the
    repacked tensor stands for the same values, and the product's terms are the
    general kernel's."""
    for rows, length in ((1, 64), (17, 192), (130, 64 * 17)):
        announce("whole-word repack g=%d m=%d %dx%d" % (g, m, rows, length))
        x = synth.draw("grads", (rows, length), 1000 + rows)
        x[0, :16] = 0.0
        xt = torch.from_numpy(x).cuda()
        t = fb.quantize_packed(xt, m=m, rounding="stochastic", seed=5) if g == 16 else fb.quantize(xt, g=g, m=m)
        want = (fb.dequantize_packed(t) if g == 16 else fb.dequantize(t)).cpu().numpy()
        got = fb.dequantize(fb.repack(t)).cpu().numpy()
        if g < 16:  # a group's values, then zeros
            got = got.reshape(rows, length // g, 16)
            assert not got[:, :, g:].any()
            got = got[:, :, :g].reshape(rows, length)
        assert np.array_equal(got.view(np.uint32) & 0x7FFFFFFF, want.view(np.uint32) & 0x7FFFFFFF)
        assert np.array_equal(got, want)
        f = fb.gemm_packed if g == 16 else fb.gemm
        for use in {m, m - 2 if m in (5, 6) else m - 4 if m > 6 else m}:
            C, D = f(t, t, use, use), f(t, t, use, use, workspace=False)
            assert float((C - D).abs().max()) <= 2e-6 * float(D.abs().max())
