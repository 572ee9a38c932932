"""Every tile of the few-output kernel, and the tiled kernel in one run over K at
the shapes that the default call gives to the few-output kernel, against the
oracle (|C_gpu - C_oracle| <= 1e-6 * sum_G |T_G|).  The kernel that a shape is
meant for is asserted (bfp_gemm_ws_route), so that a change of the plan shows."""
from __future__ import annotations

import itertools

import numpy as np
import pytest
import torch

import oracle
import paper_2110_15456_amd as fb
from paper_2110_15456_amd import _lib
from gpu_util import announce, chunk_drops, THREADS
from test_gemm_route import route
from test_gpu_gemm_plan import MODES, TOL, against_oracle, full_size, make

pytestmark = pytest.mark.gpu

WIDTHS = (2, 4, 6, 8)
# Rows and columns one past, one short of and between tile edges; K of whole and
# of ragged supersteps (256 values) and K slabs (128).
SHAPES = sorted(((M, N, K) for M in (1, 17, 33, 49, 65, 100, 130) for N in (40, 97, 161, 530, 1000, 2050, 4090)
                 for K in (96, 512, 1120, 2048, 4640)), key=lambda s: s[0] * s[1] * s[2])


def guarded(A, B, m_a, m_b, extra, full=True):
    """bfp_gemm_ws into rows `extra` longer than N; the words behind them must stay."""
    M, N = A.rows, B.rows
    out = torch.full((M + 1, N + extra), float("nan"), device="cuda")
    need = full_size(A, B) if full else 0
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device="cuda")
    st = _lib.load().bfp_gemm_ws(A.mant.data_ptr(), A.exp.data_ptr(), A.m, B.mant.data_ptr(), B.exp.data_ptr(), B.m, M,
                                 N, A.len, A.g, m_a, m_b, 0, out.data_ptr(), N + extra, ws.data_ptr() if need else None,
                                 need, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert bool(out[:M, N:].isnan().all()) and bool(out[M].isnan().all())
    return out[:M, :N].contiguous()


def shapes_of(tile, m_a, m_b, g, use, columns=1):
    """The smallest shape on that tile with whole and with ragged supersteps."""
    found = []
    for ragged in (False, True):
        s = next((s for s in SHAPES if s[1] % columns == 0 and bool(s[2] % 256) == ragged and s[0] > tile[0] // 2 and
                  s[2] % g == 0 and route(m_a, m_b, *s, g, None, use)[2:] == tile), None)
        if s:
            found.append(s)
    assert found, (tile, m_a, m_b, g, use)
    return found


@pytest.mark.parametrize("g", [16, 32])
@pytest.mark.parametrize("tile", [(16, 16), (32, 32), (64, 32)])
def test_few_output_tiles(tile, g):
    for m_a, m_b in itertools.product(WIDTHS, WIDTHS):
        for u_a, u_b in itertools.product(chunk_drops(m_a), chunk_drops(m_b)):
            for M, N, K in shapes_of(tile, m_a, m_b, g, (u_a, u_b)):
                announce("tile %s %dx%dx%d g=%d (%d,%d) at (%d,%d)" % (tile, M, N, K, g, m_a, m_b, u_a, u_b))
                A, B, oa, ob = make(M, N, K, g, m_a, m_b, 7600 + M + 8 * m_a + m_b)
                C = fb.gemm(A, B, u_a, u_b)
                against_oracle(C, A, B, oa, ob, u_a, u_b)
                for extra in (3, 4):  # rows that are and are not whole 16-byte pieces
                    assert torch.equal(guarded(A, B, u_a, u_b, extra, full=False), C)


@pytest.mark.parametrize("tile", [(16, 16), (32, 32), (64, 32)])
def test_few_output_tiles_converted(tile):
    shapes = {}
    for m_a, m_b in itertools.product(WIDTHS, WIDTHS):
        s = next((M, N, K) for M in (33, 49, 100, 130) for N in (48, 528, 1008, 2064, 4080) for K in (1120, 2048, 4640)
                 if route(m_a, m_b, M, N, K, 16, None)[2:] == tile)
        shapes[m_a, m_b] = s
    for (m_a, m_b), (M, N, K) in shapes.items():
        A, B, _, _ = make(M, N, K, 16, m_a, m_b, 7700 + M)
        C = fb.gemm(A, B)
        for c_m, mode in itertools.product((1, 2, 4, 6, 8), MODES):
            announce("tile %s converted %dx%dx%d (%d,%d) -> %d %s" % (tile, M, N, K, m_a, m_b, c_m, mode))
            T, R = fb.gemm_bfp(A, B, c_m, rounding=mode, seed=31), fb.quantize(C, g=16, m=c_m, rounding=mode, seed=31)
            assert torch.equal(T.exp, R.exp) and torch.equal(T.mant, R.mant)


@pytest.mark.parametrize("shape", [(300, 270, 16384), (272, 259, 65536), (260, 64, 32768)])
def test_parts_leave_what_is_behind_a_row(shape):
    M, N, K = shape
    for m in (4, 6):
        assert route(m, m, M, N, K, 16, None)[1] > 1
        announce("parts, long rows %dx%dx%d m=%d" % (M, N, K, m))
        A, B, _, _ = make(M, N, K, 16, m, m, 7800 + M)
        C = fb.gemm(A, B)
        for extra in (1, 4):
            assert torch.equal(guarded(A, B, m, m, extra), C)


# One operand format of every kernel variant (one plane of FP4 or FP6 codes, split
# at 2 bits, split at 4 bits).
PAIRS = [(2, 2), (2, 4), (4, 2), (4, 4), (1, 5), (2, 8), (4, 6), (3, 7), (5, 2), (6, 3), (8, 1), (7, 4), (6, 6), (6, 8),
         (8, 6), (8, 8)]


def check_tiled(M, N, K, g, m_a, m_b, seed):
    A, B, oa, ob = make(M, N, K, g, m_a, m_b, seed)
    against_oracle(fb.gemm(A, B, workspace=False), A, B, oa, ob, m_a, m_b)


@pytest.mark.parametrize("g", [16, 32])
@pytest.mark.parametrize("shape", [(300, 270, 576), (257, 129, 608), (129, 257, 160), (1, 1, 32), (5, 300, 4096),
                                   (520, 390, 1056)])
def test_tiled_ragged_shapes(shape, g):
    """Several tiles with ragged tails in every direction, K with and without
    whole slabs."""
    for m_a, m_b in PAIRS:
        announce("tiled %s g=%d (%d,%d)" % (shape, g, m_a, m_b))
        check_tiled(*shape, g, m_a, m_b, 7900 + shape[0] + m_a)


@pytest.mark.parametrize("g", [16, 32])
@pytest.mark.parametrize("nslabs", range(1, 10))
def test_tiled_slab_counts(nslabs, g):
    """K = 128 nslabs: every tail of the slab loops, unrolled by four."""
    for m_a, m_b in PAIRS:
        announce("tiled, %d slabs g=%d (%d,%d)" % (nslabs, g, m_a, m_b))
        check_tiled(260, 136, 128 * nslabs, g, m_a, m_b, 8000 + nslabs)


# C's rows of whole lines (past the caches), of whole 16-byte pieces only (through
# them) and of neither, with waves inside N and across its end.
@pytest.mark.parametrize("N", [256, 260, 264, 270, 288, 520])
def test_rows_of_c(N):
    for m_a, m_b in ((4, 4), (2, 2), (2, 4), (6, 6), (6, 4), (8, 8)):
        announce("rows of C, N=%d (%d,%d)" % (N, m_a, m_b))
        check_tiled(300, N, 256, 16, m_a, m_b, 8100 + N)
