"""The routes a product takes from its shape (bfp_gemm_ws): the few-output
kernel and K taken in parts, each against the oracle under the GEMM's tolerance
(|C_gpu - C_oracle| <= 1e-6 * sum_G |T_G|) and beside the tiled kernel in one
run over K, and the converted output against converting the FP32 one."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2110_15456_amd as fb
from paper_2110_15456_amd import _lib, synth
from gpu_util import announce, chunk_drops, THREADS

pytestmark = pytest.mark.gpu
TOL = 1e-6
MODES = ("nearest", "stochastic", "truncate")


def make(M, N, K, g, m_a, m_b, seed):
    a = synth.draw("half_normal", (M, K), seed)
    b = synth.draw("grads", (N, K), seed + 1)
    A, B = (fb.quantize(torch.from_numpy(x).cuda(), g=g, m=m) for x, m in ((a, m_a), (b, m_b)))
    oa, ob = (oracle.quantize(x, g=g, m=m)[:2] for x, m in ((a, m_a), (b, m_b)))
    return A, B, oa, ob


def against_oracle(C, A, B, oa, ob, m_a, m_b):
    Co, S = oracle.gemm(oa[0], oa[1], A.m, ob[0], ob[1], B.m, g=A.g, m_a=m_a, m_b=m_b, threads=THREADS)
    err = np.abs(C.cpu().numpy().astype(np.float64) - Co)
    assert np.all(err <= TOL * S), "max err/sum|T| = %.3g" % float((err / np.maximum(S, 1e-300)).max())


def full_size(A, B):
    nb = ctypes.c_size_t(0)
    assert _lib.load().bfp_gemm_ws_full_size(A.m, B.m, A.rows, B.rows, A.len, A.g, A.m, B.m, 0, ctypes.byref(nb)) == 0
    return nb.value


# edges of the 16 x 16 tile, which the plan takes for all of these (the larger
# ones: test_gpu_gemm_routes.py), odd column counts, one unit of K to ragged
# supersteps (16 units) and more supersteps than waves
@pytest.mark.parametrize("g", [16, 32])
@pytest.mark.parametrize("shape", [(1, 40, 32), (17, 33, 288), (31, 161, 1056), (65, 150, 2592), (3, 65, 4640)])
def test_few_outputs(g, shape):
    M, N, K = shape
    for m_a in (2, 4, 6, 8):
        for m_b in (2, 4, 6, 8):
            A, B, oa, ob = make(M, N, K, g, m_a, m_b, 7000 + M + 8 * m_a + m_b)
            for u_a in chunk_drops(m_a):
                for u_b in chunk_drops(m_b):
                    announce("few outputs %dx%dx%d g=%d stored (%d,%d) at (%d,%d)" % (M, N, K, g, m_a, m_b, u_a, u_b))
                    against_oracle(fb.gemm(A, B, u_a, u_b), A, B, oa, ob, u_a, u_b)
                    against_oracle(fb.gemm(A, B, u_a, u_b, workspace=False), A, B, oa, ob, u_a, u_b)


# K in parts: every plane count, full and ragged slabs, parts of unequal length,
# few and many parts (both orders of the sum), columns not a multiple of 4
@pytest.mark.parametrize("g", [16, 32])
@pytest.mark.parametrize("mm", [(2, 2), (4, 4), (4, 2), (6, 6), (4, 6), (8, 6), (8, 8)])
@pytest.mark.parametrize("shape", [(300, 270, 16384), (300, 270, 16384 + 96), (272, 259, 65536), (520, 1030, 8192)])
def test_parts(g, mm, shape):
    M, N, K = shape
    m_a, m_b = mm
    announce("parts %dx%dx%d g=%d (%d,%d)" % (M, N, K, g, m_a, m_b))
    A, B, oa, ob = make(M, N, K, g, m_a, m_b, 7100 + M + N + m_a * 10 + m_b)
    assert full_size(A, B) > 0 and fb.gemm_ws_size(A, B) == 0
    C = fb.gemm(A, B)
    idx = np.arange(0, M, 7)
    Co, S = oracle.gemm(oa[0], oa[1], m_a, ob[0], ob[1], m_b, g=g, m_a=m_a, m_b=m_b, rows=idx, threads=THREADS)
    err = np.abs(C.cpu().numpy().astype(np.float64)[idx] - Co)
    assert np.all(err <= TOL * S)
    # the same bits on every run
    out = torch.empty((M, N), device="cuda")
    for _ in range(3):
        out.fill_(float("nan"))
        assert torch.equal(fb.gemm(A, B, out=out), C)
    # without the room for the parts' sums: in one run over K
    W = fb.gemm(A, B, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert torch.equal(W, fb.gemm(A, B, workspace=False))


def test_given_workspace_is_left_alone():
    """A tensor given for a product that needs no workspace is not written, however
    large: programs share one among streams."""
    M, N, K = 300, 270, 16384
    for m in (4, 6):
        announce("given workspace %dx%dx%d m=%d" % (M, N, K, m))
        A, B, _, _ = make(M, N, K, 16, m, m, 7200)
        assert fb.gemm_ws_size(A, B) == 0 and full_size(A, B) > 0
        ws = torch.full((full_size(A, B),), 0xA5, dtype=torch.uint8, device="cuda")
        C = fb.gemm(A, B, workspace=ws)
        assert bool((ws == 0xA5).all())
        assert torch.equal(C, fb.gemm(A, B, workspace=False))


def test_without_memory_for_the_parts():
    """Products whose parts' sums find no room on the card run in one run over K."""
    M, N, K = 1024, 4096, 16384
    gen = torch.Generator(device="cuda").manual_seed(3)
    A, B = (fb.quantize(torch.randn((r, K), device="cuda", generator=gen), m=4) for r in (M, N))
    P, Q = (fb.quantize(torch.randn((r, K), device="cuda", generator=gen), g=8, m=4) for r in (M, N // 4))
    assert full_size(A, B) > 60 << 20 and full_size(P, Q) - fb.gemm_ws_size(P, Q) > 15 << 20
    want = fb.gemm(A, B, workspace=False)
    want_rep = fb.gemm(P, Q, workspace=torch.empty(fb.gemm_ws_size(P, Q), dtype=torch.uint8, device="cuda"))
    R = fb.quantize(want, m=4)
    C, D, T = torch.empty_like(want), torch.empty_like(want_rep), fb.BFPTensor.empty(M, N, 16, 4, "cuda")
    room = torch.empty(fb.gemm_ws_size(P, Q), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    held = []
    try:
        announce("no memory for parts %dx%dx%d" % (M, N, K))
        torch.cuda.set_per_process_memory_fraction(
            torch.cuda.memory_reserved() / torch.cuda.get_device_properties(0).total_memory)
        for mib in (64, 16, 4):  # what the allocator still holds free
            with pytest.raises(torch.OutOfMemoryError):
                while len(held) < 1000:
                    held.append(torch.empty(mib << 20, dtype=torch.uint8, device="cuda"))
        fb.gemm(A, B, out=C)
        fb.gemm_bfp(A, B, 4, out=T)
        del room
        fb.gemm(P, Q, out=D)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert torch.equal(C, want) and torch.equal(D, want_rep)
    assert torch.equal(T.mant, R.mant) and torch.equal(T.exp, R.exp)


@pytest.mark.parametrize("mm", [(4, 4), (6, 4), (2, 8)])
@pytest.mark.parametrize("shape", [(33, 80, 1040), (300, 272, 16384), (144, 64, 90112)])
def test_converted_output(mm, shape):
    M, N, K = shape
    A, B, _, _ = make(M, N, K, 16, mm[0], mm[1], 7300 + M)
    C = fb.gemm(A, B)
    for c_m in (2, 4, 6, 8):
        for mode in MODES:
            announce("converted %dx%dx%d (%d,%d) -> %d %s" % (M, N, K, mm[0], mm[1], c_m, mode))
            st = torch.zeros(1, dtype=torch.int32, device="cuda")
            T = fb.gemm_bfp(A, B, c_m, rounding=mode, seed=31, status=st)
            R = fb.quantize(C, g=16, m=c_m, rounding=mode, seed=31)
            assert torch.equal(T.exp, R.exp) and torch.equal(T.mant, R.mant) and int(st.item()) == 0


def close_to_values(C, A, B):
    """At most one rounding per group and chunk pair, of sums bounded by sum |x| |y|."""
    x, y = fb.dequantize(A).double(), fb.dequantize(B).double()
    S = (x[:, None, :] * y[None, :, :]).abs().sum(2)
    err = (C.double() - (x[:, None, :] * y[None, :, :]).sum(2)).abs()
    assert bool((err <= (4 * (A.len // A.g) + 4) * 2.0**-24 * S).all())


# Row tiles of 16, 32 and 64 rows up to the 65535 that the few-output kernel's grid
# holds, and one more, which goes to a taller tile or to the tiled kernel.
@pytest.mark.parametrize("m", [4, 6])
@pytest.mark.parametrize("M", [65535 * 16, 65535 * 16 + 1, 65535 * 32 + 1, 65535 * 64 + 1])
def test_tall_products(M, m):
    gen = torch.Generator(device="cuda").manual_seed(M & 0xFFFF)
    for N, K in ((1, 16), (2, 16), (1, 32)):
        announce("tall %dx%dx%d m=%d" % (M, N, K, m))
        A = fb.quantize(torch.randn((M, K), device="cuda", generator=gen), m=m)
        B = fb.quantize(torch.randn((N, K), device="cuda", generator=gen), m=m)
        close_to_values(fb.gemm(A, B), A, B)


def test_tall_converted_output():
    M, N, K = 65535 * 16 + 1, 16, 16
    gen = torch.Generator(device="cuda").manual_seed(7)
    announce("tall converted %dx%dx%d" % (M, N, K))
    A = fb.quantize(torch.randn((M, K), device="cuda", generator=gen), m=4)
    B = fb.quantize(torch.randn((N, K), device="cuda", generator=gen), m=4)
    T, R = fb.gemm_bfp(A, B, 4, rounding="stochastic", seed=5), fb.quantize(fb.gemm(A, B), m=4, rounding="stochastic",
                                                                            seed=5)
    assert torch.equal(T.exp, R.exp) and torch.equal(T.mant, R.mant)


def test_lowered_and_regrouped_operands():
    """Repacked operands (groups of 8 and 64, a precision between chunk
    boundaries) in parts and on the few-output kernel."""
    for (M, N, K) in ((20, 48, 1024), (260, 200, 32768)):
        for g, m, use in ((8, 4, 4), (64, 4, 4), (16, 4, 2), (16, 6, 3)):
            announce("repacked %dx%dx%d g=%d m=%d at %d" % (M, N, K, g, m, use))
            A, B, oa, ob = make(M, N, K, g, m, m, 7400 + g)
            against_oracle(fb.gemm(A, B, use, use), A, B, oa, ob, use, use)


def test_captured():
    """The routes under graph capture: replays give the eager result."""
    for (M, N, K) in ((16, 256, 2048), (300, 270, 16384)):
        announce("captured %dx%dx%d" % (M, N, K))
        A, B, _, _ = make(M, N, K, 16, 4, 4, 7500)
        want = fb.gemm(A, B).clone()
        out = torch.empty((M, N), device="cuda")
        s = torch.cuda.Stream()
        s.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(s):
            fb.gemm(A, B, out=out)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            fb.gemm(A, B, out=out)
        for _ in range(4):
            out.fill_(float("nan"))
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
