"""The kernel that bfp_gemm_ws takes for a product (bfp_gemm_ws_route), on the
host: a workspace without room for the parts' sums gives the tile of bfp_gemm."""
from __future__ import annotations

import ctypes
import random

import pytest

from paper_2110_15456_amd import _lib


def size(fn, m_a, m_b, M, N, K, g, use, packed):
    nb = ctypes.c_size_t(0)
    assert fn(m_a, m_b, M, N, K, g, *use, packed, ctypes.byref(nb)) == 0
    return nb.value


def route(m_a, m_b, M, N, K, g, room, use=None, packed=0):
    """(tile, parts, rows, cols) with `room` bytes of workspace; None: its full size."""
    lib = _lib.load()
    use = use or (m_a, m_b)
    if room is None:
        room = size(lib.bfp_gemm_ws_full_size, m_a, m_b, M, N, K, g, use, packed)
    out = [ctypes.c_int(-9) for _ in range(4)]
    assert lib.bfp_gemm_ws_route(m_a, m_b, M, N, K, g, *use, packed, room, *map(ctypes.byref, out)) == 0
    return tuple(x.value for x in out)


def least(m_a, m_b, M, N, K, g, use=None, packed=0):
    return size(_lib.load().bfp_gemm_ws_size, m_a, m_b, M, N, K, g, use or (m_a, m_b), packed)


def gemm_tile(m_a, m_b, M, N, g):
    """The tile that the header documents for bfp_gemm (bfp_gemm_tiled) where an
    operand takes at most 4 bits; 0 for the other formats."""
    if g != 16 or max(m_a, m_b) > 4:
        return 0

    def tiles(bm, bn):
        return -(-M // bm) * -(-N // bn)

    if N <= 64:
        return 3
    if m_a <= 2:
        return 1 if tiles(256, 128) >= 192 else 3
    if N > 128 and tiles(256, 256) >= 192:
        return 0
    return 4 if tiles(128, 128) >= 192 else 3


# A product whose plan is K in parts, on the tile that K in one run is slowest on.
@pytest.mark.parametrize("m_a,m_b,M,N,K", [(4, 4, 2304, 256, 50176), (4, 4, 1024, 4096, 16384),
                                           (4, 4, 4096, 1024, 65536), (2, 2, 576, 64, 802816)])
def test_least_workspace_takes_the_unsplit_tile(m_a, m_b, M, N, K):
    assert route(m_a, m_b, M, N, K, 16, None)[1] > 1
    full = size(_lib.load().bfp_gemm_ws_full_size, m_a, m_b, M, N, K, 16, (m_a, m_b), 0)
    for room in (0, 256, full - 256):
        assert route(m_a, m_b, M, N, K, 16, room) == (gemm_tile(m_a, m_b, M, N, 16), 1, 0, 0)


def test_least_workspace_over_drawn_products():
    rng = random.Random(5)
    split = 0
    for _ in range(4000):
        M, N = (round(2 ** rng.uniform(0, 13)) for _ in range(2))
        K = 64 * round(2 ** rng.uniform(0, 13))
        g, m_a, m_b = rng.choice((4, 8, 16, 16, 16, 32, 64)), rng.randint(1, 8), rng.randint(1, 8)
        packed = int(g == 16 and rng.random() < 0.2)
        use = rng.randint(1, m_a), rng.randint(1, m_b)
        planned = route(m_a, m_b, M, N, K, g, None, use, packed)
        small = route(m_a, m_b, M, N, K, g, least(m_a, m_b, M, N, K, g, use, packed), use, packed)
        if planned[1] == 1:
            assert small == planned
            continue
        split += 1
        assert small[1] == 1 and small[2:] == (0, 0)
        if use == (m_a, m_b):  # (a width below the stored one may leave one plane of codes)
            assert small[0] == gemm_tile(m_a, m_b, M, N, 16 if g <= 16 else 32)
    assert split > 100


MAX_Y = 65535  # blocks in a grid's y


@pytest.mark.parametrize("m_a,m_b", [(4, 4), (2, 2), (6, 6)])
def test_row_tiles_fit_the_grid(m_a, m_b):
    """Tall, narrow products: the few-output kernel's row tiles are its grid's y."""
    few = 0
    for rows in (16, 32, 64):
        for M in (1000, MAX_Y * rows, MAX_Y * rows + 1, 2 * MAX_Y * rows, 1 << 23, 1 << 25):
            for N in (1, 4, 16):
                for K in (16, 64, 1024):
                    r = route(m_a, m_b, M, N, K, 16, None)
                    if r[0] < 0:
                        few += 1
                        assert -(-M // r[2]) <= MAX_Y, (M, N, K, r)
    assert few > 0


# Many outputs, short K: rounds upon rounds of the few-output kernel's workgroups.
@pytest.mark.parametrize("m_a,m_b,M,N,K", [(2, 4, 23517, 896, 64), (2, 4, 2366, 13536, 64), (2, 4, 50589, 320, 64),
                                           (4, 2, 64994, 384, 16), (4, 8, 62361, 512, 64), (8, 8, 22816, 1360, 64)])
def test_many_outputs_stay_on_the_tiled_kernel(m_a, m_b, M, N, K):
    assert route(m_a, m_b, M, N, K, 16, None)[0] >= 0


# Mixed codes with a short K: not on the largest tile.
@pytest.mark.parametrize("M,N,K", [(27797, 704, 256), (6855, 2368, 192), (57242, 384, 192), (3004, 6944, 384)])
def test_mixed_codes_on_a_smaller_tile(M, N, K):
    assert route(2, 4, M, N, K, 16, None)[0] in (1, 3, 4)


def test_route_arguments():
    lib = _lib.load()
    out = [ctypes.byref(ctypes.c_int(0)) for _ in range(4)]

    def call(m=4, M=8, N=8, K=64, g=16, room=0, o=out):
        return lib.bfp_gemm_ws_route(m, m, M, N, K, g, m, m, 0, room, *o)

    assert call() == 0
    assert call(M=0) == 1 and call(o=[None] + out[1:]) == 1
    assert call(g=8) == 1 and call(g=8, room=1 << 20) == 0  # a workspace below the least one
    assert call(K=40) == 2 and call(m=9) == 4
