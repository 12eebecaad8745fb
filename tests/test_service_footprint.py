"""The device footprint of a solve-service request covers every buffer of its
solve (host side of libhmc; no GPU needed)."""
import os

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1212_0785_amd", "libhmc.so")
pytestmark = pytest.mark.skipif(not os.path.exists(LIB), reason="libhmc.so not built")


def ceil_div(a, b):
    return -(-a // b)


@pytest.mark.parametrize("prec", range(4))
@pytest.mark.parametrize("L", [(2, 2, 2, 2), (4, 4, 4, 6), (10, 6, 14, 6), (16, 16, 16, 32), (32, 32, 32, 64)])
def test_request_bytes_hold_every_buffer(L, prec):
    """Partials: |r|^2 and |q|^2 one per 64 sites; the update's |r|^2 one per
    block of 256 sites or, below 2^15 of them, of 64, a multiple of eight and 2048
    at most; the norms two per 256 sites."""
    from paper_1212_0785_amd import hmc as H
    Vh = L[0] * L[1] * L[2] * L[3] // 2
    half = {0: 192, 1: 96, 2: 52, 3: 48}
    link = {0: 144, 1: 72, 2: 36, 3: 36}
    norms = min(ceil_div(Vh, 256), 2048)
    update = min(8 * ceil_div(Vh * (1 if Vh >= 1 << 15 else 4), 8 * 256), 2048)
    buffers = [8 * Vh * 144, 2 * 192 * Vh, 2 * 192 * Vh] + 5 * [192 * Vh]  # links; b, x; r, rhs, q, s, t
    buffers += [192 * Vh] if prec == 0 else [8 * Vh * link[prec]] + 5 * [half[prec] * Vh] + [96 * Vh]
    buffers += [8 * n for n in 3 * [ceil_div(Vh, 64)] + [update, 2 * norms]]
    want = sum(ceil_div(n, 256) * 256 for n in buffers)
    assert H.hmc_request_bytes(H.solve_request(L, 0.15, 1, 0.3), prec) == want
