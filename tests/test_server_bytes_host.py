"""Device bytes of serving requests (fdwt_server_request_bytes, host only): no
more than the general evaluation and whole 24-byte columns per point make of a
request, so that a budget that admits one keeps admitting it whatever kernels
its net takes."""
import ctypes

import numpy as np
import pytest

from paper_0808_0487_amd import fdwt


def request_bytes(kind, p, m, s, nq):
    C, one, q = np.zeros((s, m, m), dtype=np.uint8), np.ones(s), np.zeros((s, max(nq, 1)), dtype=np.uint32)
    r = fdwt.RequestC(kind, p, m, s, 1, C.ctypes.data, 1, one.ctypes.data, 2.0, one.ctypes.data, nq,
                      q.ctypes.data if nq else None)
    jb, cb = ctypes.c_size_t(), ctypes.c_size_t()
    assert fdwt.lib().fdwt_server_request_bytes(ctypes.byref(r), 0, ctypes.byref(jb), ctypes.byref(cb)) == 0
    return jb.value, cb.value


def slices(*sizes):
    return sum((v + 255) & ~255 for v in sizes)


@pytest.mark.parametrize("p,m,s,nq", [(3, 7, 3, 3510), (2, 9, 1, 5553), (2, 11, 4, 1668), (3, 8, 1, 704), (3, 8, 6, 1497),
                                      (5, 4, 33, 4142), (2, 14, 20, 4096), (7, 6, 10, 20000), (2, 20, 3, 17), (7, 3, 60, 1)])
def test_interpolation(p, m, s, nq):
    """The job's buffers (data, transform, coefficients, queries, results) and
    the largest workspace of its steps, the evaluation's with a partial sum (8
    bytes) per query and point chunk: 2048 workgroups of 256 queries at most,
    whole chunks of 256 points."""
    N = p ** m
    qb = (nq + 255) // 256
    gy = max(1, min((2048 + qb - 1) // qb, (N + 255) // 256))
    ppc = ((N + gy - 1) // gy + 255) // 256 * 256
    gy = (N + ppc - 1) // ppc
    ev = slices(s * 68 * 4, 0 if p == 2 else s * nq * 8, gy * nq * 8)
    spec = 0 if p == 2 else slices(N * 8)
    coef = 0 if p == 2 else slices(N * 8)
    want = slices(4 * N, N * (4 if p == 2 else 8), 4 * N, s * nq * 4, nq * 4, max(ev, spec, coef))
    assert request_bytes(1, p, m, s, nq)[0] <= want


@pytest.mark.parametrize("p,m,s", [(7, 8, 11), (7, 8, 24), (5, 10, 12), (3, 15, 5), (3, 13, 40), (5, 6, 3)])
def test_effective_dimension_columns(p, m, s):
    """Kernel-data columns within the budget (1 GiB here), in whole multiples
    of 24 bytes per point, or a single multiple."""
    N = p ** m
    cols = max(24 * N, min(2 * s * 24 * N, (1 << 30) // (24 * N) * 24 * N))
    rest = slices(4 * N, 8 * N, 8 * N) + 64 * (2 * s + 2) + (1 << 20)  # data, transform, weights, sums
    assert request_bytes(2, p, m, s, 0)[0] <= cols + rest + (2 * s) * (N // p ** 3 + 1) * 8
