"""Scales of the variance columns that are transformed two to a complex column
(csrc/pair_scale.h, p odd): after scaling, the two columns of a pair have about
the same norm, so that neither takes up much more of the other's rounding than
of its own; and a pair's transform is about as exact as the columns' own."""
import os
import subprocess

import numpy as np
import pytest

from oracle import kernel, net as onet
from paper_0808_0487_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exponents(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("pair") / "pair_scale_check")
    subprocess.run(["g++", "-O2", "-std=c++17", "-I" + os.path.join(ROOT, "paper_0808_0487_amd", "csrc"),
                    os.path.join(ROOT, "tests", "pair_scale_check.cpp"), "-o", exe], check=True)

    def run(p, m, alpha, gam):
        rp = [float(kernel.rprime_closed(p, alpha, t + 1)) for t in range(m)] + [float(kernel.rprime_closed(p, alpha, 0))]
        text = " ".join([str(p), str(m), str(len(gam))] + ["%.17g" % v for v in list(gam) + rp])
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout
        return [int(v) for v in out.split()]
    return run


def columns(p, m, alpha, gam, seed):
    """U_1..U_s, Q_1..Q_s at the net's points, by their definitions."""
    s = len(gam)
    X = onet.net_int(p, m, inputs.upper_triangular_generators(p, m, s, seed))
    U, u = [], np.zeros(p ** m)
    e = [np.ones(p ** m)] + [np.zeros(p ** m) for _ in range(s)]
    for j in range(s):
        i = kernel.first_diff_digit(p, m, X[j], np.zeros_like(X[j]))
        a = gam[j] ** 2 * kernel.rprime_closed(p, alpha, i)
        u = u + a + u * a
        U.append(u)
        for k in range(j + 1, 0, -1):
            e[k] = e[k] + a * e[k - 1]
    return U + e[1:]


CASES = [(3, 8, 10, -2.0, 1.0, 2.0), (3, 8, 21, 0.0, 1.0, 2.0), (3, 6, 17, -0.5, 3.0, 2.0), (3, 1, 3, -2.0, 1.0, 2.0),
         (3, 5, 64, -1.0, 1.0, 1.5), (3, 7, 24, -6.0, 1.0, 3.0), (5, 5, 24, -0.5, 0.1, 1.2), (5, 5, 18, 0.0, 3.0, 2.0),
         (5, 4, 7, -2.0, 1.0, 2.0), (7, 2, 19, 0.0, 3.0, 1.5), (7, 4, 6, -3.0, 1.0, 2.0), (7, 3, 1, -2.0, 1.0, 2.0)]


@pytest.mark.parametrize("p,m,s,q,beta,alpha", CASES)
def test_pairs_have_equal_norms(exponents, p, m, s, q, beta, alpha):
    """The power of two leaves a factor sqrt(2); the norm is estimated from the
    kernel alone, which a factor 2 covers on nets of few points."""
    gam = inputs.kernel_weights(s, q=q, beta=beta)
    cols = columns(p, m, alpha, gam, 7 * p + m)
    ix = exponents(p, m, alpha, gam)
    assert len(ix) == s
    for i in range(s):
        a, b = cols[2 * i], cols[2 * i + 1]
        if not (np.max(np.abs(b)) > 1e-150 and np.max(np.abs(a)) > 1e-150):
            continue  # squares of the numpy norm leave the range of double
        r = np.linalg.norm(a) / np.linalg.norm(np.ldexp(b, ix[i]))
        assert 1.0 / (2 * np.sqrt(2.0)) <= r <= 2 * np.sqrt(2.0), (i, r)


def test_degenerate_weights(exponents):
    """Columns that vanish or overflow get no scale, and none leaves the range
    of ldexp."""
    for gam in ([1e-200, 1e-200, 1e-200], [1e300, 1.0, 1e300], [1e-160, 1e150, 1e-160, 1e150]):
        ix = exponents(3, 4, 2.0, np.array(gam))
        assert all(-1000 <= v <= 1000 for v in ix)


def dft(p, m, x):
    """Unnormalised transform, one digit at a time, in the precision of x; the
    weights of digits h and -h are exact conjugates, as in the kernels."""
    th = np.longdouble(2) * np.arccos(np.longdouble(-1)) * np.arange((p + 1) // 2) / p
    w = np.cos(th) - 1j * np.sin(th)
    w = np.concatenate([w, np.conj(w[:0:-1])]).astype(x.dtype)
    for d in range(m):
        v = x.reshape(-1, p, p ** d)
        x = np.stack([sum(v[:, n] * w[n * h % p] for n in range(p)) for h in range(p)], 1).reshape(-1)
    return x


@pytest.mark.parametrize("p,m,s,q,beta,alpha", [c for c in CASES if c[1] > 2 and c[2] <= 24])
def test_pair_spectra_are_as_exact_as_single_ones(exponents, p, m, s, q, beta, alpha):
    """The worst column of all pairs, relative to its norm, against the worst
    column alone: norms within a factor 2 sqrt(2) let the rounding grow by
    sqrt(1 + 8) at most for the smaller one, which the real part shares."""
    gam = inputs.kernel_weights(s, q=q, beta=beta)
    cols = columns(p, m, alpha, gam, 7 * p + m)[:2 * s - 1]
    ix = exponents(p, m, alpha, gam)

    def error(got, c):
        ref = dft(p, m, c.astype(np.clongdouble)).real
        return float(np.linalg.norm((got - ref).astype(np.float64)) / max(np.linalg.norm(ref.astype(np.float64)), 1e-300))
    alone = max(error(dft(p, m, c.astype(np.complex128)).real, c) for c in cols)
    paired = 0.0
    for i in range(s - 1):
        z = dft(p, m, cols[2 * i] + 1j * np.ldexp(cols[2 * i + 1], ix[i]))
        paired = max(paired, error(z.real, cols[2 * i]), error(np.ldexp(z.imag, -ix[i]), cols[2 * i + 1]))
    assert paired <= 3.0 * alone
