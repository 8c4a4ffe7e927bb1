"""Host emulation of a static p = 2 pass from its loads to its stores
(csrc/fwt.hip, fwt_p2 with LOGE >= 10; csrc/p2_stages.h, p2_low6, lane_bfly):
the stages on the loaded registers, those between lanes (swaps of register
halves for strided tiles, quads for contiguous ones) and those on the stored
registers, with the kernels' own element mappings and padded LDS indices, give
the transform of the pass's digits, exactly, in integers."""
import numpy as np
import pytest


def cpad(e):
    return e + (e >> 5)


def reg_bfly(v, bits):
    """Radix-2 stages over register-index bits; v [thread][register]."""
    for b in bits:
        w = v.copy()
        for j in range(v.shape[1]):
            if not (j >> b) & 1:
                w[:, j], w[:, j | 1 << b] = v[:, j] + v[:, j | 1 << b], v[:, j] - v[:, j | 1 << b]
        v = w
    return v


def lane_swap(a, b, H):
    """v_permlane16_swap / v_permlane32_swap on whole waves: a's lanes with bit
    H set and b's lanes with it clear change places."""
    lane = np.arange(64)
    hi, lo = lane[(lane & H) != 0], lane[(lane & H) == 0]
    a, b = a.reshape(-1, 64).copy(), b.reshape(-1, 64).copy()
    t = a[:, hi].copy()
    a[:, hi] = b[:, lo]
    b[:, lo] = t
    return a.reshape(-1), b.reshape(-1)


def lane_bfly(v, H):
    for j in range(0, v.shape[1], 2):
        a, b = lane_swap(v[:, j], v[:, j + 1], H)
        a, b = lane_swap(a + b, a - b, H)
        v[:, j], v[:, j + 1] = a, b
    return v


def low6(lds, th):
    """p2_low6: digits 0..3 in the registers of 16 consecutive elements, 4 and
    5 between the lanes of a quad (own + other, or other - own)."""
    tid = np.arange(th)
    idx = cpad(16 * tid)[:, None] + cpad(np.arange(16))[None, :]
    assert np.array_equal(idx, cpad(16 * tid[:, None] + np.arange(16)[None, :]))
    x = reg_bfly(lds[idx], range(4))
    for bit in (1, 2):
        other = x[tid ^ bit]
        x = np.where(((tid & bit) != 0)[:, None], other - x, x + other)
    lds[idx] = x


def transform_digits(x, bits):
    for b in bits:
        v = x.reshape(-1, 2, 1 << b)
        x = np.stack([v[:, 0] + v[:, 1], v[:, 0] - v[:, 1]], 1).reshape(-1)
    return x


@pytest.mark.parametrize("H", [16, 32])
def test_swaps_pair_the_halves(H):
    """A lane_bfly is the butterfly of lane bit H on every register."""
    g = np.random.default_rng(H)
    v = g.integers(-100, 100, size=(128, 16))
    lane = np.arange(128)
    want = np.where(((lane & H) != 0)[:, None], v[lane ^ H] - v, v + v[lane ^ H])
    assert np.array_equal(lane_bfly(v.copy(), H), want)


@pytest.mark.parametrize("loge,wdig", [(e, w) for e in range(10, 15) for w in (0, 4, 5)])
def test_pass(loge, wdig):
    E, th = 1 << loge, (1 << loge) // 16
    g = np.random.default_rng(100 * loge + wdig)
    x = g.integers(-1000, 1000, size=E)
    tid, k = np.arange(th), np.arange(16)
    v = x[tid[:, None] + k[None, :] * th]  # element tid + k TH
    v = reg_bfly(v, range(4))
    if wdig == 4:
        v = lane_bfly(v, 16)
    if wdig > 0:
        v = lane_bfly(v, 32)
    lds = np.zeros(cpad(E) + 1, dtype=np.int64)
    lds[cpad(tid)[:, None] + cpad(k * th)[None, :]] = v
    if wdig == 0:
        low6(lds, th)
    lane, wv = tid & 63, tid >> 6
    v = lds[cpad(lane + 1024 * wv)[:, None] + 66 * k[None, :]]
    v = reg_bfly(v, range(min(loge - 10, 4)))
    out = np.zeros(E, dtype=np.int64)
    out[(lane + 1024 * wv)[:, None] + 64 * k[None, :]] = v  # stored element
    assert np.array_equal(out, transform_digits(x, range(wdig, loge)))
