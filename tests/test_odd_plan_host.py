"""Host checks of the odd-p passes (csrc/pass_geom.h, csrc/odd.hip): every plan
covers the digits once with shapes that are compiled, every compiled shape
belongs to a plan, the plans depend on nothing but p, m, the type and the
number of columns, and the index arithmetic of the kernels (OddShape,
OddGroups, emulated) visits every tile element once per stage group."""
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def table():
    """{(p, f64, m): passes}, {(p, f64, le, rd): (kt, also kt 3)} (the plain
    C++ header, no device in sight)."""
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        exe = os.path.join(d, "pass_geom_check")
        subprocess.run(["g++", "-O1", "-std=c++17", "-I" + os.path.join(ROOT, "paper_0808_0487_amd", "csrc"),
                        os.path.join(ROOT, "tests", "pass_geom_check.cpp"), "-o", exe], check=True)
        out = subprocess.run([exe], capture_output=True, text=True, check=True).stdout
    plans, shapes = {}, {}
    for line in out.splitlines():
        w = line.split()
        if w[0] == "plan":
            plans[tuple(map(int, w[1:4]))] = [tuple(map(int, x.split(","))) for x in w[4:]]
        else:
            shapes[tuple(map(int, w[1:5]))] = (int(w[5]), int(w[6]))
    return plans, shapes


PLANS, SHAPES = table()


@pytest.mark.parametrize("p,f64", [(p, f) for p in (3, 5, 7) for f in (0, 1)])
def test_plans_cover_the_digits_with_compiled_shapes(p, f64):
    size, used = (16 if f64 else 8), set()
    for (q, g, m), passes in PLANS.items():
        if (q, g) != (p, f64):
            continue
        done = 0
        for i, (d0, r, wdig, le, kt3) in enumerate(passes):
            assert d0 == done and r >= 1 and wdig == le - r and wdig <= d0
            assert (i == 0) == (d0 == 0) == (r == le)           # the first pass contiguous, the others strided
            assert le <= m and p ** le * size <= 160 * 1024     # whole tiles, in the LDS of a CU
            assert (p, f64, le, r) in SHAPES
            assert not kt3 or SHAPES[(p, f64, le, r)][1]        # three register digits where they are compiled
            used.add((p, f64, le, r))
            done += r
        assert done == m
        assert len(passes) <= 2 or m > 2 * max(g[3] for g in passes) - (2 if p == 3 else 1)  # two passes where they do
    assert used == {s for s in SHAPES if s[:2] == (p, f64)}     # nothing compiled that no plan needs


def digit(v, p, i):
    return (v // p ** i) % p


@pytest.mark.parametrize("p,f64,le,rd,kt", sorted({(p, f, le, rd, k) for (p, f, le, rd), (kt, k3) in SHAPES.items()
                                                    for k in ([kt, 3] if k3 else [kt])}))
def test_index_arithmetic(p, f64, le, rd, kt):
    E, th, w = p ** le, p ** (le - kt), p ** (le - rd)
    rstep = p ** (rd - kt)
    assert th % w == 0 and th <= 1024 and rd >= kt
    tid = np.arange(th)
    # Loads and stores: element tid + k TH at goff0 + k gstep, any row stride.
    sd0 = p ** 9 + 17
    seen, rows = np.zeros(E, dtype=np.int64), []
    for k in range(p ** kt):
        e = tid + k * th
        assert np.array_equal(tid % w + (tid // w) * sd0 + k * rstep * sd0, e % w + (e // w) * sd0)
        np.add.at(seen, e, 1)
        rows.append(e // w)
    assert np.all(seen == 1)
    rows = np.stack(rows, 1)
    kk = np.arange(p ** kt)
    for i in range(rd):  # a thread's values differ in the KT top digits, in the order of k
        want = digit(kk, p, i - (rd - kt)) if i >= rd - kt else None
        assert np.all(digit(rows, p, i) == (want if want is not None else digit(rows[:, :1], p, i)))
    covered, q = list(range(rd - kt, rd)), 0
    while q < rd - kt:  # OddGroups
        kg = min(kt, rd - kt - q)
        R, pq = p ** kg, p ** q
        assert E % (R * th) == 0
        cover = np.zeros(E, dtype=np.int64)
        for g in range(E // R // th):
            u = tid // w + g * rstep
            e = (tid % w + w * (u % pq + pq * R * (u // pq)))[:, None] + np.arange(R)[None, :] * (w * pq)
            assert e.max() < E
            np.add.at(cover, e.ravel(), 1)
            r = e // w
            assert np.all(e % w == (e % w)[:, :1])
            for i in range(rd):
                want = digit(np.arange(R), p, i - q) if q <= i < q + kg else digit(r[:, :1], p, i)
                assert np.all(digit(r, p, i) == want)
        assert np.all(cover == 1)
        covered += range(q, q + kg)
        q += kg
    assert sorted(covered) == list(range(rd))
