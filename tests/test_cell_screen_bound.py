"""The certification rules of the phase cells' matrix-core screens (Eq. 7 ownership), in exact
arithmetic on the CPU.

Each screen forms its dot products from FP16 halves of FP32 components; the operands are emulated here
operation by operation (exact rationals, every rounding as the kernels do it) and their twelve products
summed exactly.  The matrix instruction's additions are taken at their stated worst, 2^-19 in all and
against the owner: the exact owner's value is lowered and every rival's raised by as much.  The index bits
then go into the values, and the rule with the kernel's own constants (read from its source) must not
certify an out-edge that is not the exact argmax.  Stencils with near-ties, exact mirror pairs and
jittered offsets; and almost every pair of a jittered stencil is certified."""
import math
import os
import re
from fractions import Fraction as Fr

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SOURCE = open(os.path.join(ROOT, "paper_2503_16037_amd", "csrc", "qbuild.hip")).read()
SCALE = 2 ** 10       # of a component; a dot product carries its square
UNIT = SCALE * SCALE
ADDITIONS = Fr(UNIT, 2 ** 19)
F = 65536


def constant(name):
    return Fr(float(re.search(r"constexpr float %s = ([0-9.]+)f;" % name, SOURCE).group(1)))


def f32(x: Fr) -> Fr:
    """x rounded to the nearest FP32 value (ties to even)."""
    if x == 0:
        return Fr(0)
    c = np.float32(float(x))  # within one ulp of the correct rounding
    best = None
    for cand in (np.nextafter(c, np.float32(-np.inf)), c, np.nextafter(c, np.float32(np.inf))):
        cf = Fr(float(cand))
        key = (abs(cf - x), int(np.float32(cand).view(np.uint32)) & 1)
        if best is None or key < best[0]:
            best = (key, cf)
    return best[1]


def f16(x: Fr, nearest: bool) -> Fr:
    """x in FP16, to nearest even or toward zero."""
    if x == 0:
        return Fr(0)
    e = max(math.frexp(float(abs(x)))[1] - 11, -24)
    n = abs(x) / Fr(2) ** e
    n = round(n) if nearest else int(n)
    return (1 if x > 0 else -1) * n * Fr(2) ** e


def fma(a, b, c):
    return f32(a * b + c)


def halves(x: Fr, nearest=False):
    hi = f16(x, nearest)
    return hi, f16(f32(x - hi), nearest)


def tagged(v: Fr, bits: int, tag: int) -> Fr:
    """An FP32 value with `bits` low bits replaced."""
    b = int(np.float32(float(f32(v))).view(np.uint32))
    return Fr(float(np.uint32((b & ~((1 << bits) - 1)) | tag).view(np.float32)))


def lattice(n):
    ga = math.pi * (3.0 - math.sqrt(5.0))
    out = []
    for i in range(n):
        z = 1.0 - (2.0 * i + 1.0) / n
        ph = math.fmod(i * ga, 2.0 * math.pi)
        r = math.sqrt(1.0 - z * z)
        out.append((r * math.cos(ph), r * math.sin(ph), z))
    return out


def rotation(u):
    ux, uy, uz = u
    h = 1.0 / (1.0 + uz)
    xy = (ux * uy) * h
    return [[uz + (uy * uy) * h, -xy, -ux], [-xy, uz + (ux * ux) * h, -uy], [ux, uy, uz]]


def unit(D):
    n = math.sqrt(float(D[0] * D[0] + D[1] * D[1] + D[2] * D[2]))
    return (D[0] / n, D[1] / n, D[2] / n)


def rotated(M, x, y, z):
    """The kernels' FP32 rotation: rows of M (FP32) times (x, y, z), one product and two FMAs."""
    return [fma(r[2], z, fma(r[1], y, f32(r[0] * x))) for r in M]


def products(a, b):
    """All four products of the halves of two vectors, summed exactly."""
    return sum((ah + al) * (bh + bl) for (ah, al), (bh, bl) in zip(a, b))


def operands(kind, R, p, D, delta):
    """The screen's exact sum for one pair.  tile: the out-edge rotated against the lattice; rest: the
    point rotated against the out-edge; dense: the same, the out-edge from its integer offset by an
    approximate reciprocal root (off by delta units in the last place)."""
    R32 = [[f32(Fr(x)) for x in row] for row in R]
    if kind == "dense":
        x, y, z = (Fr(float(np.float32(c))) for c in D)
        n2 = float(fma(z, z, fma(y, y, f32(x * x))))
        inv = np.float32(1.0 / math.sqrt(n2))
        inv = Fr(float(np.nextafter(inv, np.float32(np.inf if delta > 0 else 0)) if delta else inv)) * SCALE
        site = [f32(c * inv) for c in (x, y, z)]
    else:
        site = [f32(Fr(c)) * SCALE for c in unit(D)]
    if kind == "tile":
        return products([halves(c) for c in rotated(R32, *site)], [halves(f32(Fr(c) * SCALE), True) for c in p]), None
    T = [[R32[r][k] for r in range(3)] for k in range(3)]
    q = rotated(T, *[f32(Fr(c)) * SCALE for c in p])
    again = fma(site[2], q[2], fma(site[1], q[1], f32(site[0] * q[0])))  # the dense nodes' second look
    return products([halves(c) for c in q], [halves(c) for c in site]), again


def exact_values(R, p, D):
    q = [sum(Fr(R[r][k]) * Fr(p[r]) for r in range(3)) for k in range(3)]
    return [sum(a * Fr(b) for a, b in zip(q, unit(d))) for d in D]


def small_screen(kind, R, p, D, exact):
    """(owner, certified) of k_qbuild's rule (d <= 64) with the additions at their worst."""
    top = max(range(len(D)), key=lambda m: exact[m])
    bits = 5 if len(D) <= 32 else 6
    values = []
    for m, d in enumerate(D):
        v, _ = operands(kind, R, p, d, 0)
        v += -ADDITIONS if m == top else ADDITIONS
        values.append((tagged(v, bits, m & ~1 & ((1 << bits) - 1)), m))
    order = sorted(values, key=lambda t: -t[0])
    return order[0][1], f32(order[0][0] - order[1][0]) > constant("kCertified")


def dense_screen(R, p, D, exact, delta):
    """(owner, certified) of k_qbuild_big's rule: the tile of the largest value again in FP32, against
    the other tiles' largest."""
    top = max(range(len(D)), key=lambda m: exact[m])
    first, second = [], []
    for m, d in enumerate(D):
        v, again = operands("dense", R, p, d, delta if m != top else -delta)
        first.append(v + (-ADDITIONS if m == top else ADDITIONS))
        second.append(again)
    # a tile of a lane: 16 of 32 rows, those with (row / 4) mod 2 equal
    tile = [(m // 32, m // 4 % 2) for m in range(len(D))]
    best = tile[max(range(len(D)), key=lambda m: first[m])]
    inside = sorted(((tagged(second[m], 4, m % 16), m) for m in range(len(D)) if tile[m] == best), key=lambda t: -t[0])
    rivals = [f32(first[m]) for m in range(len(D)) if tile[m] != best] + [v for v, _ in inside[1:]]
    return inside[0][1], not rivals or f32(inside[0][0] - max(rivals)) > constant("kBigCertified")


def near_tie_stencil(n, rng):
    """Out-edges with duplicates a few fixed-point units apart (1e-6 .. 1e-4 rad), at distant
    indices, exact mirror pairs and a jittered shell."""
    head = [(F, 0, 0), (-F, 0, 0), (0, F, 0), (0, 0, F), (0, 0, -F), (F, F, 0), (F, -F, 0), (-F, F, F)]
    tail = [(F, 3, 0), (F, 0, 7), (0, F, 1), (F, F, 2), (-F, F, F + 5), (1, 2, F)]
    jit = [tuple(int(x) for x in rng.integers(-2 * F, 2 * F, 3)) for _ in range(n - len(head) - len(tail))]
    return head + jit + tail


def directions(D, rng):
    out = [tuple(-c for c in unit(D[m])) for m in (0, 5, 7, len(D) - 1)]
    v = rng.standard_normal((2, 3))
    out += [tuple(x / np.linalg.norm(x)) for x in v]
    return [tuple(float(c) for c in u) for u in out]


def points_near_ties(R, D, rng):
    """Lattice-like unit points, the bisectors of pairs of out-edges among them."""
    pts = lattice(100)[3::17]
    for a, b in ((0, len(D) - 6), (2, len(D) - 4), (5, len(D) - 3), (0, 5)):
        s = np.array(unit(D[a])) + np.array(unit(D[b])) + rng.standard_normal(3) * 1e-5
        q = s / np.linalg.norm(s)
        pts.append(tuple(float(x) for x in np.array(R) @ q))
    return pts


@pytest.mark.parametrize("kind, n", [("tile", 22), ("rest", 22), ("tile", 50), ("dense", 70)])
def test_no_certificate_for_another_owner(kind, n):
    rng = np.random.default_rng(n)
    D = near_tie_stencil(n, rng)
    worst, worst_again, certified, total = Fr(0), Fr(0), 0, 0
    for u in directions(D, rng):
        R = rotation(u)
        for p in points_near_ties(R, D, rng):
            exact = exact_values(R, p, D)
            order = sorted(exact)
            for m in range(0, n, 7):  # the operands' own error, before the additions
                v, again = operands(kind, R, p, D[m], 1)
                worst = max(worst, abs(v / UNIT - exact[m]))
                if kind == "dense":
                    worst_again = max(worst_again, abs(again / UNIT - exact[m]))
            if kind == "dense":
                runs = [dense_screen(R, p, D, exact, delta) for delta in (0, 1, -1)]
            else:
                runs = [small_screen(kind, R, p, D, exact)]
            for owner, sure in runs:
                total += 1
                certified += sure
                if sure:
                    assert exact[owner] == order[-1] and order[-1] - order[-2] > Fr(1, 2 ** 50), (u, p, owner)
    print(kind, n, "operands off by 2^%.2f" % math.log2(worst), "certified", certified, "of", total)
    # the stated shares of the error, and that two values' errors together stay below the gap: 10.5 of a
    # component's 2^-24 by the operands (13 where the points are rotated, and 6 for the reciprocal root, of dense nodes; 5, 6 and three
    # roundings in the second look), the additions, and the index where a value has one
    eps = Fr(1, 2 ** 24)
    root3 = Fr(17321, 10000)
    if kind == "dense":
        first, second, gap = (13 * root3 + 6) * eps, (5 * root3 + 9) * eps, constant("kBigCertified") / UNIT
        assert worst < first and worst_again < second
        assert first + ADDITIONS / UNIT + second + Fr(1, 2 ** 19) < gap
    else:
        first = Fr(21 if kind == "tile" else 26, 2) * root3 * eps
        assert worst < first
        assert 2 * (first + ADDITIONS / UNIT + Fr(1, 2 ** 17)) < constant("kCertified") / UNIT
    assert certified > total / 4


@pytest.mark.parametrize("kind", ["tile", "dense"])
def test_jittered_stencils_are_certified(kind):
    rng = np.random.default_rng(3)
    D = [tuple(int(c * F + rng.integers(-F // 4, F // 4)) for c in (x, y, z))
         for x in (-1, 0, 1) for y in (-1, 0, 1) for z in (-1, 0, 1) if (x, y, z) != (0, 0, 0)]
    R = rotation(tuple(-c for c in unit(D[4])))
    sure = 0
    pts = lattice(100)[::2]
    for p in pts:
        exact = exact_values(R, p, D)
        sure += (dense_screen(R, p, D, exact, 0) if kind == "dense" else small_screen(kind, R, p, D, exact))[1]
    assert sure >= len(pts) - 1
