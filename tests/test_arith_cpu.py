"""The double per-cell and per-face arithmetic of csrc/device.h and adjoint.h, compiled for the
CPU with the fused multiply-adds of the device build, against the same formulas in
80-bit floating point (64-bit mantissa).

The parity tests measure a row against its largest value.  Here every value is
measured on its own scale, which is what a trace phase beside an interface needs.
"""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
LD = np.longdouble
EPS64 = 2.0 ** -53
JS, Z, M = 0, 1, 3


@pytest.fixture(scope="session")
def arith(tmp_path_factory):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    so = str(tmp_path_factory.mktemp("arith") / "arith_host.so")
    subprocess.run([hipcc, "--offload-host-only", "-x", "hip", "-O2", "-std=c++17", "-mfma", "-fPIC", "-shared",
                    os.path.join(HERE, "native", "arith_host.hip"), "-o", so], check=True, capture_output=True)
    return ctypes.CDLL(so)


def _ptr(a):
    assert a.dtype == np.float64 and a.flags.c_contiguous
    return a.ctypes.data_as(ctypes.POINTER(ctypes.c_double))


def weno(lib, variant, f, eps=1e-6):
    f = np.ascontiguousarray(f)
    fl, fr = np.empty(f.shape[1]), np.empty(f.shape[1])
    lib.arith_weno(variant, ctypes.c_double(eps), f.shape[1], _ptr(f), _ptr(fl), _ptr(fr))
    return fl, fr


def weno_exact(variant, f, eps=1e-6):
    """Left-biased value at the face above the centre, in 80 bits; each candidate
    as the centre value plus its correction."""
    a, b, c, d, e = (x.astype(LD) for x in f)
    D0, D1, D2, D3 = b - a, c - b, d - c, e - d
    beta = [LD(13) / 12 * (D1 - D0) ** 2 + LD(1) / 4 * (3 * D1 - D0) ** 2,
            LD(13) / 12 * (D2 - D1) ** 2 + LD(1) / 4 * (D1 + D2) ** 2,
            LD(13) / 12 * (D3 - D2) ** 2 + LD(1) / 4 * (D3 - 3 * D2) ** 2]
    lin = [LD(1) / 10, LD(6) / 10, LD(3) / 10]
    if variant == Z:
        tau = abs(beta[0] - beta[2])
        w = [g * (1 + tau / (x + LD(eps))) for g, x in zip(lin, beta)]
    else:
        w = [g / (LD(eps) + x) ** 2 for g, x in zip(lin, beta)]
    if variant == M:
        t = w[0] + w[1] + w[2]
        w = [x / t for x in w]
        w = [x * (g + g * g - 3 * g * x + x * x) / (g * g + x * (1 - 2 * g)) for g, x in zip(lin, w)]
    t = w[0] + w[1] + w[2]
    parts = [w[0] * (5 * D1 - 2 * D0) / (6 * t), w[1] * (D1 + 2 * D2) / (6 * t), w[2] * (4 * D2 - D3) / (6 * t)]
    return c + (parts[0] + parts[1] + parts[2]), parts


# small smooth side, other side: pressure, a trace partial density, a volume
# fraction at its floor, a gas density
JUMPS = [(1e5, 7e8), (1e-3, 1e3), (1e-6, 0.5), (0.125, 1.0)]


def jump_stencils(small, large, cut, m=20000, seed=0):
    """Stencils with `small` (1 +- 5 %, smooth) in the cells before `cut` and `large` in the others."""
    rng = np.random.default_rng(seed)
    x0, k = rng.uniform(0, 6, m), rng.uniform(0.01, 0.3, m)
    f = np.stack([(small if i < cut else large) * (1 + 0.05 * np.sin(x0 + i * k)) for i in range(5)])
    return np.ascontiguousarray(f)


@pytest.mark.parametrize("cut", (3, 4))
@pytest.mark.parametrize("small,large", JUMPS)
@pytest.mark.parametrize("variant", (JS, Z, M))
def test_weno_beside_a_jump_on_the_scale_of_the_value(arith, variant, small, large, cut):
    """The value at a face on the small, smooth side of a jump.  Bar: the sum of a
    centre value and three weighted corrections, each formed in at most ten
    roundings (differences, indicator, its square, weight, normalization, sum), so
    10 eps of the terms' magnitudes; the centre and the jump's own term, where its
    weight leaves it any, included."""
    f = jump_stencils(small, large, cut)
    got = weno(arith, variant, f)[0]
    mirrored = weno(arith, variant, f[::-1])[1]
    ref, parts = weno_exact(variant, f)
    size = abs(f[2].astype(LD)) + sum(abs(p) for p in parts)
    for y in (got, mirrored):
        err = np.abs((y.astype(LD) - ref) / size).astype(float)
        print(f"variant {variant} {small:g} | {large:g}, {cut} small cells: rms {np.sqrt((err ** 2).mean()):.1e} max {err.max():.1e}")
        assert err.max() <= 10 * 2 * EPS64


def js_derivative(f, eps=1e-6):
    """d(left-biased WENO5-JS value)/dD_j in 80 bits, and the sum of the magnitudes of the terms that make it up."""
    a, b, c, d, e = (x.astype(LD) for x in f)
    D = [b - a, c - b, d - c, e - d]
    corr = [(5 * D[1] - 2 * D[0]) / 6, (D[1] + 2 * D[2]) / 6, (4 * D[2] - D[3]) / 6]
    dcorr = np.array([[-2, 5, 0, 0], [0, 1, 2, 0], [0, 0, 4, -1]], LD) / 6
    # beta_k as quadratic forms of the differences: 13/12 u^2 + 1/4 v^2
    uv = [((-1, 1, 0, 0), (-1, 3, 0, 0)), ((0, -1, 1, 0), (0, 1, 1, 0)), ((0, 0, -1, 1), (0, 0, -3, 1))]
    dot = lambda w: sum(LD(x) * y for x, y in zip(w, D))
    beta = [LD(13) / 12 * dot(u) ** 2 + LD(1) / 4 * dot(v) ** 2 for u, v in uv]
    w = [g / (LD(eps) + x) ** 2 for g, x in zip((LD(1) / 10, LD(6) / 10, LD(3) / 10), beta)]
    t = w[0] + w[1] + w[2]
    w = [x / t for x in w]
    y = w[0] * corr[0] + w[1] * corr[1] + w[2] * corr[2]
    out, size = [], []
    for j in range(4):
        g, m = 0, 0
        for k in range(3):
            u, v = uv[k]
            db = LD(13) / 6 * dot(u) * u[j] + LD(1) / 2 * dot(v) * v[j]
            mag = sum(abs(LD(13) / 6 * u[i] * u[j] + LD(1) / 2 * v[i] * v[j]) * abs(D[i]) for i in range(4))
            r = 2 * w[k] / (LD(eps) + beta[k])
            g = g + w[k] * dcorr[k, j] - r * (corr[k] - y) * db
            m = m + w[k] * abs(dcorr[k, j]) + r * (abs(corr[k]) + abs(y)) * mag
        out.append(g)
        size.append(m)
    return out, size


@pytest.mark.parametrize("cut", (1, 2, 3, 4, 5))
@pytest.mark.parametrize("small,large", JUMPS)
def test_weno_js_adjoint_beside_a_jump(arith, small, large, cut):
    """The derivative of both biased values in the four differences, each entry
    against the magnitudes of the terms that make it up (the largest entry of the
    stencil where its own are smaller: one difference's entry holds a share of its
    neighbours' weights).  Bar: 30 roundings."""
    f = jump_stencils(small, large, cut, seed=1)
    m = f.shape[1]
    ref, size = js_derivative(f)
    top = np.maximum.reduce(size)
    one, zero = np.ones(m), np.zeros(m)
    gD = np.empty((4, m))
    arith.arith_weno_js_vjp(ctypes.c_double(1e-6), m, _ptr(f), _ptr(one), _ptr(zero), _ptr(gD))
    left = [np.abs((gD[j].astype(LD) - ref[j]) / top).max() for j in range(4)]
    g = np.ascontiguousarray(f[::-1])
    arith.arith_weno_js_vjp(ctypes.c_double(1e-6), m, _ptr(g), _ptr(zero), _ptr(one), _ptr(gD))
    right = [np.abs((-gD[3 - j].astype(LD) - ref[j]) / top).max() for j in range(4)]
    print(f"{small:g} | {large:g}, {cut} small cells: {float(max(left)):.1e} {float(max(right)):.1e}")
    assert max(max(left), max(right)) <= 30 * 2 * EPS64


def nu_exact(base, f, eps):
    """Both face values of the tabulated scheme in 80 bits from the table's candidates
    and ideal weights, and the magnitudes of their terms: [right, left]."""
    D = [f[i + 1].astype(LD) - f[i].astype(LD) for i in range(4)]
    b = base.astype(LD)
    lin = lambda row, r: (b[row + 2 * r] * D[r], b[row + 2 * r + 1] * D[r + 1])
    m0, m1, m2 = ([lin(row, r) for r in range(3)] for row in (0, 6, 12))
    beta = [sum(m1[r]) ** 2 + LD(13) / 3 * sum(m2[r]) ** 2 for r in range(3)]
    out = []
    for row, sign in ((18, 1), (21, -1)):
        w = [b[row + r] / (LD(eps) + beta[r]) ** 2 for r in range(3)]
        t = w[0] + w[1] + w[2]
        y = sum(w[r] * (sum(m0[r]) + sum(m2[r]) / 4 + sign * sum(m1[r]) / 2) for r in range(3)) / t
        mag = sum(abs(w[r]) * sum(abs(m0[r][j]) + abs(m2[r][j]) / 4 + abs(m1[r][j]) / 2 for j in (0, 1)) for r in range(3))
        out.append((f[2].astype(LD) + y, abs(f[2].astype(LD)) + mag / abs(t)))
    return out


@pytest.mark.parametrize("kind", ("smooth", "random", "jump"))
@pytest.mark.parametrize("ratio", (1.2, 2.0, 10.0))
def test_weno_on_a_stretched_grid_on_the_scale_of_the_value(arith, ratio, kind):
    """The folded table entries against the candidates and ideal weights that they
    come from, widths within `ratio` of each other, smooth and random data and both
    sides of jumps.  Bar: 10 eps of the magnitudes of the terms, as on a uniform
    grid."""
    rng = np.random.default_rng(5)
    worst, sq, count = 0.0, 0.0, 0
    for g in range(60):
        widths = ratio ** rng.uniform(-0.5, 0.5, 5)
        faces = np.concatenate([[0.0], np.cumsum(widths)])
        x = np.cumsum(widths)[:, None] - 0.5 * widths[:, None]
        m = 400
        smooth = 1 + 0.05 * np.sin(rng.uniform(0, 6, m) + 10 ** rng.uniform(-2, 0, m) * x)
        if kind == "smooth":
            f = smooth
        elif kind == "random":
            f = rng.uniform(-1, 1, (5, m))
        else:
            small, large = JUMPS[g % 4]
            f = smooth * np.where(np.arange(5)[:, None] < rng.integers(1, 5, m), small, large)
            f = f if g % 2 else f[::-1]
        f = np.ascontiguousarray(f)
        fl, fr, base = np.empty(m), np.empty(m), np.empty(24)
        assert arith.arith_weno_nu(ctypes.c_double(1e-6), _ptr(faces), m, _ptr(f), _ptr(fl), _ptr(fr), _ptr(base)) == 0
        for got, (ref, size) in zip((fl, fr), nu_exact(base, f, 1e-6)):  # fl: the right face
            e = np.abs((got.astype(LD) - ref) / size).astype(float)
            worst, sq, count = max(worst, e.max()), sq + (e ** 2).sum(), count + m
    print(f"{kind}, widths to {ratio}: rms {np.sqrt(sq / count):.1e} max {worst:.1e}")
    assert worst <= 10 * 2 * EPS64


def test_weno_on_extremely_stretched_grids_stays_finite(arith):
    """Cells up to 1e12 times their neighbours: the folded entries are products, none a quotient that may have no divisor."""
    rng = np.random.default_rng(6)
    f = np.ascontiguousarray(rng.uniform(-1, 1, (5, 100)))
    for ratio in (1e3, 1e6, 1e12):
        for _ in range(20):
            faces = np.concatenate([[0.0], np.cumsum(ratio ** rng.uniform(-0.5, 0.5, 5))])
            fl, fr, base = np.empty(100), np.empty(100), np.empty(24)
            if arith.arith_weno_nu(ctypes.c_double(1e-6), _ptr(faces), 100, _ptr(f), _ptr(fl), _ptr(fr), _ptr(base)):
                continue
            if np.isfinite(base).all():
                assert np.isfinite(fl).all() and np.isfinite(fr).all(), (ratio, faces)


HLLC, HLL, THORNBER, APC = 0, 1, 2, 4
GAS, WATER_AIR = ((1.4,), (0.0,)), ((6.12, 1.4), (3.43e8, 0.0))


def faces(lib, options, fluids, wl, wr):
    gamma, pi_inf = (np.array(x, dtype=np.float64) for x in fluids)
    wl, wr = np.ascontiguousarray(wl), np.ascontiguousarray(wr)
    n, m = wl.shape
    flux, uf, vjp_uf = np.empty((n, m)), np.empty(m), np.empty(m)
    lib.arith_face(options, len(gamma), _ptr(gamma), _ptr(pi_inf), m, _ptr(wl), _ptr(wr), _ptr(flux), _ptr(uf), _ptr(vjp_uf))
    return flux, uf, vjp_uf


@pytest.mark.parametrize("unit", (1.0, 1e3, 1e6, 1e9))
@pytest.mark.parametrize("mach", (0.1, 0.9, 1.5, 5.0))
@pytest.mark.parametrize("options", (HLLC, HLL, APC))
def test_uniform_stream_in_any_unit_of_velocity(arith, options, mach, unit):
    """The energy flux of a uniform stream of air is (E + p) u, whatever the unit of
    velocity (pressure in its square).  Bar: the flux takes less than 20 roundings of
    its terms, all of one sign here."""
    rng = np.random.default_rng(9)
    m = 5000
    rho = rng.uniform(0.5, 2.0, m)
    p = rng.uniform(0.5e5, 2e5, m) * unit ** 2
    u = mach * np.sqrt(1.4 * p / rho)
    w = np.stack([rho, u, 0.3 * u, p])
    flux, uf, _ = faces(arith, options, GAS, w, w)
    r, p, u, v = (x.astype(LD) for x in (rho, p, u, 0.3 * u))
    E = p / (LD(1.4) - 1) + r * (u * u + v * v) / 2
    err = np.abs(flux[3] / ((E + p) * u) - 1).max()
    print(f"options {options} Mach {mach} unit {unit:g}: {float(err):.1e}")
    assert err <= 20 * 2 * EPS64


def interface_faces(m, seed, speed):
    """Two-fluid face states on both sides of smeared interfaces, pressure equal up to its rounding, velocity noise of size `speed`."""
    rng = np.random.default_rng(seed)
    w = []
    p = 1e5 * (1 + 0.1 * rng.uniform(-1, 1, m))
    for _ in range(2):
        a = rng.uniform(1e-6, 1 - 1e-6, m)
        noise = 1 + rng.integers(-2, 3, m) * 2.0 ** -52
        w.append(np.stack([1000.0 * a, 1.0 * (1 - a), speed * rng.uniform(-1, 1, m), 10 * rng.uniform(-1, 1, m), p * noise, a, 1 - a]))
    return w


@pytest.mark.parametrize("speed", (0.0, 1e-12, 1.0, 2000.0))
@pytest.mark.parametrize("options", (HLLC, HLL, THORNBER, APC))
def test_adjoint_face_velocity_is_the_solvers(arith, options, speed):
    """The adjoint recomputes the face velocity; its last bit decides the side of a
    face at rest (the volume fraction that rides the contact), so it has to be the
    solver's own, bit for bit."""
    wl, wr = interface_faces(20000, 11, speed)
    _, uf, vjp_uf = faces(arith, options, WATER_AIR, wl, wr)
    print(f"options {options} speed {speed:g}: {np.mean(uf != vjp_uf):.3f} differ, {np.mean((uf >= 0) != (vjp_uf >= 0)):.4f} on the other side")
    assert np.array_equal(uf, vjp_uf)
