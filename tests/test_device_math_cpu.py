"""The device's per-cell and per-face arithmetic (csrc/device_math.hpp)
compiled for the host, against extended precision (64-bit mantissa)."""
from __future__ import annotations

import ctypes
import os
import subprocess

import numpy as np
import pytest

HERE = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host_math")
LD = np.longdouble
EPS = 2.0 ** -52


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    assert np.finfo(LD).nmant >= 63
    so = str(tmp_path_factory.mktemp("host_math") / "host_math.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-w", "-ffp-contract=off", "-shared", "-fPIC", f"-I{HERE}",
                           "-o", so, os.path.join(HERE, "host_math.cpp")])
    return ctypes.CDLL(so)


def _p(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def _srhd_states(rng, n, g, gamma, p_rho):
    """Conserved SRHD states (D, m, tau) of Lorentz factor `gamma`."""
    d = rng.normal(size=(n, 3))
    d *= (np.sqrt(gamma ** 2 - 1.0) / np.linalg.norm(d, axis=1))[:, None]
    rho = rng.uniform(0.3, 3.0, n)
    p = p_rho * rho * rng.uniform(0.5, 2.0, n)
    h = rho + g / (g - 1.0) * p
    U = np.empty((n, 5))
    U[:, 0] = gamma * rho
    U[:, 1:4] = (gamma * h)[:, None] * d
    U[:, 4] = gamma ** 2 * h - p - U[:, 0]
    return U


def _srhd_prims(U, g):
    """Primitives by Newton from a bisected bracket, in extended precision."""
    U = U.astype(LD)
    g = LD(g)
    gg = (g - 1) / g
    D, e = U[:, 0], U[:, 4] + U[:, 0]
    m2 = (U[:, 1:4] ** 2).sum(axis=1)
    lo, hi = np.sqrt(m2), g * e
    x = (lo + hi) / 2
    for _ in range(150):
        q = m2 / (x * x)
        ig = np.sqrt(1 - q)
        f = x - gg * (x * (1 - q) - D * ig) - e
        lo, hi = np.where(f > 0, lo, x), np.where(f > 0, x, hi)
        xn = x - f / (1 - gg * (1 + q - D * q / (ig * x)))
        x = np.where((xn > lo) & (xn < hi), xn, (lo + hi) / 2)
    ig = np.sqrt(1 - m2 / (x * x))
    return np.concatenate([(D * ig)[:, None], U[:, 1:4] / (x * ig)[:, None],
                           (gg * (x * ig * ig - D * ig))[:, None]], axis=1), x * ig * ig


# A root known to a few ulp (the residual's rounding over f' >= 1 - 2 (g-1)/g)
# moves 1/Gamma^2 = 1 - m^2/xi^2 by 2 Gamma^2 of that, and the pressure, a
# difference of terms of size rho h, by rho h / p more: 16 ulp times those.
@pytest.mark.parametrize("g", [4.0 / 3.0, 5.0 / 3.0])
@pytest.mark.parametrize("gamma", [1.0001, 1.15, 2.0, 5.0, 8.0, 12.0, 16.0, 24.0, 64.0, 100.0, 1000.0])
def test_srhd_state_recovered_at_every_lorentz_factor(lib, gamma, g):
    rng = np.random.default_rng(7)
    for p_rho in (1e-4, 1e-3, 1e-2, 0.1, 1.0, 100.0):
        U = _srhd_states(rng, 400, g, gamma, p_rho)
        w = np.empty_like(U)
        ok = np.empty(len(U), dtype=np.int32)
        lib.srhd_con2prim(ctypes.c_long(len(U)), _p(U), ctypes.c_double(g), _p(w), _p(ok))
        R, rhoh = _srhd_prims(U, g)
        tol = 16 * EPS * gamma ** 2
        assert ok.all()
        assert (np.abs(w[:, 0] - R[:, 0]) <= tol * R[:, 0]).all(), p_rho
        assert (np.abs(w[:, 1:4] - R[:, 1:4]).max(axis=1) <= tol * np.linalg.norm(R[:, 1:4].astype(float), axis=1)).all(), p_rho
        assert (np.abs(w[:, 4] - R[:, 4]) <= tol * rhoh).all(), p_rho


# Supersonic HLLC flux: the physical flux of the upwind side, from products and
# sums of at most four roundings each of numbers no larger than its terms.
@pytest.mark.parametrize("mach", [3.0, 10.0, 100.0, 1e4, 1e6])
@pytest.mark.parametrize("side", [1.0, -1.0])
def test_supersonic_hllc_flux_is_the_upwind_sides(lib, side, mach):
    rng = np.random.default_rng(11)
    g, n = 1.4, 20000
    c = np.sqrt(g)
    wL, wR = (np.stack([rng.uniform(0.8, 1.2, n), side * mach * c * rng.uniform(0.8, 1.2, n),
                        *(mach * c * rng.uniform(-1, 1, (2, n))), rng.uniform(0.8, 1.2, n)], axis=1) for _ in range(2))
    F = np.empty_like(wL)
    lib.euler_flux(1, ctypes.c_long(n), _p(wL), _p(wR), ctypes.c_double(g), _p(F))
    r, u, v, w, p = (wL if side > 0 else wR).astype(LD).T
    h = p * LD(g) / (LD(g) - 1) + r * (u * u + v * v + w * w) / 2
    R = np.stack([r * u, r * u * u + p, r * v * u, r * w * u, u * h], axis=1)
    assert (np.abs(F - R) <= 4 * EPS * np.abs(R)).all(), (np.abs(F - R) / np.abs(R)).max(axis=0)


# Slow flow of one density and transverse velocity: the mass and transverse
# momentum fluxes are the weighted mean of two small mass fluxes, each
# off by the weights' reciprocal (20 ulp) and four roundings of itself; the dissipation
# (sound speed times density, 1e4 times larger here) has to leave nothing.
@pytest.mark.parametrize("rs", [0, 2])
def test_slow_flow_keeps_the_digits_of_its_mass_flux(lib, rs):
    rng = np.random.default_rng(5)
    g, n = 1.4, 20000
    rho, v, w = rng.uniform(0.5, 2.0, n), rng.uniform(-1, 1, n), rng.uniform(-1, 1, n)
    wL, wR = (np.stack([rho, 1e-4 * rng.uniform(0.5, 1.0, n), v, w, rng.uniform(0.8, 1.2, n)], axis=1) for _ in range(2))
    F = np.empty_like(wL)
    lib.euler_flux(rs, ctypes.c_long(n), _p(wL), _p(wR), ctypes.c_double(g), _p(F))
    L, R = wL.astype(LD), wR.astype(LD)
    cL, cR = (np.sqrt(LD(g) * q[:, 4] / q[:, 0]) for q in (L, R))
    sr, sl = np.maximum(L[:, 1] + cL, R[:, 1] + cR), np.minimum(L[:, 1] - cL, R[:, 1] - cR)
    al = sr / (sr - sl) if rs == 0 else LD(0.5)
    m = rho * (al * L[:, 1] + (1 - al) * R[:, 1])
    tol = 24 * EPS * np.abs(m)
    assert (np.abs(F[:, 0] - m) <= tol).all()
    assert (np.abs(F[:, 2] - m * v) <= tol * np.abs(v)).all()
    assert (np.abs(F[:, 3] - m * w) <= tol * np.abs(w)).all()


# The same for MHD with a transverse field equal on both sides (its flux is the
# field times the mean velocity); the weights here carry the fast speeds'
# error too, up to 17 ulp each.
def test_slow_mhd_flow_keeps_the_digits_of_its_fluxes(lib):
    rng = np.random.default_rng(6)
    g, n = 5.0 / 3.0, 20000
    rho, v, w, b1, b2 = rng.uniform(0.5, 2.0, n), *rng.uniform(-1, 1, (4, n))
    zero = np.zeros(n)
    wL, wR = (np.stack([rho, 1e-4 * rng.uniform(0.5, 1.0, n), v, w, rng.uniform(0.8, 1.2, n), zero, b1, b2, zero],
                       axis=1) for _ in range(2))
    F = np.empty_like(wL)
    lib.mhd_flux(ctypes.c_long(n), _p(wL), _p(wR), ctypes.c_double(g), ctypes.c_double(5.0), _p(F))
    L, R = wL.astype(LD), wR.astype(LD)
    cL, cR = (np.sqrt((LD(g) * q[:, 4] + q[:, 6] ** 2 + q[:, 7] ** 2) / q[:, 0]) for q in (L, R))
    sr, sl = np.maximum(L[:, 1] + cL, R[:, 1] + cR), np.minimum(L[:, 1] - cL, R[:, 1] - cR)
    al = sr / (sr - sl)
    u = al * L[:, 1] + (1 - al) * R[:, 1]
    for var, q in ((0, rho), (2, rho * v), (3, rho * w), (6, b1), (7, b2)):
        assert (np.abs(F[:, var] - u * q) <= 64 * EPS * np.abs(u * q)).all(), var


# SRHD energy flux of one hot state, m_n - D v_n with m = Gamma rho h u and D v_n
# = rho u_n: Gamma comes from a reciprocal root within 14 of these eps, once in m
# and twice in D v_n; six roundings besides.
def test_srhd_energy_flux_takes_gamma_once(lib):
    rng = np.random.default_rng(8)
    g, n = 4.0 / 3.0, 20000
    u = rng.normal(size=(n, 3))
    u *= (np.exp(rng.uniform(-1, 3, n)) / np.linalg.norm(u, axis=1))[:, None]
    rho = rng.uniform(0.5, 2.0, n)
    w = np.stack([rho, *u.T, 10.0 * rho * rng.uniform(0.5, 2.0, n)], axis=1)
    F = np.empty_like(w)
    lib.srhd_flux(ctypes.c_long(n), _p(w), _p(w), ctypes.c_double(g), _p(F))
    r, u1, u2, u3, p = w.astype(LD).T
    m = np.sqrt(1 + u1 * u1 + u2 * u2 + u3 * u3) * (r + LD(g) / (LD(g) - 1) * p) * u1
    assert (np.abs(F[:, 4] - (m - r * u1)) <= EPS * (20 * np.abs(m) + 34 * np.abs(r * u1))).all()
