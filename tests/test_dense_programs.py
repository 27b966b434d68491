"""The dense forms of the fifth-dimension programs (CPU only): the library's tables
and rho against the operators' definitions, and the way the kernel hands a wave's
slices to the matrix instructions, modelled lane by lane."""
import ctypes

import numpy as np
import pytest

from paper_1811_08095_amd import odwf

N, CHI, LEN, COUNT = 16, 16 * 16 + 32, 2 * (16 * 16 + 32), 8
NAMES = ["AINV", "AINV_T", "A", "A_T", "1PL", "1PL_T", "1PL_INV", "AINV_WINV"]


def _tables(Ns, m0, omega):
    f = getattr(odwf.lib(), "_ZN4odwf12dense_tablesEidPKdPdPA2_d")
    f.restype = None
    f.argtypes = [ctypes.c_int, ctypes.c_double] + [ctypes.c_void_p] * 3
    w = np.ascontiguousarray(omega, dtype=np.float64)
    tab, q = np.full((COUNT, 2, CHI), np.nan), np.full((COUNT, 2), np.nan)
    f(Ns, m0, w.ctypes.data, tab.ctypes.data, q.ctypes.data)
    return tab, q


def _operators(Ns, m0, omega, mu, chi):
    """In slice order: L_+ hands slice s - 1 to s, L_- hands s + 1 to s, corner -mu."""
    S = np.eye(Ns, k=-1)
    S[0, Ns - 1] = -mu
    L = S if chi == 0 else S[::-1, ::-1]
    one, W = np.eye(Ns), np.diag(omega)
    A = (4 - m0) * one + np.linalg.inv(W) @ (one - L) @ np.linalg.inv(one + L)
    Ai = np.linalg.inv(A)
    return dict(AINV=Ai, AINV_T=Ai.T, A=A, A_T=A.T, AINV_WINV=Ai @ np.linalg.inv(W),
                **{"1PL": one + L, "1PL_T": (one + L).T, "1PL_INV": np.linalg.inv(one + L)})


@pytest.mark.parametrize("m0", [1.3, 1.8])
@pytest.mark.parametrize("Ns", [4, 8, 16])
def test_tables_are_the_operators(Ns, m0):
    rng = np.random.default_rng(Ns)
    for omega in (odwf.zolotarev_omega(Ns, 0.05, 6.2), np.exp(rng.uniform(-2, 3, Ns))):
        tab, q = _tables(Ns, m0, omega)
        for mu in (0.0, 1e-3, 0.3, 1.0):
            for chi in range(2):
                ref = _operators(Ns, m0, omega, mu, chi)
                for d, name in enumerate(NAMES):
                    M, u, w = tab[d, chi, :256].reshape(N, N), tab[d, chi, 256:272], tab[d, chi, 272:]
                    rho = -mu / (1 - mu * q[d, chi])
                    for b in range(0, N, Ns):
                        own = slice(b, b + Ns)
                        got = M[own, own] + rho * np.outer(u[own], w[own])
                        # (the reference goes through general inverses)
                        assert np.abs(got - ref[name]).max() <= 1e-12 * np.abs(ref[name]).max(), (name, mu, chi)
                    blocks = np.kron(np.eye(N // Ns), np.ones((Ns, Ns)))
                    assert not M[blocks == 0].any()


# row of a result register, and the (set, real) that an operand row stands for
LAYOUT = {np.float32: (lambda g, v: 4 * g + v, lambda row: (row >> 2, row & 3)),
          np.float64: (lambda g, v: 4 * v + g, lambda row: (row & 3, row >> 2))}


def _mfma(a, b, c):
    """16 x 16 x 4: operands hold row (column) lane % 16, element lane / 16."""
    return c + a.reshape(4, 16).T @ b.reshape(4, 16)


@pytest.mark.parametrize("real", [np.float32, np.float64])
@pytest.mark.parametrize("Ns", [4, 8, 16])
def test_wave_mapping(Ns, real):
    """24 reals of 64 lanes through three groups of five matrix instructions a
    chirality, and back in the lanes and registers they came from."""
    result_row, meaning = LAYOUT[real]
    rng = np.random.default_rng(5)
    tab, q = _tables(Ns, 1.3, odwf.zolotarev_omega(Ns, 0.05, 6.2))
    y = rng.standard_normal((64, 24))
    mu = np.repeat(rng.uniform(0, 1, 64 // Ns), Ns)  # a column's right-hand side
    lane = np.arange(64)
    slot, k = lane % 16, lane // 16
    out = np.full_like(y, np.nan)
    for chi in range(2):
        M, u, w = tab[0, chi, :256].reshape(N, N), tab[0, chi, 256:272], tab[0, chi, 272:]
        rho = -mu / (1 - mu * q[0, chi])
        lds = y[:, 12 * chi:12 * chi + 12].reshape(4, 16, 12)  # set, slot, real
        for g in range(3):
            st, re = np.array([meaning(s) for s in slot]).T
            x = [lds[st, 4 * k + e, 4 * g + re] for e in range(4)]
            d = np.zeros((16, 16))
            for e in range(4):
                d = _mfma(x[e], M[slot, 4 * k + e], d)
            t = sum(w[4 * k + e] * x[e] for e in range(4)) * rho[16 * st + 4 * k]
            d = _mfma(t, np.where(slot // Ns == 4 * k // Ns, u[slot], 0.0), d)
            for v in range(4):
                out[lane, 12 * chi + 4 * g + v] = d[result_row(k, v), slot]
    for c0 in range(0, 64, Ns):
        for chi in range(2):
            ref = _operators(Ns, 1.3, odwf.zolotarev_omega(Ns, 0.05, 6.2), mu[c0], chi)["AINV"]
            col = slice(12 * chi, 12 * chi + 12)
            assert np.allclose(out[c0:c0 + Ns, col], ref @ y[c0:c0 + Ns, col], rtol=0, atol=1e-12)
