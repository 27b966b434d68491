"""The fermion-force kernel (odwf_force) against the FP64 CPU oracle, link by
link: F_mu(x) = TA(U_mu(x) M_mu(x)) of Re <chi, W psi>, the derivative the
oracle's force is pinned to (tests/test_oracle_force.py).  FP64 bar: normwise
and per link <= 1e-12 relative.  Lattices cover the 2^4 aliasing case, non-cubic
extents, a ragged final block, both time boundary conditions and Ns 4 .. 32;
accumulation sums two bilinears."""
import numpy as np
import pytest

from oracle import oracle
from paper_1811_08095_amd import odwf, synth

pytestmark = pytest.mark.gpu

M0 = 1.3
CASES = [((2, 2, 2, 2), 4, -1, 3), ((4, 2, 6, 4), 8, 1, 5), ((6, 2, 2, 2), 16, -1, 7),
         ((4, 4, 4, 4), 16, -1, 0), ((2, 4, 2, 6), 32, 1, 9)]


def _rel(a, b):
    per = np.linalg.norm((a - b).reshape(-1, 9), axis=1).max() / np.linalg.norm(b.reshape(-1, 9), axis=1).max()
    return np.linalg.norm(a - b) / np.linalg.norm(b), per


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c[0])) + f"_Ns{c[1]}_bc{c[2]}")
def test_force_matches_oracle(case):
    import torch
    dims, Ns, bc, seed = case
    U = synth.make_gauge(dims, 0.6, seed)
    lat = odwf.Lattice(dims, bc_t=bc)
    lat.load_gauge(U)
    sol = odwf.Solver(lat, Ns, M0, odwf.zolotarev_omega(Ns))
    chi = synth.make_source(dims, Ns, 2, 500 + seed)
    psi = synth.make_source(dims, Ns, 2, 600 + seed)
    print(f"force {dims} Ns={Ns} bc={bc}", flush=True)
    F = sol.force(torch.from_numpy(chi[0]).cuda(), torch.from_numpy(psi[0]).cuda()).cpu().numpy()
    ref = oracle.force(U, chi[0], psi[0], bc)
    en, ep = _rel(F, ref)
    print(f"  normwise {en:.2e}, per link {ep:.2e}")
    assert en <= 1e-12 and ep <= 1e-12
    # a second bilinear added to the first
    Fd = torch.from_numpy(F).cuda()
    sol.force(torch.from_numpy(chi[1]).cuda(), torch.from_numpy(psi[1]).cuda(), F=Fd, accumulate=True)
    ref2 = ref + oracle.force(U, chi[1], psi[1], bc)
    en2, ep2 = _rel(Fd.cpu().numpy(), ref2)
    assert en2 <= 1e-12 and ep2 <= 1e-12
    sol.close()
    lat.close()


def test_force_argument_errors():
    import torch
    dims = (2, 2, 2, 2)
    lat = odwf.Lattice(dims)
    lat.load_gauge(synth.make_gauge(dims, 0.3, 0))
    sol = odwf.Solver(lat, 4, M0, odwf.zolotarev_omega(4))
    chi = torch.from_numpy(synth.make_source(dims, 4, 1, 1)).cuda()
    with pytest.raises(ValueError):
        sol.force(chi, torch.zeros((2, 4, 2, 2, 2, 2, 4, 3), dtype=torch.complex128, device="cuda"))
    with pytest.raises(odwf.OdwfError) as e:
        odwf._check(odwf.lib().odwf_force(sol._h, odwf._dev_ptr(chi, "chi"), odwf._dev_ptr(chi, "psi"), 0,
                                          odwf._dev_ptr(chi, "F"), odwf._stream(None)))
    assert e.value.status == odwf.EINVAL
    sol.close()
    lat.close()


def force_extended(U, chi, psi, bc):
    """F in extended precision (64-bit mantissa) from the definition in the header."""
    s2 = [np.array([[0, 1], [1, 0]]), np.array([[0, -1j], [1j, 0]]), np.array([[1, 0], [0, -1]])]
    zero = np.zeros((2, 2))
    gam = [np.block([[zero, -1j * s], [1j * s, zero]]) for s in s2] + [np.block([[zero, np.eye(2)], [np.eye(2), zero]])]
    U, chi, psi = (np.asarray(v, np.clongdouble) for v in (U, chi, psi))
    F = np.zeros_like(U)
    for mu in range(4):
        ax = 4 - mu  # of [s][t][z][y][x]
        pf, cf = np.roll(psi, -1, ax), np.roll(chi, -1, ax)
        hop = lambda v, sg: np.einsum("ab,...bc->...ac", (np.eye(4) + sg * gam[mu]).astype(np.clongdouble), v)
        A = np.einsum("s...ab,s...ac->...bc", hop(pf, -1), chi.conj())
        B = np.einsum("s...ab,s...ac->...bc", hop(psi, +1), cf.conj())
        M = -(A + B.conj().swapaxes(-1, -2)) / 2
        if mu == 3 and bc < 0:
            M[-1] = -M[-1]
        X = np.einsum("...ab,...bc->...ac", U[..., mu, :, :], M)
        X = (X - X.conj().swapaxes(-1, -2)) / 2
        F[..., mu, :, :] = X - np.einsum("...aa->...", X)[..., None, None] * np.eye(3) / 3
    return F


def test_force_rounds_once_a_slice():
    """16 slices: an entry's eight products of a slice are summed before they join the
    sum over slices.  With independent roundings of 0.4 u rms (u = 2^-53), spinors and
    links of independent Gaussians, the error is 1.65 u of the force for this order
    and 2.55 u for one running sum of all 128 products; the bound lies between."""
    import torch
    dims, Ns, bc = (8, 4, 4, 4), 16, -1
    U = synth.make_gauge(dims, 0.6, 11)
    chi, psi = synth.make_source(dims, Ns, 2, 700)
    ref = force_extended(U, chi, psi, bc)
    assert _rel(oracle.force(U, chi, psi, bc), ref)[0] <= 1e-15
    lat = odwf.Lattice(dims, bc_t=bc)
    lat.load_gauge(U)
    sol = odwf.Solver(lat, Ns, M0, odwf.zolotarev_omega(Ns))
    F = sol.force(torch.from_numpy(chi).cuda(), torch.from_numpy(psi).cuda()).cpu().numpy()
    err = float(np.linalg.norm((F - ref).ravel()) / np.linalg.norm(ref.ravel())) / 2.0 ** -53
    print(f"force error {err:.2f} u")
    assert err <= 2.1
    sol.close()
    lat.close()
