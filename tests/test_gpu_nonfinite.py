"""Non-finite values stay in their own column (site, right-hand side).

At N_s = 4 and 8 several columns share an operand row of the matrix
instructions, separated by zeros of the matrix; 0 * NaN and 0 * Inf must not
carry one right-hand side or site into another.  A good right-hand side beside
a bad one gives the same bits as beside a source of zeros (same launches, so
the same order of every sum), in every precision.
"""
import numpy as np
import pytest

from paper_1811_08095_amd import odwf, synth

pytestmark = pytest.mark.gpu

M0 = 1.3
DIMS = (4, 4, 2, 4)
PRECS = [odwf.FP64, odwf.FP32, odwf.FP16S, odwf.BF16S]
# finite values whose products leave the range of the arithmetic, in every component of a site
HUGE = {odwf.FP64: 1.5e308, odwf.FP32: 3e38, odwf.FP16S: 3e38, odwf.BF16S: 3e38}


def _mk(Ns):
    lat = odwf.Lattice(DIMS, bc_t=-1)
    lat.load_gauge(synth.make_gauge(DIMS, 0.5, 21))
    return lat, odwf.Solver(lat, Ns, M0, odwf.zolotarev_omega(Ns, 0.05, 6.2))


def _spoil(b, kind, prec):
    """One component of one site (all of the site for huge finite values)."""
    if kind == "huge":
        b[:, 1, 1, 2, 2] = HUGE[prec]
    else:
        b[1, 1, 1, 2, 2, 1, 1] = {"nan": np.nan, "inf": np.inf}[kind]


@pytest.mark.parametrize("kind", ["nan", "inf", "huge"])
@pytest.mark.parametrize("prec", PRECS, ids=lambda p: odwf.PREC_NAMES[p])
@pytest.mark.parametrize("Ns", [4, 8, 16, 32])
def test_applications_keep_right_hand_sides_apart(Ns, prec, kind):
    import torch
    lat, sol = _mk(Ns)
    for n, bad in ((2, 0), (3, 1)):
        psi = synth.make_source(DIMS, Ns, n, 5100)
        psi[bad] = 0
        masses = [0.02, 0.9, 0.3][:n]
        good = [r for r in range(n) if r != bad]
        spoiled = psi.copy()
        _spoil(spoiled[bad], kind, prec)
        for op in range(odwf.OP_HOP_EO, odwf.OP_SCHUR_NORMAL + 1):
            print(f"Ns={Ns} prec={prec} {kind} op={op} n={n}", flush=True)
            ref = sol.apply(op, torch.from_numpy(psi).cuda(), masses, prec=prec).cpu().numpy()
            out = sol.apply(op, torch.from_numpy(spoiled).cuda(), masses, prec=prec).cpu().numpy()
            for r in good:
                assert np.isfinite(ref[r]).all()
                assert np.array_equal(out[r], ref[r]), (op, n, r)
    sol.close()
    lat.close()


@pytest.mark.parametrize("prec", PRECS, ids=lambda p: odwf.PREC_NAMES[p])
@pytest.mark.parametrize("Ns", [4, 8, 16])
def test_singular_mass_stays_alone(Ns, prec):
    """mu = -1 makes 1 + L singular: that right-hand side alone is not finite."""
    import torch
    lat, sol = _mk(Ns)
    psi = torch.from_numpy(synth.make_source(DIMS, Ns, 3, 5150)).cuda()
    for op in (odwf.OP_D, odwf.OP_DDAG, odwf.OP_SCHUR_NORMAL):
        ref = sol.apply(op, psi, [0.3, 0.5, 0.02], prec=prec).cpu().numpy()
        out = sol.apply(op, psi, [0.3, -2 * M0, 0.02], prec=prec).cpu().numpy()
        assert np.isfinite(ref).all() and not np.isfinite(out[1]).all()
        assert np.array_equal(out[[0, 2]], ref[[0, 2]]), op
    sol.close()
    lat.close()


@pytest.mark.parametrize("prec", [odwf.FP64, odwf.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("Ns", [4, 8])
def test_large_values_are_applied(Ns, prec):
    """Finite values near the end of the range: A^{-1} is linear, and scales exactly."""
    import torch
    lat, sol = _mk(Ns)
    psi = synth.make_source(DIMS, Ns, 2, 5160)
    f = 2.0 ** (1015 if prec == odwf.FP64 else 119)
    big = psi.copy()
    big[0] *= f
    ref = sol.apply(odwf.OP_M5INV, torch.from_numpy(psi).cuda(), [0.3, 0.1], prec=prec).cpu().numpy()
    out = sol.apply(odwf.OP_M5INV, torch.from_numpy(big).cuda(), [0.3, 0.1], prec=prec).cpu().numpy()
    assert np.array_equal(out[0], ref[0] * f) and np.array_equal(out[1], ref[1])
    sol.close()
    lat.close()


@pytest.mark.parametrize("kind", ["nan", "inf", "huge"])
@pytest.mark.parametrize("prec", PRECS, ids=lambda p: odwf.PREC_NAMES[p])
@pytest.mark.parametrize("Ns", [4, 8, 16, 32])
def test_site_local_operator_keeps_sites_apart(Ns, prec, kind):
    """A^{-1} acts on each site alone: only the bad site's outputs change."""
    import torch
    lat, sol = _mk(Ns)
    psi = synth.make_source(DIMS, Ns, 1, 5200)
    spoiled = psi.copy()
    _spoil(spoiled[0], kind, prec)
    ref = sol.apply(odwf.OP_M5INV, torch.from_numpy(psi).cuda(), [0.3], prec=prec).cpu().numpy()[0]
    out = sol.apply(odwf.OP_M5INV, torch.from_numpy(spoiled).cuda(), [0.3], prec=prec).cpu().numpy()[0]
    assert kind == "huge" or not np.isfinite(out[:, 1, 1, 2, 2]).all()
    out[:, 1, 1, 2, 2] = ref[:, 1, 1, 2, 2]
    assert np.array_equal(out, ref)
    sol.close()
    lat.close()


@pytest.mark.parametrize("kind", ["nan", "inf"])
@pytest.mark.parametrize("prec", PRECS, ids=lambda p: odwf.PREC_NAMES[p])
@pytest.mark.parametrize("Ns", [4, 8, 16])
def test_solves_keep_right_hand_sides_apart(Ns, prec, kind):
    import torch
    lat, sol = _mk(Ns)
    b = synth.make_source(DIMS, Ns, 3, 5300)
    b[1] = 0
    masses, tols = [0.3, 0.5, 0.4], [1e-9] * 3
    spoiled = b.copy()
    _spoil(spoiled[1], kind, prec)
    print(f"solve Ns={Ns} prec={prec} {kind}", flush=True)
    ref, st0 = sol.solve(torch.from_numpy(b).cuda(), masses, tols, inner=prec)
    out, st = sol.solve(torch.from_numpy(spoiled).cuda(), masses, tols, inner=prec, raise_on_noconv=False)
    assert st[1]["status"] == odwf.ENAN
    for r in (0, 2):
        assert st[r]["status"] == odwf.OK and st[r]["true_rel_resid"] <= 1e-9, r
        assert st[r]["iters"] == st0[r]["iters"]
        assert torch.equal(out[r], ref[r]), r
    sol.close()
    lat.close()


@pytest.mark.parametrize("inner", [odwf.FP64, odwf.FP32], ids=["fp64", "fp32"])
@pytest.mark.parametrize("Ns", [4, 8])
def test_batch_keeps_slots_apart(Ns, inner):
    """A slot whose source is not finite fails alone."""
    import torch
    lat, sol = _mk(Ns)
    srcs = synth.make_source(DIMS, Ns, 2, 5400)
    dev = [torch.from_numpy(s).cuda().contiguous() for s in srcs]
    bad = dev[1].clone()
    bad[1, 1, 1, 2, 2, 1, 1] = float("nan")

    def run(with_bad):
        bt = odwf.Batch(sol, 3, inner=inner)
        if with_bad:
            q0 = bt.admit(bad, 0.5, 1e-9)
            assert bt.poll(q0)[1]["status"] == odwf.ENAN
        q = bt.admit(dev[0], 0.3, 1e-9)
        for _ in range(200):
            bt.step(8)
            if bt.poll(q)[0]:
                break
        x = torch.zeros_like(dev[0])
        assert bt.retire(q, x)["status"] == odwf.OK
        return x

    assert torch.equal(run(True), run(False))
    sol.close()
    lat.close()
