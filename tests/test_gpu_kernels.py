"""The kernels' own edges, against the FP64 CPU oracle: remainders of the layout
tiles and of the dense fifth-dimension programs, the limits at which a launch
changes kernel (four-wave hops, half blocks along an x-row, the CG scalars formed
inside the vector step, the looping launch of a wide batch engine's updates) and
the ragged blocks of the force.

Bounds: FP64 operators 1e-12 relative (rounding order only, up to four hops and
five fifth-dimension programs of 16 or 32 terms); reduced precisions as in
test_gpu_parity; solutions by the residual their tolerance asks for."""
import numpy as np
import pytest

from oracle import oracle
from paper_1811_08095_amd import odwf, synth

pytestmark = pytest.mark.gpu

M0 = 1.3
PREC_BOUND = {odwf.FP64: 1e-12, odwf.FP32: 1e-5, odwf.FP16S: 4e-3, odwf.BF16S: 3e-2}


def _mk(dims, Ns, seed, bc=-1, eps=0.5):
    U = synth.make_gauge(dims, eps, seed)
    w = odwf.zolotarev_omega(Ns, 0.05, 6.2)
    lat = odwf.Lattice(dims, bc_t=bc)
    lat.load_gauge(U)
    return U, w, lat, odwf.Solver(lat, Ns, M0, w)


def _rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


# half-row lengths 1 .. 12 (row segments, half blocks, linear), tiles of sites that
# end inside a block, one to four right-hand sides of different masses
DENSE = [((2, 2, 2, 2), 4, 1, 1), ((6, 2, 2, 4), 4, 3, -1), ((10, 2, 4, 2), 8, 2, -1), ((4, 6, 2, 6), 8, 1, 1),
         ((16, 2, 4, 6), 16, 1, -1), ((6, 10, 2, 4), 16, 3, 1), ((24, 4, 2, 2), 16, 1, -1), ((8, 4, 4, 2), 16, 4, -1),
         ((6, 2, 2, 4), 32, 2, -1)]


@pytest.mark.parametrize("prec", sorted(PREC_BOUND))
@pytest.mark.parametrize("case", DENSE, ids=lambda c: "x".join(map(str, c[0])) + f"_Ns{c[1]}_r{c[2]}")
def test_operators_at_tile_edges(case, prec):
    import torch
    dims, Ns, n, bc = case
    U, w, lat, sol = _mk(dims, Ns, 11, bc)
    psi = synth.make_source(dims, Ns, n, 4100)
    masses = [0.02, 0.9, 0.3, 0.05][:n]
    for op in (odwf.OP_D, odwf.OP_DDAG, odwf.OP_SCHUR_NORMAL):
        print(f"op {op} {dims} Ns={Ns} r={n} prec={prec}", flush=True)
        out = sol.apply(op, torch.from_numpy(psi).cuda(), masses, prec=prec).cpu().numpy()
        for r in range(n):
            ref = oracle.apply(op, U, psi[r], M0, w, masses[r] / (2 * M0), bc)
            assert _rel(out[r], ref) <= PREC_BOUND[prec], (op, r)
    sol.close()
    lat.close()


# (lattice, right-hand sides): 512 partial sums and the first launch above, the last
# launch of the four-wave kernel in FP64 (768 blocks) and the first above, the same
# in FP32 (1024); three right-hand sides leave 16 lanes of a wave idle, five are
# too many for it
SMALL = [((8, 8, 8, 8), 1), ((8, 8, 8, 10), 1), ((8, 8, 8, 12), 1), ((8, 8, 8, 14), 1), ((8, 8, 8, 16), 1), ((8, 8, 8, 18), 1), ((4, 4, 4, 16), 3), ((8, 4, 8, 4), 4), ((4, 4, 4, 4), 5)]


@pytest.mark.parametrize("prec", [odwf.FP64, odwf.FP32])
@pytest.mark.parametrize("dims,n", SMALL, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else f"r{v}")
def test_small_launches(dims, n, prec):
    """Operator and solve on both sides of the limits, the partial sums read by the
    vector step (at most 512) and by a launch of their own."""
    import torch
    Ns = 16
    U, w, lat, sol = _mk(dims, Ns, 12)
    b = synth.make_source(dims, Ns, n, 4200)
    masses = [0.3 + 0.1 * r for r in range(n)]
    dev = torch.from_numpy(b).cuda()
    print(f"small {dims} r={n} prec={prec}", flush=True)
    out = sol.apply(odwf.OP_SCHUR_NORMAL, dev, masses, prec=prec).cpu().numpy()
    for r in range(n):
        ref = oracle.apply(odwf.OP_SCHUR_NORMAL, U, b[r], M0, w, masses[r] / (2 * M0), -1)
        assert _rel(out[r], ref) <= PREC_BOUND[prec], r
    x, st = sol.solve(dev, masses, [1e-9] * n, inner=prec)
    for r in range(n):
        assert st[r]["status"] == odwf.OK and st[r]["true_rel_resid"] <= 1e-9
        Dx = oracle.apply(oracle.OP_D, U, x[r].cpu().numpy(), M0, w, masses[r] / (2 * M0), -1)
        assert _rel(Dx, b[r]) <= 1e-6
    # a second solve reads none of the first one's scalars or partial sums
    y, _ = sol.solve(dev, masses, [1e-9] * n, inner=prec)
    assert torch.equal(x, y)
    sol.close()
    lat.close()


def test_wide_batch_updates():
    """Twelve slots on 1024 blocks: the gated FP64 updates loop over the sites.
    Every slot meets its own tolerance, and a slot's solution is the same bits
    with the others idle."""
    import torch
    dims, Ns, k = (8, 8, 4, 8), 16, 12
    U, w, lat, sol = _mk(dims, Ns, 13)
    srcs = synth.make_source(dims, Ns, 3, 4300)
    dev = [torch.from_numpy(s).cuda().contiguous() for s in srcs]
    masses, tols = [0.2, 0.6, 0.35], [1e-10, 1e-8, 1e-9]

    def run(which):
        bt = odwf.Batch(sol, k, inner=odwf.FP32)
        slots = {i: bt.admit(dev[i], masses[i], tols[i]) for i in which}
        for _ in range(200):
            bt.step(8)
            if all(bt.poll(q)[0] for q in slots.values()):
                break
        out = {}
        for i, q in slots.items():
            x = torch.zeros_like(dev[i])
            st = bt.retire(q, x)
            assert st["status"] == odwf.OK and st["true_rel_resid"] <= tols[i], i
            out[i] = x
        return out

    print(f"batch {dims} k={k}", flush=True)
    mixed = run([0, 1, 2])
    for i, x in mixed.items():
        Dx = oracle.apply(oracle.OP_D, U, x.cpu().numpy(), M0, w, masses[i] / (2 * M0))
        assert _rel(Dx, srcs[i]) <= 1e3 * tols[i], i
    assert torch.equal(run([0])[0], mixed[0])


# (lattice, N_s, slots, inner): the gated updates in one span of blocks that walk on
# their own (up to eight spans: 4096 blocks of 256 threads) and in pairs above, with
# a last pair that is not whole; blocks of 128, 192 and 256 threads
LOOPING = [((8, 8, 8, 8), 4, 16, odwf.FP32), ((6, 8, 8, 8), 8, 12, odwf.FP64), ((8, 8, 8, 12), 16, 12, odwf.FP64),
           ((8, 8, 8, 18), 32, 6, odwf.FP32), ((10, 8, 10, 12), 16, 12, odwf.FP32), ((8, 12, 16, 16), 16, 1, odwf.FP64),
           ((16, 16, 8, 10), 8, 16, odwf.FP32)]


@pytest.mark.parametrize("dims,Ns,k,inner", LOOPING, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_looping_updates(dims, Ns, k, inner):
    """A slot's solution meets its tolerance, and is the same bits beside others."""
    import torch
    U, w, lat, sol = _mk(dims, Ns, 16)
    b = synth.make_source(dims, Ns, 1, 4600)[0]
    dev = torch.from_numpy(b).cuda().contiguous()
    other = torch.from_numpy(synth.make_source(dims, Ns, 1, 4601)[0]).cuda().contiguous()

    def run(mixed):
        bt = odwf.Batch(sol, k, inner=inner)
        q = bt.admit(dev, 0.4, 1e-9)
        if mixed:
            bt.step(3)
            bt.admit(other, 0.9, 1e-7)
        for _ in range(200):
            bt.step(8)
            if bt.poll(q)[0]:
                break
        x = torch.zeros_like(dev)
        st = bt.retire(q, x)
        assert st["status"] == odwf.OK and st["true_rel_resid"] <= 1e-9
        return x

    print(f"looping {dims} Ns={Ns} k={k} inner={inner}", flush=True)
    x = run(False)
    Dx = oracle.apply(oracle.OP_D, U, x.cpu().numpy(), M0, w, 0.4 / (2 * M0))
    assert _rel(Dx, b) <= 1e-6
    assert k == 1 or torch.equal(run(True), x)
    sol.close()
    lat.close()


# rows shorter and longer than a block's 16 sites, rows that end inside a block, a
# ragged last block, planes that are no whole number of blocks
FORCE = [((10, 2, 2, 4), 4, -1), ((18, 2, 4, 2), 8, 1), ((34, 2, 2, 2), 4, -1), ((6, 6, 2, 4), 4, -1),
         ((16, 4, 8, 4), 4, -1), ((8, 8, 2, 6), 8, 1)]


@pytest.mark.parametrize("dims,Ns,bc", FORCE, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_force_block_edges(dims, Ns, bc):
    import torch
    U, w, lat, sol = _mk(dims, Ns, 14, bc)
    chi, psi = synth.make_source(dims, Ns, 2, 4400)
    print(f"force {dims} Ns={Ns} bc={bc}", flush=True)
    F = sol.force(torch.from_numpy(chi).cuda(), torch.from_numpy(psi).cuda()).cpu().numpy()
    ref = oracle.force(U, chi, psi, bc)
    assert _rel(F, ref) <= 1e-12
    per = np.linalg.norm((F - ref).reshape(-1, 9), axis=1).max() / np.linalg.norm(ref.reshape(-1, 9), axis=1).max()
    assert per <= 1e-12
    sol.close()
    lat.close()


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("where", ["chi end", "psi end", "psi start"])
def test_force_into_its_inputs(where, accumulate):
    """F that starts inside chi or psi, or ends inside psi: as if it lay apart.
    Blocks enough that some still read when others have written."""
    import torch
    dims, Ns = (16, 8, 8, 8), 4
    U, w, lat, sol = _mk(dims, Ns, 15)
    V = int(np.prod(dims))
    nf, nF = Ns * V * 12, V * 36
    buf = torch.from_numpy(synth.make_source(dims, Ns, 3, 4500)).cuda().reshape(-1)
    # [chi | psi | rest] with F over the end of chi and the start of psi, or the end of psi
    at = {"chi end": nf - nF // 2, "psi end": 2 * nf - nF + 12, "psi start": nf - nF + 12}[where]
    chi, psi, F = buf[:nf], buf[nf:2 * nf], buf[at:at + nF]
    shape, fshape = sol.spinor_shape(1), lat.shape_tzyx + (4, 3, 3)
    F0, chi0, psi0 = F.clone().view(fshape), chi.clone().view(shape), psi.clone().view(shape)
    ref = sol.force(chi0, psi0, F=F0, accumulate=accumulate)
    out = sol.force(chi.view(shape), psi.view(shape), F=F.view(fshape), accumulate=accumulate)
    assert torch.equal(out, ref)
    sol.close()
    lat.close()
