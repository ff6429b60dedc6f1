"""Parity of the leapfrog driver (nbody_leapfrog_kdk: Move_bodies after the
force calculation, Section IV.B, as kick-drift-kick) and of its HIP-graph
capture with the oracle and with eager launches."""
import numpy as np
import pytest

import ics
from nbtest import gpu, host, rms_rel, to_dev, widen32

pytestmark = pytest.mark.gpu


def test_ball4096_f64_ten_steps(orc):
    """One force evaluation then 10 KDK steps, dt = 1e-3, FP64: <= 1e-12."""
    torch, nb = gpu()
    w = ics.WORKLOADS["ball4096_f64"]
    pm, v = ics.uniform_ball(w["n"], w["seed"])
    p = to_dev(torch, pm, torch.float64)
    vv = to_dev(torch, v, torch.float64)
    a = torch.empty_like(p)
    en = nb.leapfrog_kdk(p, vv, a, w["eps"], w["dt"], w["steps"], energy=True)
    torch.cuda.synchronize()
    ref = orc.leapfrog(pm, v, w["eps"], w["dt"], w["steps"])
    assert rms_rel(host(p)[:, :3], ref["x"]) <= 1e-12
    assert rms_rel(host(vv)[:, :3], ref["v"]) <= 1e-12
    assert rms_rel(host(a)[:, :3], ref["acc"]) <= 1e-12
    assert rms_rel(host(a)[:, 3], ref["pot"]) <= 1e-12
    e = en.cpu().numpy()
    assert e[0, 0] == 0.0
    np.testing.assert_allclose(e[:, 1], ref["energy"][:, 1], rtol=1e-12)
    np.testing.assert_allclose(e[1:, 0], ref["energy"][1:, 0], rtol=1e-10)


@pytest.mark.parametrize("mode", ["F32_KAHAN", "F32_F64ACC", "F32"])
def test_f32_modes_few_steps(orc, mode):
    torch, nb = gpu()
    pm, v = ics.plummer(8192, 50)
    p = to_dev(torch, pm, torch.float32)
    vv = to_dev(torch, v, torch.float32)
    a = torch.empty_like(p)
    en = nb.leapfrog_kdk(p, vv, a, 0.01, 1e-3, 5, prec=getattr(nb, mode), energy=True)
    torch.cuda.synchronize()
    ref = orc.leapfrog(widen32(pm), widen32(v), 0.01, 1e-3, 5)
    assert rms_rel(host(p)[:, :3], ref["x"]) <= 1e-6
    # force at the GPU's own final state
    acc, pot = orc.accel(host(p), 0.01, targets=np.arange(0, 8192, 8))
    assert rms_rel(host(a)[::8, :3], acc) <= (1e-4 if mode == "F32" else 1e-5)
    e = en.cpu().numpy().sum(axis=1)
    assert abs(e[-1] / e[0] - 1) < 1e-5


def test_kepler_orbit_on_gpu():
    """Circular Kepler pair (period 2 pi), FP64: back at the start after one
    period to O(dt^2)."""
    torch, nb = gpu()
    pm, v = ics.kepler_pair(0.0)
    for nstep, tol in [(400, 2e-3), (800, 5e-4)]:
        p = to_dev(torch, pm, torch.float64)
        vv = to_dev(torch, v, torch.float64)
        a = torch.empty_like(p)
        nb.leapfrog_kdk(p, vv, a, 0.0, 2 * np.pi / nstep, nstep)
        torch.cuda.synchronize()
        assert np.abs(host(p)[:, :3] - pm[:, :3]).max() < tol


@pytest.mark.parametrize("mode", ["F32_KAHAN", "F64"])
def test_graph_replays_match_eager(mode):
    """Captured step loop == eager launches, bitwise, on every replay, with
    eager work and synchronisation between replays."""
    torch, nb = gpu()
    dtype = torch.float64 if mode == "F64" else torch.float32
    prec = getattr(nb, mode)
    pm, v = ics.plummer(3000, 51)
    pg, vg = to_dev(torch, pm, dtype), to_dev(torch, v, dtype)
    pe, ve = pg.clone(), vg.clone()
    ag, ae = torch.empty_like(pg), torch.empty_like(pe)
    eg = torch.empty((8, 2), dtype=torch.float64, device="cuda")
    ee = torch.empty_like(eg)
    for rep in range(4):
        nb.leapfrog_kdk(pg, vg, ag, 0.01, 1e-3, 7, prec=prec, graph=True, energy=True, energy_out=eg)
        torch.cuda.synchronize()
        junk = torch.randn(1000, device="cuda").sum()  # unrelated eager work
        nb.leapfrog_kdk(pe, ve, ae, 0.01, 1e-3, 7, prec=prec, graph=False, energy=True, energy_out=ee)
        torch.cuda.synchronize()
        assert torch.equal(pg, pe) and torch.equal(vg, ve) and torch.equal(ag, ae), rep
        assert torch.equal(eg, ee), rep
        del junk


def test_acc_valid_flag_skips_first_evaluation():
    torch, nb = gpu()
    pm, v = ics.plummer(2000, 52)
    p1, v1 = to_dev(torch, pm, torch.float32), to_dev(torch, v, torch.float32)
    p2, v2 = p1.clone(), v1.clone()
    a1, a2 = torch.empty_like(p1), torch.empty_like(p1)
    nb.leapfrog_kdk(p1, v1, a1, 0.01, 1e-3, 6)
    nb.leapfrog_kdk(p2, v2, a2, 0.01, 1e-3, 3)
    nb.leapfrog_kdk(p2, v2, a2, 0.01, 1e-3, 3, acc_valid=True)
    torch.cuda.synchronize()
    assert torch.equal(p1, p2) and torch.equal(v1, v2) and torch.equal(a1, a2)


@pytest.mark.parametrize("steps", [0, 1, 62, 63, 64, 130])
def test_energies_of_many_steps(steps):
    """The energies of up to 64 states wait for one reduction launch: around
    that count, each equals nbody_energy on the state that steps taken one at
    a time reach, bit for bit."""
    torch, nb = gpu()
    pm, v = ics.plummer(700, 53)
    p1, v1 = to_dev(torch, pm, torch.float32), to_dev(torch, v, torch.float32)
    p2, v2 = p1.clone(), v1.clone()
    a1, a2 = torch.empty_like(p1), torch.empty_like(p1)
    en = nb.leapfrog_kdk(p1, v1, a1, 0.01, 1e-3, steps, energy=True)
    nb.leapfrog_kdk(p2, v2, a2, 0.01, 1e-3, 0, energy=True)
    ref = [nb.energy(p2, v2, a2)]
    for _ in range(steps):
        nb.leapfrog_kdk(p2, v2, a2, 0.01, 1e-3, 1, acc_valid=True, energy=True)
        ref.append(nb.energy(p2, v2, a2))
    torch.cuda.synchronize()
    assert torch.equal(p1, p2) and torch.equal(v1, v2)
    assert torch.equal(en, torch.stack(ref))


@pytest.mark.parametrize("n", [527, 4096, 4097])
@pytest.mark.parametrize("steps", [62, 63, 64, 130])
@pytest.mark.parametrize("given", [False, True])
def test_energies_of_many_fused_steps(n, steps, given):
    """The same for FP64 runs whose step is fused with the force (up to 4096
    bodies), which leave rows' sums: from a computed force and from a given
    one, whose first state comes from the step kernel and is reduced by
    itself, before, at and past the 64 states of one reduction."""
    torch, nb = gpu()
    pm, v = ics.plummer(n, 59)
    p1, v1 = to_dev(torch, pm, torch.float64), to_dev(torch, v, torch.float64)
    p2, v2 = p1.clone(), v1.clone()
    a2 = nb.accel(p2, 0.01)
    a1 = a2.clone() if given else torch.empty_like(p1)
    en = nb.leapfrog_kdk(p1, v1, a1, 0.01, 1e-3, steps, energy=True, acc_valid=given)
    ref = [nb.energy(p2, v2, a2)]
    for _ in range(steps):
        nb.leapfrog_kdk(p2, v2, a2, 0.01, 1e-3, 1, acc_valid=True)
        ref.append(nb.energy(p2, v2, a2))
    torch.cuda.synchronize()
    assert torch.equal(p1, p2) and torch.equal(v1, v2) and torch.equal(a1, a2)
    assert torch.equal(en, torch.stack(ref))


@pytest.mark.parametrize("mode,n", [("F32_KAHAN", 511), ("F32_KAHAN", 512), ("F32", 513), ("F32_F64ACC", 8192),
                                    ("F64", 527), ("F64", 4096)])
@pytest.mark.parametrize("steps", [1, 2, 5])
def test_fused_small_steps(mode, n, steps):
    """Small problems step in the force's launch, the positions going back and
    forth between two buffers: odd and even counts of steps, from a given and
    from a computed force, equal force and kick_drift by hand bit for bit, and
    so do energies and graph replays with other work in between."""
    torch, nb = gpu()
    prec, eps, dt = getattr(nb, mode), 0.01, 1e-3
    dtype = torch.float64 if mode == "F64" else torch.float32
    pm, v = ics.plummer(n, 67)
    p0, v0 = to_dev(torch, pm, dtype), to_dev(torch, v, dtype)
    ph, vh = p0.clone(), v0.clone()
    ah = nb.accel(ph, eps, prec=prec)
    a0 = ah.clone()
    en = [nb.energy(ph, vh, ah)]
    for k in range(steps):
        nb.kick_drift(ph, vh, ah, dt / 2, dt, close=False, open=True, prec=prec)
        ah = nb.accel(ph, eps, prec=prec)
        nb.kick_drift(ph, vh, ah, dt / 2, dt, close=True, open=False, prec=prec)
        en.append(nb.energy(ph, vh, ah))
    for given in (False, True):
        for graph in (False, True):
            pg, vg = p0.clone(), v0.clone()
            ag = a0.clone()
            for rep in range(3 if graph else 1):
                pg.copy_(p0)
                vg.copy_(v0)
                ag.copy_(a0 if given else torch.zeros_like(a0))
                got = nb.leapfrog_kdk(pg, vg, ag, eps, dt, steps, prec=prec, acc_valid=given, graph=graph, energy=mode == "F64")
                nb.accel(p0, 2 * eps, prec=prec)
                torch.cuda.synchronize()
                assert torch.equal(pg, ph) and torch.equal(vg, vh) and torch.equal(ag, ah)
                assert mode != "F64" or torch.equal(got, torch.stack(en))


@pytest.mark.parametrize("mode", ["F32", "F32_KAHAN", "F32_F64ACC", "F64"])
@pytest.mark.parametrize("n", [300, 1987, 8192, 10007, 30001])
def test_runs_with_and_without_energies(mode, n):
    """What NBODY_ENERGY may change: nothing in FP64 or with a pinned shape;
    otherwise in FP32 the rounding of the forces, where the unpinned force is
    not the sweep (10007 bodies: it is, and nothing changes).  Bars for four
    steps: each force is within 2e-6 (RMS, as for single forces), four of them
    times dt move velocities of order 1 by under 1e-8, so what remains is a
    few roundings of the FP32 state, 4 x 2^-24; potentials, under 2e-7 each
    (a few 2^-24), bound the potential energy, and velocities the kinetic."""
    torch, nb = gpu()
    prec = getattr(nb, mode)
    dtype = torch.float64 if mode == "F64" else torch.float32
    pm, v = ics.plummer(n, 73)
    p0, v0 = to_dev(torch, pm, dtype), to_dev(torch, v, dtype)

    def run(energy):
        p, w, a = p0.clone(), v0.clone(), torch.empty_like(p0)
        en = nb.leapfrog_kdk(p, w, a, 0.01, 1e-3, 4, prec=prec, energy=energy)
        return p, w, a, (en[-1] if energy else nb.energy(p, w, a))

    nb.set_tuning(0, prec, *nb.get_tuning(0, prec, n))
    try:
        x, y = run(True), run(False)
    finally:
        nb.set_tuning(0, prec)
    torch.cuda.synchronize()
    assert all(torch.equal(b, c) for b, c in zip(x, y))
    x, y = run(True), run(False)
    torch.cuda.synchronize()
    if mode == "F64" or n == 10007:
        assert all(torch.equal(b, c) for b, c in zip(x, y))
        return
    far = [float((b.double() - c.double()).norm() / c.double().norm()) for b, c in zip(x, y)]
    assert not torch.equal(x[2], y[2])  # (the two kernels did run)
    assert far[0] <= 2.0 ** -22 and far[1] <= 2.0 ** -22 and far[2] <= 2 * 2e-6, far
    assert float(((x[3] - y[3]) / y[3]).abs().max()) <= 4e-7


def test_pairwise_records_do_not_fit():
    """Where the pairwise kernels' records (1000 MiB for 2^18 bodies) cannot be
    had, a force, a run and a captured run take the split sweep (128 MiB):
    the bits of the sweep's pinned shape.  The rest of the device's memory is
    held by another tensor meanwhile; afterwards the pairwise kernels run."""
    torch, nb = gpu()
    n, eps, dt, prec = 1 << 18, 0.01, 1e-3, nb.F32_KAHAN
    pm, v = ics.plummer(n, 71)
    p0, v0 = to_dev(torch, pm, torch.float32), to_dev(torch, v, torch.float32)
    pe, ve, ae = p0.clone(), v0.clone(), torch.empty_like(p0)
    pr, vr, ar = p0.clone(), v0.clone(), torch.empty_like(p0)
    out = torch.empty_like(p0)
    nb.set_tuning(0, prec, *nb.get_tuning(0, prec, n))
    try:
        force = nb.accel(p0, eps, prec=prec)
        nb.leapfrog_kdk(pr, vr, ar, eps, dt, 3, prec=prec)
    finally:
        nb.set_tuning(0, prec)
    torch.cuda.synchronize()
    nb.release()
    torch.cuda.empty_cache()
    held = []
    for _ in range(4):  # (memory just freed may be counted late)
        free = torch.cuda.mem_get_info()[0]
        if free > (900 << 20):
            held.append(torch.empty(free - (700 << 20), dtype=torch.uint8, device="cuda"))
    try:
        print("free MiB", torch.cuda.mem_get_info()[0] >> 20, flush=True)
        assert torch.cuda.mem_get_info()[0] < (1000 << 20)
        nb.accel(p0, eps, prec=prec, out=out)
        torch.cuda.synchronize()
        assert torch.equal(out, force)
        for graph in (False, True, True):
            pe.copy_(p0)
            ve.copy_(v0)
            nb.leapfrog_kdk(pe, ve, ae, eps, dt, 3, prec=prec, graph=graph)
            torch.cuda.synchronize()
            assert torch.equal(pe, pr) and torch.equal(ve, vr) and torch.equal(ae, ar), graph
    finally:
        del held
        nb.release()
        torch.cuda.empty_cache()
    again = nb.accel(p0, eps, prec=prec)
    torch.cuda.synchronize()
    assert not torch.equal(again, force)  # the pairwise kernels' order of summation
    nb.release()
