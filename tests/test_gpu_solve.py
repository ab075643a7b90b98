"""Parity of the HIP solve (outer reflection loop + GMRES on eq. (18)) with the oracle.

Both sides solve to tight tolerances, so the fields agree to the conditioning
of the discrete system times the tolerance: FP64 field error <= 1e-8, orders
<= 1e-9 absolute; mixed precision (FP32 Arnoldi, FP64 residual) converges to
the same FP64 solution.
"""
import time

import numpy as np
import pytest

import oracle as O
from paper_2606_25541_amd import clips

from gpu_util import device, rel, say, torch

pytestmark = pytest.mark.gpu


def small(nx, ny, nz, pol=0, theta=6.0, phi=0.0, pairs=40, L=None, t=30.0):
    layers, es = clips.mo_si_stack(pairs)
    L = L or 2.0 * nx
    return clips.Problem(nx=nx, ny=ny, nz=nz, lx_nm=L, ly_nm=2.0 * ny, t_nm=t, theta_deg=theta,
                         phi_deg=phi, pol=pol, layers=layers, eps_sub=es)


CASES = [
    ("ls16_te", (16, 16, 8), 0, 0.0, "line"),
    ("mh16_tm", (16, 8, 8), 1, 30.0, "manhattan"),
    ("mh32_te", (32, 32, 16), 0, 10.0, "manhattan"),
    ("tiny4", (4, 4, 2), 0, 0.0, "manhattan"),
]


def clip_of(kind, p):
    if kind == "line":
        return clips.line_space(p.nx, p.ny, p.nz, p.lx_nm, p.ly_nm, p.lx_nm / 4, 3 * p.lx_nm / 4)
    return clips.manhattan(p.nx, p.ny, p.nz, p.lx_nm, p.ly_nm, seed=p.nx * 7 + p.nz)


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
@pytest.mark.parametrize("prec", ["fp64", "mixed"])
@pytest.mark.parametrize("coupling", ["outer", "mono"])
def test_solve_matches_oracle(case, prec, coupling):
    from paper_2606_25541_amd import api
    dev = device()
    name, (nx, ny, nz), pol, phi, kind = case
    say("solve", name, prec, coupling)
    p = small(nx, ny, nz, pol=pol, phi=phi)
    de = clip_of(kind, p)
    ref = O.solve(p, de, rtol=1e-12)
    plan = api.Plan(p, rtol=1e-10, precision=prec, restart=20, coupling=coupling, max_outer=400)
    em, orders, info = plan.psfd_solve(torch.from_numpy(de).to(dev))
    em = em.cpu().numpy()
    orders = orders.cpu().numpy()
    say("  info", info)
    assert info["status"] == 0
    assert rel(em, ref["emask"]) < 1e-8
    assert np.max(np.abs(orders - ref["orders"])) < 1e-9
    assert info["mono_residual"] < 1e-8
    assert info["outer_iters"] >= (2 if coupling == "outer" else 1)


_REF128 = {}


def _ref_128():
    """128 x 128 x 2 (64 nm clip, TE, azimuth 20 deg) and its oracle solve, computed once:
    the oracle's outer reflection loop is slow on 128-point planes, so 6 planes
    and a 64 nm period keep it to seconds (mono residual ~5e-11)."""
    if not _REF128:
        layers, es = clips.mo_si_stack(40)
        p = clips.Problem(nx=128, ny=128, nz=2, lx_nm=64.0, ly_nm=64.0, t_nm=30.0, theta_deg=6.0,
                          phi_deg=20.0, pol=0, layers=layers, eps_sub=es)
        de = clips.manhattan(p.nx, p.ny, p.nz, p.lx_nm, p.ly_nm, seed=900)
        _REF128.update(p=p, de=de, ref=O.solve(p, de, rtol=1e-11, max_outer=40))
    return _REF128["p"], _REF128["de"], _REF128["ref"]


@pytest.mark.parametrize("jh", ["lockstep", "server"])
def test_solve_128_planes_projections_in_plane_kernel(jh, monkeypatch):
    """128 x 128 planes, mixed: the inverse square-plane kernel also forms the
    Gram-Schmidt projections (6 planes, so most partial slots are zero-filled;
    the update stays a separate pass here: the pencil blocks of a padded z
    length of 4 are too small for the Givens task).
    The solve must match the oracle, and so must the separate projection pass
    (PSFD_FUSE_DOTS=0), within one restart cycle of the same step count;
    "server" runs it through the serving path (Krylov index read per slot)."""
    from paper_2606_25541_amd import api
    dev = device()
    say("solve 128x128x2 mixed", jh)
    p, de, ref = _ref_128()
    d = torch.from_numpy(de).to(dev)

    def run():
        if jh == "lockstep":
            plan = api.Plan(p, rtol=1e-10, precision="mixed", restart=8, coupling="mono")
            return plan.psfd_solve(d)
        srv = api.Server(hbm_budget=8 << 30, max_slots=2, rtol=1e-10, precision="mixed", restart=8)
        em = torch.empty((3, p.nz, p.ny, p.nx), dtype=torch.complex128, device=dev)
        od = torch.empty((p.ny, p.nx, 3), dtype=torch.complex128, device=dev)
        t = srv.submit(p, d, em, od)
        deadline = time.perf_counter() + 60
        done = False
        while not done and time.perf_counter() < deadline:
            done, info, _ = srv.poll(t)
            time.sleep(0.002)
        srv.close()
        assert done, "served request not finished within 60 s"
        return em, od, info

    em, orders, info = run()
    say("  fused", info)
    assert info["status"] == 0
    assert rel(em.cpu().numpy(), ref["emask"]) < 1e-8
    assert np.max(np.abs(orders.cpu().numpy() - ref["orders"])) < 1e-9
    monkeypatch.setenv("PSFD_FUSE_DOTS", "0")
    em2, orders2, info2 = run()
    say("  separate pass", info2)
    assert info2["status"] == 0
    # the two paths differ only in the FP32 rounding order of the projections
    assert abs(info2["iters"] - info["iters"]) <= 8
    assert rel(em2.cpu().numpy(), ref["emask"]) < 1e-8


@pytest.mark.parametrize("n", [64, 128])
def test_update_in_forward_plane_kernel_matches_separate_pass(n, monkeypatch):
    """n x n x 32 (n = 64, 128), mixed, lock-step: the Gram-Schmidt update in the forward
    plane kernel (pencil with the Givens step, last column from the projections)
    against the separate update pass (PSFD_FUSE_UPDATE=0, the path the oracle
    parity cases run): the same solution to the solve tolerance, within one
    restart cycle of the same step count, and deterministic."""
    from paper_2606_25541_amd import api
    dev = device()
    layers, es = clips.mo_si_stack(40)
    L = 2.0 * n
    p = clips.Problem(nx=n, ny=n, nz=32, lx_nm=L, ly_nm=L, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=1, layers=layers, eps_sub=es)
    d = torch.from_numpy(clips.contact_holes(n, n, 32, L, L, 6, seed=77)).to(dev)
    say("solve %dx%dx32 mixed, update fused vs separate" % (n, n))
    plan = api.Plan(p, rtol=1e-10, precision="mixed", restart=8)
    e1, o1, i1 = plan.psfd_solve(d)
    e1b, o1b, i1b = plan.psfd_solve(d)
    monkeypatch.setenv("PSFD_FUSE_UPDATE", "0")
    e2, o2, i2 = plan.psfd_solve(d)
    say("  fused", i1, "separate", i2)
    assert i1["status"] == 0 and i2["status"] == 0
    assert torch.equal(e1, e1b) and i1 == i1b
    assert abs(i1["iters"] - i2["iters"]) <= 8
    assert rel(e1.cpu().numpy(), e2.cpu().numpy()) < 1e-8
    assert np.max(np.abs(o1.cpu().numpy() - o2.cpu().numpy())) < 1e-9


@pytest.mark.parametrize("shape", [(64, 64, 8), (128, 128, 16), (256, 16, 32), (16, 256, 64), (32, 128, 32),
                                   (64, 128, 64), (256, 64, 32), (256, 256, 8)])
def test_gram_schmidt_in_quarter_planes_matches_separate_passes(shape, monkeypatch):
    """Mixed solves on planes of 4096 and more values: the Gram-Schmidt work in the
    quarter-plane kernels (projections only below 32 z planes, where the partials
    are padded for the separate update pass; with the update from 32 on) against
    the separate passes (PSFD_FUSE_DOTS=0), for every split of a block (4, 8 and 16
    values per thread, 1024 threads). Both stop at the same tolerance, so the
    fields agree to the conditioning times it, within one restart cycle of the
    same step count; repeated solves and a served slot are bitwise the same."""
    from paper_2606_25541_amd import api
    dev = device()
    nx, ny, nz = shape
    layers, es = clips.mo_si_stack(40)
    p = clips.Problem(nx=nx, ny=ny, nz=nz, lx_nm=2.0 * nx, ly_nm=2.0 * ny, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=1, layers=layers, eps_sub=es)
    d = torch.from_numpy(clips.contact_holes(nx, ny, nz, 2.0 * nx, 2.0 * ny, 6, seed=78)).to(dev)
    say("solve %dx%dx%d mixed, Gram-Schmidt in quarter planes" % shape)
    plan = api.Plan(p, rtol=1e-9, precision="mixed", restart=8)
    e1, o1, i1 = plan.psfd_solve(d)
    e1b, o1b, i1b = plan.psfd_solve(d)
    srv = api.Server(hbm_budget=8 << 30, max_slots=2, rtol=1e-9, precision="mixed", restart=8)
    es_, os_ = torch.empty_like(e1), torch.empty_like(o1)
    t = srv.submit(p, d, es_, os_)
    deadline = time.perf_counter() + 60
    done = False
    while not done and time.perf_counter() < deadline:
        done, info, _ = srv.poll(t)
        time.sleep(0.002)
    srv.close()
    assert done, "served request not finished within 60 s"
    monkeypatch.setenv("PSFD_FUSE_DOTS", "0")
    e2, o2, i2 = plan.psfd_solve(d)
    say("  fused", i1, "served", info, "separate", i2)
    assert i1["status"] == 0 and i2["status"] == 0 and info["status"] == 0
    assert torch.equal(e1, e1b) and i1 == i1b
    if nz >= 32:
        assert torch.equal(e1, es_) and info["iters"] == i1["iters"]
    else:
        assert rel(e1.cpu().numpy(), es_.cpu().numpy()) < 1e-7
    assert abs(i1["iters"] - i2["iters"]) <= 8
    assert rel(e1.cpu().numpy(), e2.cpu().numpy()) < 1e-7


def test_batch_beyond_the_infinity_cache_matches_alone():
    """Ten 64 x 64 x 32 mixed instances in lock-step (basis 9 x 3.1 MB each, 283 MB in
    all: the slots are read nontemporally) against a lone solve (28 MB: through the
    caches): the loads differ, the arithmetic does not, so fields and step counts
    are bitwise the same."""
    from paper_2606_25541_amd import api
    dev = device()
    layers, es = clips.mo_si_stack(40)
    p = clips.Problem(nx=64, ny=64, nz=32, lx_nm=128.0, ly_nm=128.0, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=1, layers=layers, eps_sub=es)
    ds = [torch.from_numpy(clips.contact_holes(64, 64, 32, 128.0, 128.0, 6, seed=200 + i)).to(dev) for i in range(10)]
    opts = dict(rtol=1e-8, precision="mixed", restart=8)
    say("solve 10 x 64x64x32 mixed, batch vs alone")
    em, od, infos = api.psfd_solve_batch([p] * 10, ds, **opts)
    plan = api.Plan(p, **opts)
    for i in (0, 9):
        e, o, info = plan.psfd_solve(ds[i])
        say("  instance", i, infos[i]["iters"], info["iters"])
        assert info["status"] == 0 and infos[i]["status"] == 0
        assert infos[i]["iters"] == info["iters"]
        assert torch.equal(em[i], e) and torch.equal(od[i], o)


def test_fp64_solve_quarter_planes_match_strips(monkeypatch):
    """128 x 128 x 32, FP64, lock-step: the Arnoldi steps and b - A x on quarter
    planes (four blocks per plane, the radix-4 y combine in the pencil) against
    the row and column strips (PSFD_QUARTER_PLANES=0), in one process: the
    switch is part of the captured restart cycle's key, so the second solve
    captures the strip kernels instead of replaying the quarter-plane ones. Both
    reach the tolerance and the same field to the conditioning times it."""
    from paper_2606_25541_amd import api
    dev = device()
    layers, es = clips.mo_si_stack(40)
    p = clips.Problem(nx=128, ny=128, nz=32, lx_nm=256.0, ly_nm=256.0, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=0, layers=layers, eps_sub=es)
    d = torch.from_numpy(clips.contact_holes(128, 128, 32, 256.0, 256.0, 6, seed=91)).to(dev)
    say("solve 128x128x32 fp64, quarter planes vs strips")
    plan = api.Plan(p, rtol=1e-10, precision="fp64", restart=8)
    e1, o1, i1 = plan.psfd_solve(d)
    e1b, o1b, i1b = plan.psfd_solve(d)
    monkeypatch.setenv("PSFD_QUARTER_PLANES", "0")
    e2, o2, i2 = plan.psfd_solve(d)
    say("  quarter", i1, "strips", i2)
    assert i1["status"] == 0 and i2["status"] == 0
    assert torch.equal(e1, e1b) and i1 == i1b
    assert not torch.equal(e1, e2)  # the strip kernels ran: other rounding
    assert abs(i1["iters"] - i2["iters"]) <= 2
    assert rel(e1.cpu().numpy(), e2.cpu().numpy()) < 1e-8
    assert np.max(np.abs(o1.cpu().numpy() - o2.cpu().numpy())) < 1e-9


def test_fused_krylov_64_planes_matches_oracle_monolithic():
    """64 x 64 x 32, mixed, lock-step with the projections and the update inside
    the transform kernels, against the oracle: the oracle's GMRES on its
    monolithic operator (I - M V) u = e_bg (the system the GPU solves), the mask
    field x = K V u and the reflected orders from u. Both sides stop at a
    residual of 1e-10 or below, so the fields agree to the conditioning times
    that: <= 1e-7 relative, orders <= 1e-8."""
    from paper_2606_25541_amd import api
    dev = device()
    layers, es = clips.mo_si_stack(40)
    n = 64
    p = clips.Problem(nx=n, ny=n, nz=32, lx_nm=2.0 * n, ly_nm=2.0 * n, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=1, layers=layers, eps_sub=es)
    de = clips.contact_holes(n, n, 32, 2.0 * n, 2.0 * n, 6, seed=77)
    plan = api.Plan(p, rtol=1e-10, precision="mixed", restart=8)
    em, orders, info = plan.psfd_solve(torch.from_numpy(de).to(dev))
    say("  gpu", info, "; oracle monolithic GMRES next")
    assert info["status"] == 0
    S = O.Setup(p)
    u, oi = O.gmres(lambda v: O.apply_monolithic(S, de, v), O.background_field(S), None, 1e-10, 30, 4000)
    say("  oracle", oi["iters"], oi["rel_residual"])
    V = O.potential(S, de)
    x = O.conv_K(S, V[None] * u)
    a_up = O.reflect(S, O.incident_down(S) + O.read_down(S, V[None] * u))
    ords = O.reflected_orders(S, de, u, a_up)
    assert rel(em.cpu().numpy(), x) < 1e-7
    assert np.max(np.abs(orders.cpu().numpy() - ords)) < 1e-8


@pytest.mark.parametrize("prec", ["fp64", "mixed"])
def test_cancellation_restarts_converge(prec, monkeypatch):
    """A Gram-Schmidt update that cancels below the threshold ends the Arnoldi
    cycle; forcing it on (threshold 0.95) must still reach the oracle's solution,
    through more, shorter cycles."""
    from paper_2606_25541_amd import api
    dev = device()
    p = small(16, 8, 8, pol=1, phi=30.0)
    de = clip_of("manhattan", p)
    ref = O.solve(p, de, rtol=1e-12)
    plan = api.Plan(p, rtol=1e-10, precision=prec, restart=20, coupling="mono")
    _, _, base = plan.psfd_solve(torch.from_numpy(de).to(dev))
    monkeypatch.setenv("PSFD_CANCEL", "0.95")
    em, orders, info = plan.psfd_solve(torch.from_numpy(de).to(dev))
    say("  forced", info, "default", base)
    assert info["status"] == 0
    assert info["cycles"] > base["cycles"]
    assert rel(em.cpu().numpy(), ref["emask"]) < 1e-8
    assert np.max(np.abs(orders.cpu().numpy() - ref["orders"])) < 1e-9


@pytest.mark.parametrize("coupling", ["outer", "mono"])
def test_bare_multilayer_on_gpu(coupling):
    from paper_2606_25541_amd import api
    dev = device()
    p = small(8, 8, 4)
    de = np.zeros((4, 8, 8), complex)
    S = O.Setup(p)
    plan = api.Plan(p, rtol=1e-10, precision="fp64", coupling=coupling)
    em, orders, info = plan.psfd_solve(torch.from_numpy(de).to(dev))
    orders = orders.cpu().numpy()
    ref = S.TR[0, 0] @ S.e_inc * np.exp(1j * S.beta[0, 0] * S.t)
    assert np.max(np.abs(orders[0, 0] - ref)) < 1e-13
    o2 = orders.copy()
    o2[0, 0] = 0
    assert np.max(np.abs(o2)) == 0.0
    assert np.max(np.abs(em.cpu().numpy())) == 0.0


def test_config1_line_space_fp64():
    """32x32x32, 64x64 nm clip, 32 nm line, TE 6 deg, GMRES(30) to 1e-8 (FP64)."""
    from paper_2606_25541_amd import api
    dev = device()
    p = clips.config_problem("G1")
    de = clips.line_space(32, 32, 32, 64.0, 64.0, 16.0, 48.0)
    say("config1")
    ref = O.solve(p, de, rtol=1e-11)
    plan = api.Plan(p, rtol=1e-8, precision="fp64", restart=30, coupling="outer")
    em, orders, info = plan.psfd_solve(torch.from_numpy(de).to(dev))
    say("  info", info, "oracle its", ref["iters"], "outer", ref["outer_iters"])
    assert info["status"] == 0
    assert rel(em.cpu().numpy(), ref["emask"]) < 1e-6
    assert rel(orders.cpu().numpy(), ref["orders"]) < 1e-6


def test_solve_deterministic_and_reusable():
    from paper_2606_25541_amd import api
    dev = device()
    p = small(16, 16, 8)
    de = clip_of("manhattan", p)
    plan = api.Plan(p, rtol=1e-8, precision="mixed")
    d = torch.from_numpy(de).to(dev)
    a, oa, ia = plan.psfd_solve(d)
    b, ob, ib = plan.psfd_solve(d)
    assert torch.equal(a, b) and torch.equal(oa, ob)
    assert ia == ib


def test_batch_whose_instances_leave_matches_alone():
    """Ten 64 x 64 x 32 mixed instances in lock-step at restart 16: early steps read the
    basis through the caches, later ones past them, and as the instances of weak
    contrast converge the later ones read through the caches again. The loads
    differ, the arithmetic does not: fields and step counts equal the lone
    solves' bitwise."""
    from paper_2606_25541_amd import api
    dev = device()
    layers, es = clips.mo_si_stack(40)
    p = clips.Problem(nx=64, ny=64, nz=32, lx_nm=128.0, ly_nm=128.0, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=1, layers=layers, eps_sub=es)
    ds = [torch.from_numpy(clips.contact_holes(64, 64, 32, 128.0, 128.0, 6, seed=220 + i) * (1.0 if i < 3 else 0.2)).to(dev)
          for i in range(10)]
    opts = dict(rtol=1e-8, precision="mixed", restart=16)
    say("solve 10 x 64x64x32 mixed, restart 16, batch vs alone")
    em, od, infos = api.psfd_solve_batch([p] * 10, ds, **opts)
    plan = api.Plan(p, **opts)
    for i in (0, 2, 9):
        e, o, info = plan.psfd_solve(ds[i])
        say("  instance", i, infos[i]["iters"], info["iters"])
        assert info["status"] == 0 and infos[i]["status"] == 0
        assert infos[i]["iters"] == info["iters"]
        assert torch.equal(em[i], e) and torch.equal(od[i], o)
    assert infos[9]["iters"] < infos[0]["iters"]


@pytest.mark.parametrize("shape", [(128, 128, 64), (256, 64, 64), (256, 256, 32)])
def test_gram_schmidt_update_of_16_values_per_thread(shape, monkeypatch):
    """The forward quarter-plane kernels whose threads hold 16 values (4096-value
    quarters above 32 z planes, 16384-value ones) with the update fused: against the
    separate passes (PSFD_FUSE_DOTS=0; fields to the conditioning times the
    tolerance, within one restart cycle of the same step count), and bitwise the
    same in a repeat, in a served slot, and in a lock-step batch of two, whose
    slots are read past the caches from some step on."""
    from paper_2606_25541_amd import api
    dev = device()
    nx, ny, nz = shape
    layers, es = clips.mo_si_stack(40)
    p = clips.Problem(nx=nx, ny=ny, nz=nz, lx_nm=2.0 * nx, ly_nm=2.0 * ny, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=1, layers=layers, eps_sub=es)
    ds = [torch.from_numpy(clips.contact_holes(nx, ny, nz, 2.0 * nx, 2.0 * ny, 6, seed=s)).to(dev) for s in (78, 79)]
    say("solve %dx%dx%d mixed, update of 16 values per thread" % shape)
    opts = dict(rtol=1e-9, precision="mixed", restart=8)
    plan = api.Plan(p, **opts)
    alone = [plan.psfd_solve(d) for d in ds]
    e1, o1, i1 = alone[0]
    e1b, o1b, i1b = plan.psfd_solve(ds[0])
    assert i1["status"] == 0 and i1 == i1b and torch.equal(e1, e1b) and torch.equal(o1, o1b)
    em, od, infos = api.psfd_solve_batch([p, p], ds, **opts)
    for (e, o, i), eb, ob, ib in zip(alone, em, od, infos):
        say("  batched", ib, "alone", i)
        assert ib["status"] == 0 and ib["iters"] == i["iters"]
        assert torch.equal(e, eb) and torch.equal(o, ob)
    api.psfd_release_cached_workspaces()
    srv = api.Server(hbm_budget=16 << 30, max_slots=2, **opts)
    es_, os_ = torch.empty_like(e1), torch.empty_like(o1)
    t = srv.submit(p, ds[0], es_, os_)
    deadline = time.perf_counter() + 60
    done = False
    while not done and time.perf_counter() < deadline:
        done, info, _ = srv.poll(t)
        time.sleep(0.002)
    srv.close()
    assert done, "served request not finished within 60 s"
    assert info["status"] == 0 and info["iters"] == i1["iters"]
    assert torch.equal(e1, es_) and torch.equal(o1, os_)
    monkeypatch.setenv("PSFD_FUSE_DOTS", "0")
    e2, _, i2 = plan.psfd_solve(ds[0])
    say("  fused", i1, "separate", i2)
    assert i2["status"] == 0
    assert abs(i1["iters"] - i2["iters"]) <= 8
    assert rel(e1.cpu().numpy(), e2.cpu().numpy()) < 1e-7


@pytest.mark.parametrize("shape", [(64, 64, 8), (64, 64, 16), (128, 128, 16), (256, 256, 8), (64, 64, 4)])
def test_served_slot_equals_lone_solve_with_separate_update(shape):
    """Mixed solves below 32 z planes: the projections in the inverse kernel, the update
    a pass of its own, the Givens step beside it. A served slot runs the same
    arithmetic as the lone solve: step counts, fields and orders are bitwise the
    same."""
    from paper_2606_25541_amd import api
    dev = device()
    nx, ny, nz = shape
    layers, es = clips.mo_si_stack(40)
    p = clips.Problem(nx=nx, ny=ny, nz=nz, lx_nm=2.0 * nx, ly_nm=2.0 * ny, t_nm=60.0, theta_deg=6.0,
                      phi_deg=15.0, pol=1, layers=layers, eps_sub=es)
    d = torch.from_numpy(clips.contact_holes(nx, ny, nz, 2.0 * nx, 2.0 * ny, 6, seed=78)).to(dev)
    say("solve %dx%dx%d mixed, served and alone" % shape)
    opts = dict(rtol=1e-9, precision="mixed", restart=8)
    e1, o1, i1 = api.Plan(p, **opts).psfd_solve(d)
    srv = api.Server(hbm_budget=8 << 30, max_slots=2, **opts)
    e2, o2 = torch.empty_like(e1), torch.empty_like(o1)
    t = srv.submit(p, d, e2, o2)
    deadline = time.perf_counter() + 60
    done = False
    while not done and time.perf_counter() < deadline:
        done, info, _ = srv.poll(t)
        time.sleep(0.002)
    srv.close()
    assert done, "served request not finished within 60 s"
    say("  alone", i1, "served", info, "rel", rel(e2.cpu().numpy(), e1.cpu().numpy()))
    assert i1["status"] == 0 and info["status"] == 0
    assert info["iters"] == i1["iters"]
    assert torch.equal(e1, e2) and torch.equal(o1, o2)
