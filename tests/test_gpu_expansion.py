"""Order-2 cells (the paper's pseudo-particle plus each accepted cell's first moment; an accuracy variant
beyond the paper) through the C ABI against the oracle's order-2 traversal, whose pins are the opposed-pair
closed forms and the parallel-axis identity.  FP64 within 1e-12 (relative L2: the GPU forms a parent's
first moment from its children's, the oracle from the members), FP32-mixed within 1e-5.  The acceptance
decisions are the paper's, so interaction counts equal the order-1 counts."""
import numpy as np
import pytest
import torch

from paper_1212_2934_amd import workloads
from paper_1212_2934_amd.binding import BarnesHut, md_params
from gpu_util import run_field

pytestmark = pytest.mark.gpu
TOL = {"fp64": 1e-12, "fp32_mixed": 1e-5}


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("kind,theta", [("uniform", 0.5), ("uniform", 0.8), ("chains", 0.5), ("chains", 0.3)])
def test_field_matches_oracle(oracle_mod, precision, kind, theta):
    w = workloads.uniform_cube(4096, 32.0, seed=1001) if kind == "uniform" else workloads.config3(seed=77, n=5000)
    out = run_field(w.pos, w.mom, theta=theta, precision=precision, expansion=2)
    assert out["flags"] == 0
    H2, nf, nr = oracle_mod.Tree(w.pos, w.mom, 16).field(theta, order=2)
    assert rel(out["H"], H2) <= TOL[precision]
    assert (out["n_far"] == nf).all() and (out["n_near"] == nr).all()
    # the energy follows the order-2 field
    E = -0.5 * np.sum(w.mom * H2)
    assert abs(out["E"][0] - E) <= TOL[precision] * abs(E)


def test_batched_ragged(oracle_mod):
    B, n = 3, 2000 + 77
    ws = [workloads.uniform_cube(n, 26.0, seed=40 + b) for b in range(B)]
    pos = np.stack([x.pos for x in ws])
    mom = np.stack([x.mom for x in ws])
    out = run_field(pos, mom, theta=0.6, precision="fp32_mixed", counters=False, expansion=2)
    for b, x in enumerate(ws):
        H2, _, _ = oracle_mod.Tree(x.pos, x.mom, 16).field(0.6, order=2)
        assert rel(out["H"][b], H2) <= 1e-5


def test_opposed_pair_closed_form():
    """+m z at (0,0,+delta), -m z at (0,0,-delta), target on the axis at R: 12 delta m / R^4 along z."""
    R, delta = 40.0, 0.3
    pos = np.array([[0.0, 0.0, 0.0], [0.0, 0.0, 0.0], [delta, -delta, R]])
    mom = np.array([[0.0, 0.0, 1.0], [0.0, 0.0, 0.0], [1.0, -1.0, 0.0]])
    out = run_field(pos, mom, theta=0.9, leaf=2, precision="fp64", expansion=2)
    assert out["n_far"][2] == 1
    np.testing.assert_allclose(out["H"][:, 2], [0.0, 0.0, 12.0 * delta / R ** 4], rtol=1e-13, atol=1e-20)
    out1 = run_field(pos, mom, theta=0.9, leaf=2, precision="fp64", expansion=1)
    assert np.abs(out1["H"][:, 2]).max() == 0.0


@pytest.mark.parametrize("n", [1, 2, 5, 17, 300])
def test_small_systems(oracle_mod, n):
    w = workloads.uniform_cube(n, 4.0 + 2.0 * n ** (1.0 / 3.0), seed=90 + n)
    out = run_field(w.pos, w.mom, theta=0.7, precision="fp64", expansion=2)
    H2, _, _ = oracle_mod.Tree(w.pos, w.mom, 16).field(0.7, order=2)
    if n == 1:
        assert np.abs(out["H"]).max() == 0.0
    else:
        assert rel(out["H"], H2) <= 1e-12


def test_more_accurate_than_order_one(oracle_mod):
    w = workloads.uniform_cube(6000, 40.0, seed=13)
    Ha = oracle_mod.allpairs_field(w.pos, w.mom)
    e1 = rel(run_field(w.pos, w.mom, theta=0.5, precision="fp32_mixed", counters=False)["H"], Ha)
    e2 = rel(run_field(w.pos, w.mom, theta=0.5, precision="fp32_mixed", counters=False, expansion=2)["H"], Ha)
    assert e2 < 0.6 * e1, (e1, e2)


@pytest.mark.parametrize("tuning_id", [0, 3, 6, 9])
@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("theta", [0.5, 0.8])
def test_adjoint_matches_oracle(oracle_mod, precision, theta, tuning_id):
    """dE/dr and dE/dm with order-2 cells against the oracle's order-2 adjoint (pinned by finite
    differences of the order-2 frozen energy), three calls (persistent shapes reorder after the first)."""
    w = workloads.uniform_cube(4096, 32.0, seed=1001, hext=(0.0, 0.0, 1.0))
    _, _, dr, dm = oracle_mod.Tree(w.pos, w.mom, 16).energy_grad(theta, w.hext, order=2)
    bh = BarnesHut(w.n, 1, 16, theta, precision, tuning_id=tuning_id, expansion=2)
    p = torch.from_numpy(w.pos).cuda()
    m = torch.from_numpy(w.mom).cuda()
    he = torch.from_numpy(w.hext).cuda()
    bh.build(p)
    for _ in range(3):
        gdr, gdm = bh.field_backward(m, he, gE=torch.ones(1, dtype=torch.float64, device="cuda"))
        assert bh.check_status() == 0
        assert rel(gdr.cpu().numpy(), dr) <= TOL[precision]
        assert rel(gdm.cpu().numpy(), dm) <= TOL[precision]


def test_adjoint_general_vjp_batched(oracle_mod):
    """A general upstream gradient (dL/dH and dL/dE) on a ragged batch of chains, FP64."""
    B, n = 2, 1500 + 13
    ws = [workloads.config3(seed=140 + b, n=n) for b in range(B)]
    pos = np.stack([x.pos for x in ws])
    mom = np.stack([x.mom for x in ws])
    rng = np.random.default_rng(5)
    gH = rng.standard_normal(pos.shape)
    gE = np.array([0.7, -1.3])
    bh = BarnesHut(n, B, 16, 0.6, "fp64", expansion=2)
    bh.build(torch.from_numpy(pos).cuda())
    gdr, gdm = bh.field_backward(torch.from_numpy(mom).cuda(), None, gH=torch.from_numpy(gH).cuda(),
                                 gE=torch.from_numpy(gE).cuda())
    assert bh.check_status() == 0
    gdr, gdm = gdr.cpu().numpy(), gdm.cpu().numpy()
    for b, x in enumerate(ws):
        t = oracle_mod.Tree(x.pos, x.mom, 16)
        H, _, _ = t.field(0.6, order=2)
        # L = gH . H + gE E, E = -1/2 m.H: hbar = gH - gE/2 m; dL/dm adds gE (-1/2 H)
        dr, dm = t.vjp(0.6, gH[b] - 0.5 * gE[b] * x.mom, order=2)
        dm = dm - 0.5 * gE[b] * H
        assert rel(gdr[b], dr) <= 1e-12 and rel(gdm[b], dm) <= 1e-12


@pytest.mark.parametrize("n", [1, 2, 17, 300])
def test_adjoint_small_systems(oracle_mod, n):
    w = workloads.uniform_cube(n, 4.0 + 2.0 * n ** (1.0 / 3.0), seed=150 + n, hext=(0.2, 0.1, -0.3))
    _, _, dr, dm = oracle_mod.Tree(w.pos, w.mom, 16).energy_grad(0.7, w.hext, order=2)
    bh = BarnesHut(w.n, 1, 16, 0.7, "fp64", expansion=2)
    bh.build(torch.from_numpy(w.pos).cuda())
    gdr, gdm = bh.field_backward(torch.from_numpy(w.mom).cuda(), torch.from_numpy(w.hext).cuda(),
                                 gE=torch.ones(1, dtype=torch.float64, device="cuda"))
    assert bh.check_status() == 0
    gdr, gdm = gdr.cpu().numpy(), gdm.cpu().numpy()
    if n == 1:
        assert np.abs(gdr).max() == 0.0
        np.testing.assert_allclose(gdm, dm, rtol=1e-14)
    else:
        assert rel(gdr, dr) <= 1e-12 and rel(gdm, dm) <= 1e-12


@pytest.mark.parametrize("precision,tol,tuning_id", [("fp64", 1e-11, -1), ("fp32_mixed", 1e-8, -1),
                                                     ("fp64", 1e-11, 11)])
def test_md_trajectory_matches_reference(precision, tol, tuning_id):
    """MD steps with order-2 cells against the reference integrator with order-2 forces and torques."""
    from oracle import md as omd
    import ctypes
    w = workloads.uniform_cube(1200, 18.0, seed=8)
    rng = np.random.default_rng(9)
    st = dict(pos=w.pos[None].copy(), vel=rng.standard_normal((1, 3, w.n)), mom=w.mom[None].copy(),
              omega=rng.standard_normal((1, 3, w.n)) * np.sqrt(10.0))
    p = dict(dt=1e-3, kT=1.0, gamma_t=0.1, gamma_r=0.1, mass=1.0, inertia=0.1, wca_eps=1.0, wca_sigma=1.0,
             box_lo=(0.0, 0.0, 0.0), box_hi=(18.0, 18.0, 18.0), hext=np.array([[0.0, 0.0, 0.5]]), seed=77)
    bh = BarnesHut(w.n, 1, 16, 0.6, precision, tuning_id=tuning_id, expansion=2)
    d = {k: torch.from_numpy(np.ascontiguousarray(v)).cuda() for k, v in st.items()}
    d["step"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    he = torch.from_numpy(p["hext"]).cuda()
    C3 = ctypes.c_double * 3
    mdp = md_params(p["dt"], p["kT"], p["gamma_t"], p["gamma_r"], p["mass"], p["inertia"], p["wca_eps"],
                    p["wca_sigma"], C3(*p["box_lo"]), C3(*p["box_hi"]), he.data_ptr(), p["seed"])
    ref = st
    for k in range(3):
        bh.md_step(d, mdp)
        ref = omd.md_step(ref, p, k, theta=0.6, leaf=16, order=2)
    assert bh.check_status() == 0
    for key in ("pos", "vel", "mom", "omega"):
        g = d[key].cpu().numpy()
        err = np.abs(g - ref[key]).max() / np.abs(ref[key]).max()
        assert err <= tol, (key, err)


@pytest.mark.parametrize("expansion", [1, 2])
@pytest.mark.parametrize("n,batch", [(1, 8193), (10, 8192), (10, 8193), (16, 8193), (17, 8193)])
def test_moments_of_many_tiny_systems(oracle_mod, n, batch, expansion):
    """Above 8192 systems those of one leaf (up to 16 particles) are summed by a thread each.  Copies of three systems:
    field and gradient are those of the three alone, and the field is the oracle's."""
    rng = np.random.default_rng(n + batch)
    pos, mom = rng.random((3, 3, n)) * (2.0 * n ** (1 / 3) + 1.0), rng.standard_normal((3, 3, n))
    out = []
    for pick in (np.arange(3), np.arange(batch) % 3):
        p, m = torch.from_numpy(pos[pick]).cuda(), torch.from_numpy(mom[pick]).cuda()
        bh = BarnesHut(n, pick.size, 16, 0.5, "fp64", expansion=expansion)
        bh.build(p)
        H, E = bh.field(m)
        dr, dm = bh.field_backward(m, gE=torch.ones(pick.size, dtype=torch.float64, device="cuda"))
        assert bh.check_status() == 0
        out.append([x.cpu().numpy() for x in (H, E, dr, dm)])
    pick = np.arange(batch) % 3
    for a, b in zip(*out):
        assert np.abs(b - a[pick]).max() <= 1e-13 * max(np.abs(a).max(), 1e-300)
    for b in range(3):
        H = oracle_mod.Tree(pos[b], mom[b], 16).field(0.5, order=expansion)[0]
        assert np.linalg.norm(out[0][0][b] - H) <= 1e-12 * np.linalg.norm(H)


@pytest.mark.parametrize("n,leaf", [(17, 16), (64, 16), (64, 1), (65, 4), (256, 16), (256, 2), (512, 16), (512, 4), (513, 16)])
def test_first_moments_at_the_edges_of_the_workgroup_shapes(oracle_mod, n, leaf):
    """Up to 512 particles nine lanes sum a node's first moment, where the nodes fit on the chip (not with leaf size 1 or
    2), above a thread: three systems, field and gradient against the oracle's order-2 traversal."""
    ws = [workloads.uniform_cube(n, 4.0 + 2.0 * n ** (1 / 3), seed=900 + n + b, hext=(0.2, 0.0, 1.0)) for b in range(3)]
    pos, mom = np.stack([w.pos for w in ws]), np.stack([w.mom for w in ws])
    out = run_field(pos, mom, leaf=leaf, theta=0.7, expansion=2)
    hext = torch.from_numpy(np.tile(np.asarray(ws[0].hext), (3, 1))).cuda()
    dr, dm = out["bh"].field_backward(torch.from_numpy(mom).cuda(), hext,
                                      gE=torch.ones(3, dtype=torch.float64, device="cuda"))
    assert out["flags"] == 0 and out["bh"].check_status() == 0
    for b, w in enumerate(ws):
        t = oracle_mod.Tree(w.pos, w.mom, leaf)
        H, nf, nr = t.field(0.7, order=2)
        assert rel(out["H"][b], H) <= 1e-12
        assert (out["n_far"][b] == nf).all() and (out["n_near"][b] == nr).all()
        _, _, gr, gm = t.energy_grad(0.7, w.hext, order=2)
        assert rel(dr[b].cpu().numpy(), gr) <= 1e-12 and rel(dm[b].cpu().numpy(), gm) <= 1e-12
