"""Barnes-Hut field and energy through the C ABI against the oracle, element by element.

FP64 path: relative L2 <= 1e-12 and energy <= 1e-12 (only summation order differs).
FP32-mixed path (pair arithmetic in FP32 on FP64 offsets, FP64 acceptance test and accumulation):
relative L2 <= 1e-5, 99.9th percentile per-particle relative error <= 1e-5 (floor 1e-3 rms|H|),
energy error normalised by 1/2 sum|m.H| <= 1e-5.  Interaction counts must be identical in both paths:
the acceptance decisions are the definition's, not an approximation of it.
"""
import numpy as np
import pytest

from paper_1212_2934_amd import workloads
from gpu_util import energy_err, errors, run_field

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32_mixed": 1e-5}


def _check(out, H, E, nf, nr, mom, precision):
    assert out["flags"] == 0
    assert (out["n_far"] == nf).all() and (out["n_near"] == nr).all()
    e = errors(out["H"], H)
    tol = TOL[precision]
    assert e["l2"] <= tol, e
    if precision == "fp32_mixed":
        assert e["p999"] <= tol, e
    else:
        assert e["max"] <= 1e-10, e
    assert energy_err(out["E"][0], E, mom, H) <= tol


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
def test_config1_uniform_4096(oracle_mod, precision):
    w = workloads.config1()
    t = oracle_mod.Tree(w.pos, w.mom, 16)
    H, nf, nr = t.field(0.5)
    E = oracle_mod.energy(w.mom, H, None)
    out = run_field(w.pos, w.mom, theta=0.5, precision=precision)
    _check(out, H, E, nf, nr, w.mom, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("theta", [0.0, 0.3, 0.7, 1.2])
def test_theta_sweep_chains(oracle_mod, precision, theta):
    w = workloads.config3(seed=31, n=6000 + 13)  # several tiles and a ragged last wave
    hext = np.array([0.1, 0.0, 0.4])
    t = oracle_mod.Tree(w.pos, w.mom, 16)
    H, nf, nr = t.field(theta)
    E = oracle_mod.energy(w.mom, H, hext)
    out = run_field(w.pos, w.mom, hext=hext, theta=theta, precision=precision)
    _check(out, H, E, nf, nr, w.mom, precision)


@pytest.mark.parametrize("leaf", [1, 3, 8, 32, 64])
def test_leaf_sizes(oracle_mod, leaf):
    w = workloads.uniform_cube(3000, 26.0, seed=41)
    t = oracle_mod.Tree(w.pos, w.mom, leaf)
    H, nf, nr = t.field(0.5)
    out = run_field(w.pos, w.mom, theta=0.5, leaf=leaf, precision="fp64")
    _check(out, H, E=oracle_mod.energy(w.mom, H), nf=nf, nr=nr, mom=w.mom, precision="fp64")


@pytest.mark.parametrize("n", [1, 2, 5, 16, 17, 63, 64, 65, 129])
def test_small_and_ragged(oracle_mod, n):
    w = workloads.uniform_cube(n, 5.0 + n ** (1 / 3), seed=50 + n)
    Hap = oracle_mod.allpairs_field(w.pos, w.mom)
    t = oracle_mod.Tree(w.pos, w.mom, 4)
    H, nf, nr = t.field(0.5)
    for precision in ("fp64", "fp32_mixed"):
        out = run_field(w.pos, w.mom, theta=0.5, leaf=4, precision=precision)
        if n == 1:
            assert (out["H"] == 0).all() and out["E"][0] == 0.0
            continue
        _check(out, H, oracle_mod.energy(w.mom, H), nf, nr, w.mom, precision)
    out0 = run_field(w.pos, w.mom, theta=0.0, leaf=4, precision="fp64")
    if n > 1:
        assert errors(out0["H"], Hap)["l2"] <= 1e-12


def test_batch_equals_single_runs(oracle_mod):
    B, n = 4, 2500
    ws = [workloads.uniform_cube(n, 30.0, seed=60 + b) for b in range(B)]
    pos = np.stack([w.pos for w in ws])
    mom = np.stack([w.mom for w in ws])
    hext = np.array([[0.0, 0.0, 0.5 * b] for b in range(B)])
    for precision in ("fp64", "fp32_mixed"):
        out = run_field(pos, mom, hext=hext, precision=precision)
        assert out["flags"] == 0
        for b, w in enumerate(ws):
            single = run_field(w.pos, w.mom, hext=hext[b], precision=precision)
            assert (out["H"][b] == single["H"]).all()
            assert out["E"][b] == single["E"][0]
            assert (out["n_far"][b] == single["n_far"]).all()
            H, nf, nr = oracle_mod.Tree(w.pos, w.mom, 16).field(0.5)
            assert (out["n_far"][b] == nf).all() and (out["n_near"][b] == nr).all()
            assert errors(out["H"][b], H)["l2"] <= TOL[precision]


def test_permutation_and_repeatability():
    w = workloads.uniform_cube(5000, 36.0, seed=71)
    p = np.random.default_rng(72).permutation(w.n)
    a = run_field(w.pos, w.mom, precision="fp64")
    b = run_field(w.pos[:, p], w.mom[:, p], precision="fp64")
    c = run_field(w.pos, w.mom, precision="fp64")
    assert (b["H"] == a["H"][:, p]).all()
    assert (c["H"] == a["H"]).all() and c["E"][0] == a["E"][0]


@pytest.mark.parametrize("tuning_id", list(range(15)))
def test_launch_shape_invariance(tuning_id):
    w = workloads.config3(seed=81, n=5000)
    ref = run_field(w.pos, w.mom, precision="fp32_mixed", tuning_id=0)
    out = run_field(w.pos, w.mom, precision="fp32_mixed", tuning_id=tuning_id)
    assert (out["H"] == ref["H"]).all() and (out["n_far"] == ref["n_far"]).all()


def test_degenerate_inputs_flagged():
    w = workloads.uniform_cube(300, 12.0, seed=91)
    pos = w.pos.copy()
    pos[:, 5] = pos[:, 9]  # two particles at one position
    out = run_field(pos, w.mom, precision="fp64")
    assert out["flags"] & 2  # coincident
    assert np.isfinite(out["H"]).all()
    pos = w.pos.copy()
    pos[1, 3] = np.nan
    out = run_field(pos, w.mom, precision="fp64", counters=False)
    assert out["flags"] & 1  # non-finite


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
def test_field_with_and_without_the_side_stream(oracle_mod, precision):
    """Above 16384 particles bh_build puts the targets in Hilbert order on the handle's own stream, beside
    the octree; a handle in caller-owned memory has no second stream and does it on the caller's.  Both
    give the same bits, on the first field call, after a rebuild and on a second field call on the same
    tree, and match the oracle."""
    import torch
    from paper_1212_2934_amd.binding import BarnesHut
    w = workloads.config3(seed=97, n=40003)
    t = oracle_mod.Tree(w.pos, w.mom, 16)
    H, nf, nr = t.field(0.5)
    E = oracle_mod.energy(w.mom, H, None)
    p = torch.from_numpy(w.pos).cuda()
    m = torch.from_numpy(w.mom).cuda()
    outs = []
    for caller_memory in (False, True):
        bh = BarnesHut(w.n, 1, 16, 0.5, precision, caller_memory=caller_memory)
        cnt = bh.enable_counters()
        runs = []
        for rebuild in (True, True, False):
            if rebuild:
                bh.build(p)
            Hd, Ed = bh.field(m)
            runs.append((Hd.cpu().numpy(), Ed.cpu().numpy(), cnt[0].cpu().numpy().copy(), cnt[1].cpu().numpy().copy()))
        assert bh.check_status() == 0
        for r in runs[1:]:
            assert all((a == b).all() for a, b in zip(r, runs[0]))
        outs.append(runs[0])
    assert all((a == b).all() for a, b in zip(outs[0], outs[1]))
    out = dict(H=outs[0][0], E=outs[0][1], flags=0, n_far=outs[0][2].reshape(-1), n_near=outs[0][3].reshape(-1))
    _check(out, H, E, nf, nr, w.mom, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("n,leaf,theta,expansion", [
    (3, 16, 0.5, 1), (70, 1, 0.5, 1), (3001, 64, 0.5, 1), (3001, 33, 0.3, 2), (64 * 192, 16, 0.5, 1),
    (64 * 192 + 1, 16, 0.9, 1), (64 * 768 + 1, 16, 0.7, 1), (64 * 1600 + 1, 16, 0.5, 1)])
def test_divided_walks_at_the_edges_of_their_range(oracle_mod, precision, n, leaf, theta, expansion):
    """16, 8, 4 or 1 waves walk the tree for 64 targets, by the number of target groups.  Field and interaction
    counts against the oracle on either side of each change, with leaves of more than one chunk of sixteen
    members and with order-2 cells."""
    w = workloads.uniform_cube(n, workloads.cube_side(n, 0.05) + 1.0, seed=n + leaf)
    t = oracle_mod.Tree(w.pos, w.mom, leaf)
    H, nf, nr = t.field(theta, expansion)
    out = run_field(w.pos, w.mom, theta=theta, leaf=leaf, precision=precision, expansion=expansion)
    _check(out, H, oracle_mod.energy(w.mom, H), nf, nr, w.mom, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
def test_divided_walk_keeps_the_sums_of_the_undivided_walk(precision):
    """101 copies of a system of 1000 particles are 1616 target groups and walk undivided, one copy is walked
    by sixteen waves per group.  The division regroups FP64 sums only, also in the FP32-mixed walk, so the
    fields agree to FP64 rounding (about 300 terms of either sign: 1e-14)."""
    w = workloads.config3(seed=99, n=1000)
    one = run_field(w.pos, w.mom, precision=precision, counters=False)
    many = run_field(np.repeat(w.pos[None], 101, 0), np.repeat(w.mom[None], 101, 0), precision=precision,
                     counters=False)
    assert one["flags"] == 0 and many["flags"] == 0
    for b in (0, 57, 100):
        assert np.linalg.norm(many["H"][b] - one["H"]) <= 1e-14 * np.linalg.norm(one["H"])


@pytest.mark.parametrize("n,batch,expansion", [(3, 3, 1), (17, 1, 1), (1000, 5, 2), (64 * 64, 1, 1), (64 * 64 + 1, 1, 1),
                                               (64 * 128, 1, 2), (64 * 128 + 1, 1, 1)])
def test_groups_of_fewer_targets(oracle_mod, n, batch, expansion):
    """The divided FP64 walk takes 16, 32 or 64 targets per group, by the number of groups over the batch (the
    FP32-mixed walk always 64).  Field, energy and interaction counts against the oracle on either side of each change."""
    ws = [workloads.uniform_cube(n, workloads.cube_side(n, 0.05) + 1.0, seed=n + b) for b in range(batch)]
    out = run_field(np.stack([w.pos for w in ws]), np.stack([w.mom for w in ws]), expansion=expansion)
    for b, w in enumerate(ws):
        H, nf, nr = oracle_mod.Tree(w.pos, w.mom, 16).field(0.5, expansion)
        one = dict(flags=out["flags"], H=out["H"][b], E=out["E"][b:b + 1], n_far=out["n_far"][b], n_near=out["n_near"][b])
        _check(one, H, oracle_mod.energy(w.mom, H), nf, nr, w.mom, "fp64")


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("n,batch,same", [(2500, 5, False), (2500, 4, True), (64 * 1600 + 1, 2, True)])
def test_a_system_alone_and_in_a_batch(precision, n, batch, same):
    """The number of waves that share a walk follows the groups of the whole batch.  Where it is the same, and above
    102400 particles always, a system's field and energy have the same bits alone and in the batch; elsewhere (40
    groups alone, 200 in the batch) they agree to FP64 rounding in both precisions."""
    w = workloads.uniform_cube(n, workloads.cube_side(n, 0.05) + 1.0, seed=n)
    hext = np.array([0.0, 0.0, 0.5])
    one = run_field(w.pos, w.mom, hext=hext, precision=precision, counters=False)
    many = run_field(np.repeat(w.pos[None], batch, 0), np.repeat(w.mom[None], batch, 0), hext=np.tile(hext, (batch, 1)),
                     precision=precision, counters=False)
    assert one["flags"] == 0 and many["flags"] == 0
    for b in (0, batch - 1):
        if same:
            assert (many["H"][b] == one["H"]).all() and many["E"][b] == one["E"][0]
        else:
            assert np.linalg.norm(many["H"][b] - one["H"]) <= 1e-14 * np.linalg.norm(one["H"])
            scale = 0.5 * np.abs(w.mom * one["H"]).sum() + np.abs(w.mom * hext[:, None]).sum()
            assert abs(many["E"][b] - one["E"][0]) <= 1e-14 * scale
