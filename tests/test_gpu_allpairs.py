"""All-pairs GPU kernel (bh_allpairs, the paper's all-pairs step) through the C ABI against the oracle's
plain FP64 all-pairs sums: field, energy gradient and energy, FP64 and FP32-mixed, ragged sizes around the
512-target workgroup and the 256-source tile, batches, and the Barnes-Hut path at theta = 0 (which sums
every pair directly and must agree with it).  At 2^20 the GPU all-pairs field is checked on sampled
targets, which the oracle computes one by one."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import errors, run_field
from paper_1212_2934_amd import workloads
from paper_1212_2934_amd.binding import allpairs

pytestmark = pytest.mark.gpu

TOL = {"fp64": 1e-12, "fp32_mixed": 1e-5}


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
def test_field_gradient_energy_against_oracle(precision):
    w = workloads.uniform_cube(3000, 30.0, seed=41, hext=(0.3, -0.2, 0.5))
    H, G, E = allpairs(_dev(w.pos), _dev(w.mom), _dev(w.hext), precision, want_dEdr=True, want_E=True)
    Href = oracle.allpairs_field(w.pos, w.mom)
    Gref = oracle.allpairs_grad_r(w.pos, w.mom)
    Eref = oracle.energy(w.mom, Href, w.hext)
    eh, eg = errors(H.cpu().numpy(), Href), errors(G.cpu().numpy(), Gref)
    tol = TOL[precision]
    assert eh["l2"] <= tol and eh["p999"] <= 10 * tol, eh
    assert eg["l2"] <= tol and eg["p999"] <= 10 * tol, eg
    assert abs(E.item() - Eref) <= tol * abs(Eref)


@pytest.mark.parametrize("n", [1, 2, 3, 255, 256, 257, 511, 512, 513, 1025])
def test_ragged_sizes(n):
    rng = np.random.default_rng(n)
    pos = rng.uniform(0.0, 2.0 * n ** (1.0 / 3.0) + 2.0, (3, n))
    mom = workloads.unit_vectors(rng, n)
    H, G, _ = allpairs(_dev(pos), _dev(mom), precision="fp64", want_dEdr=True)
    H, G = H.cpu().numpy(), G.cpu().numpy()
    if n == 1:
        assert (H == 0).all() and (G == 0).all()
        return
    assert errors(H, oracle.allpairs_field(pos, mom))["max"] <= 1e-11
    assert errors(G, oracle.allpairs_grad_r(pos, mom))["max"] <= 1e-11


def test_batch_equals_single_runs():
    rng = np.random.default_rng(43)
    B, n = 3, 700
    pos = np.stack([workloads.rsa_uniform(rng, n, (0, 0, 0), (14.0, 14.0, 14.0)) for _ in range(B)])
    mom = np.stack([workloads.unit_vectors(rng, n) for _ in range(B)])
    hext = rng.standard_normal((B, 3))
    H, G, E = allpairs(_dev(pos), _dev(mom), _dev(hext), "fp64", want_dEdr=True, want_E=True)
    for b in range(B):
        h1, g1, e1 = allpairs(_dev(pos[b]), _dev(mom[b]), _dev(hext[b]), "fp64", want_dEdr=True, want_E=True)
        assert torch.equal(H[b], h1) and torch.equal(G[b], g1) and torch.equal(E[b:b + 1], e1)


def test_barnes_hut_at_theta_zero_is_all_pairs():
    w = workloads.uniform_cube(2500, 28.0, seed=44)
    H, _, _ = allpairs(_dev(w.pos), _dev(w.mom), precision="fp64")
    bh = run_field(w.pos, w.mom, theta=0.0, precision="fp64", counters=False)
    assert errors(bh["H"], H.cpu().numpy())["max"] <= 1e-12


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
def test_chains_2p20_sampled_targets(precision):
    w = workloads.cached("chains_n1048576_seed1003", lambda: workloads.config3())
    H, _, _ = allpairs(_dev(w.pos), _dev(w.mom), precision=precision)
    idx = np.sort(np.random.default_rng(45).choice(w.n, 256, replace=False))
    Href = oracle.allpairs_field_subset(w.pos, w.mom, idx)
    e = errors(H.cpu().numpy()[:, idx], Href)
    tol = TOL[precision]
    assert e["l2"] <= tol and e["max"] <= 10 * tol, e


def test_fp64_pair_field_to_rounding_over_distances():
    """Two particles on the z axis, moments along z: the field at each is 2 m / r^3 along z (Eq. H_dip).
    Over distances from 1e-3 to 1e3 the FP64 kernel (hardware 1/sqrt estimate plus one refinement step)
    must agree to about ten units in the last place (a refinement short of full precision would not)."""
    B = 241
    r = np.logspace(-3.0, 3.0, B)
    pos = np.zeros((B, 3, 2))
    pos[:, 2, 0] = 0.37
    pos[:, 2, 1] = 0.37 + r
    mom = np.zeros((B, 3, 2))
    mom[:, 2, :] = 1.0
    H, _, _ = allpairs(_dev(pos), _dev(mom), None, "fp64")
    H = H.cpu().numpy()
    exact = 2.0 / ((pos[:, 2, 1] - pos[:, 2, 0]) ** 3)  # the distance the kernel sees, formed in FP64
    for k in range(2):
        rel = np.abs(H[:, 2, k] - exact) / exact
        assert rel.max() <= 2e-15, (k, rel.max())  # a few roundings; a 2^-46 or worse 1/sqrt fails
        assert np.abs(H[:, :2, k]).max() == 0.0


@pytest.mark.parametrize("precision", ["fp64", "fp32_mixed"])
@pytest.mark.parametrize("n,batch", [(1, 1), (15, 2), (17, 1), (64, 3), (65, 1), (255, 2), (257, 1), (1025, 1),
                                     (8191, 1), (8193, 1), (1000, 40), (1000, 70)])
def test_source_split_at_the_edges_of_units_and_target_groups(oracle_mod, n, batch, precision):
    """Sizes around the source units (16 to 256), the target groups (16, 32 or 64) and the sizes where the
    split changes; field and gradient of the first and last system against the oracle (bars: FP64 sums of up
    to 8193 terms, 1e-12; FP32 pairs, 1e-5)."""
    rng = np.random.default_rng(1000 * n + batch)
    side = 1.5 * n ** (1.0 / 3.0)
    pos = rng.random((batch, 3, n)) * side
    mom = workloads.unit_vectors(rng, n * batch).reshape(3, batch, n).transpose(1, 0, 2).copy()
    H, G, E = allpairs(torch.from_numpy(pos).cuda(), torch.from_numpy(mom).cuda(), precision=precision,
                       want_dEdr=True, want_E=True)
    H, G, E = H.cpu().numpy(), G.cpu().numpy(), E.cpu().numpy()
    tol = 1e-12 if precision == "fp64" else 1e-5
    for b in {0, batch - 1}:
        Href, Gref = oracle_mod.allpairs_field(pos[b], mom[b]), oracle_mod.allpairs_grad_r(pos[b], mom[b])
        if n == 1:
            assert (H[b] == 0).all() and (G[b] == 0).all() and E[b] == 0
            continue
        assert np.linalg.norm(H[b] - Href) <= tol * np.linalg.norm(Href)
        assert np.linalg.norm(G[b] - Gref) <= tol * np.linalg.norm(Gref)
        assert abs(E[b] - oracle_mod.energy(mom[b], Href)) <= tol * 0.5 * np.abs(mom[b] * Href).sum()


@pytest.mark.parametrize("n,batch,precision", [(1000, 70, "fp64"), (8193, 8, "fp64"), (8193, 8, "fp32_mixed")])
def test_a_system_alone_and_in_a_batch(n, batch, precision):
    """The targets of a workgroup, and with them the order of the FP64 sums, follow the groups of the whole batch (16
    targets alone, 64 in these batches): field and gradient agree to FP64 rounding in both precisions, since the
    FP32-mixed sums of 256 sources are the same."""
    rng = np.random.default_rng(n)
    pos = torch.from_numpy(rng.random((3, n)) * 1.5 * n ** (1.0 / 3.0)).cuda()
    mom = torch.from_numpy(workloads.unit_vectors(rng, n)).cuda()
    one = allpairs(pos, mom, precision=precision, want_dEdr=True)
    many = allpairs(pos.expand(batch, 3, n).contiguous(), mom.expand(batch, 3, n).contiguous(), precision=precision,
                    want_dEdr=True)
    for a, b in zip(one[:2], many[:2]):
        for k in (0, batch - 1):
            assert ((b[k] - a).norm() / a.norm()).item() <= 1e-13
