"""GPU tree against the oracle's tree: same sorted order (bitwise), same cells (each run of unary cells
of the oracle's uncollapsed tree appears once on the GPU, at its deepest cell; leaves at the first cell of
their run), same geometric centres (bitwise: same sums in the same order, Eq. magCenter)."""
import numpy as np
import pytest

from paper_1212_2934_amd import workloads
from gpu_util import run_field

pytestmark = pytest.mark.gpu


def _oracle_cells(t):
    keep = {}
    for i in range(t["level"].size):
        if t["nchild"][i] != 1:
            keep[(int(t["first"][i]), int(t["count"][i]))] = (int(t["level"][i]), t["c"][i],
                                                              int(t["nchild"][i]) == 0)
    return keep


def _compare(pos, mom, leaf, oracle_mod, offset=0, gtree=None):
    t = oracle_mod.Tree(pos, mom, leaf).export()
    n = pos.shape[1]
    assert (gtree["perm"][offset:offset + n] - offset == t["perm"]).all()
    ocells = _oracle_cells(t)
    gcells = {}
    for i in range(gtree["first"].size):
        f = int(gtree["first"][i]) - offset
        if 0 <= f < n and f + int(gtree["count"][i]) <= n:
            gcells[(f, int(gtree["count"][i]))] = (int(gtree["level"][i]), gtree["centroid"][i],
                                                   int(gtree["nchild"][i]) == 0)
    assert set(gcells) == set(ocells)
    for k, (lev, c, leafy) in ocells.items():
        glev, gc, gleafy = gcells[k]
        assert glev == lev and gleafy == leafy, k
        assert (gc == c).all(), (k, gc, c)
    return len(ocells)


@pytest.mark.parametrize("n,side,leaf,seed", [(4096, 32.0, 16, 1001), (5000, 36.0, 4, 7),
                                             (777, 20.0, 1, 8), (20000 + 37, 60.0, 16, 9),
                                             (32000 + 11, 80.0, 16, 10), (40000 + 3, 85.0, 16, 11)])
def test_tree_matches_oracle(oracle_mod, n, side, leaf, seed):
    w = workloads.uniform_cube(n, side, seed)
    out = run_field(w.pos, w.mom, leaf=leaf, counters=False)
    assert out["flags"] == 0
    g = out["bh"].export_tree()
    ncells = _compare(w.pos, w.mom, leaf, oracle_mod, gtree=g)
    assert ncells == g["first"].size


def test_tree_chains_and_batch(oracle_mod):
    ws = [workloads.config3(seed=100 + b, n=3000) for b in range(3)]
    pos = np.stack([w.pos for w in ws])
    mom = np.stack([w.mom for w in ws])
    out = run_field(pos, mom, counters=False)
    g = out["bh"].export_tree()
    total = 0
    for b, w in enumerate(ws):
        total += _compare(w.pos, w.mom, 16, oracle_mod, offset=b * 3000, gtree=g)
    assert total == g["first"].size
    assert (g["first"][:3] == np.array([0, 3000, 6000])).all()  # roots are nodes 0..B-1


@pytest.mark.parametrize("n", [1, 2, 3, 16, 17, 64, 65])
def test_tree_small_systems(oracle_mod, n):
    w = workloads.uniform_cube(n, 6.0 + n ** (1 / 3), seed=n)
    out = run_field(w.pos, w.mom, leaf=16, counters=False)
    g = out["bh"].export_tree()
    _compare(w.pos, w.mom, 16, oracle_mod, gtree=g)


def test_tree_dense_cluster_in_a_large_tree(oracle_mod):
    """A tree of more than 2^16 nodes whose cells below level 10 are populated: 2000 of 40000 particles
    packed in a cube 0.01 wide, so cells of levels 10 to about 16 hold more than a leaf.  Those levels
    take the one-workgroup upward launch; their centres must still equal the oracle's bitwise."""
    rng = np.random.default_rng(12)
    w = workloads.uniform_cube(38000, 85.0, seed=12)
    cluster = np.array([[40.0], [41.0], [42.0]]) + 0.01 * rng.random((3, 2000))
    pos = np.concatenate([w.pos, cluster], axis=1)
    mom = np.concatenate([w.mom, workloads.uniform_cube(2000, 85.0, seed=13).mom], axis=1)
    t = oracle_mod.Tree(pos, mom, 16).export()
    assert t["level"].max() >= 14 and (t["level"] >= 10).sum() > 100  # the deep levels are populated
    out = run_field(pos, mom, leaf=16, counters=False)
    assert out["flags"] == 0
    g = out["bh"].export_tree()
    assert g["first"].size > 0
    ncells = _compare(pos, mom, 16, oracle_mod, gtree=g)
    assert ncells == g["first"].size


def test_sort_order_with_runs_of_equal_upper_code_bits(oracle_mod):
    """The tiled sort orders the codes by their bits above the low 32 and then orders each run of equal
    upper bits by the low bits: short runs by insertion, runs of more than 32 by a merge.  Clusters of 24
    and of 80 particles 1e-4 wide (runs of 24 and 80 equal upper parts whose low bits are out of index
    order) and 300 particles at one point (all 63 bits equal: ties stay in index order), inside 6000
    uniform ones: the order must be the oracle's, bit for bit."""
    rng = np.random.default_rng(21)
    w = workloads.uniform_cube(6000, 50.0, seed=21)
    parts = [w.pos]
    for cnt, c in [(24, 11.0), (80, 23.0)]:
        parts.append(np.array([[c], [c + 1.0], [c + 2.0]]) + 1e-4 * rng.random((3, cnt)))
    parts.append(np.tile(np.array([[31.5], [7.25], [19.75]]), (1, 300)))
    pos = np.concatenate(parts, axis=1)
    # interleave the clusters with the uniform particles so that index order and code order differ
    order = rng.permutation(pos.shape[1])
    pos = np.ascontiguousarray(pos[:, order])
    mom = workloads.uniform_cube(pos.shape[1], 50.0, seed=22).mom
    t = oracle_mod.Tree(pos, mom, 16).export()
    out = run_field(pos, mom, leaf=16, counters=False)
    g = out["bh"].export_tree()
    assert (g["perm"] == t["perm"]).all()


@pytest.mark.parametrize("n", [2000, 2048, 2049])
def test_tree_batch_around_the_one_workgroup_sort(oracle_mod, n):
    """Systems of at most 2048 particles sort in one workgroup each (all passes in LDS); 2049 takes the
    multi-workgroup passes.  Both must give the oracle's order and cells for every system of a batch."""
    ws = [workloads.config3(seed=200 + b, n=n) for b in range(3)]
    pos = np.stack([w.pos for w in ws])
    mom = np.stack([w.mom for w in ws])
    out = run_field(pos, mom, counters=False)
    assert out["flags"] == 0
    g = out["bh"].export_tree()
    total = 0
    for b, w in enumerate(ws):
        total += _compare(w.pos, w.mom, 16, oracle_mod, offset=b * n, gtree=g)
    assert total == g["first"].size


@pytest.mark.parametrize("n,leaf", [(65, 16), (127, 1), (1023, 1), (1024, 16), (1025, 64), (2047, 3), (2048, 16),
                                    (2049, 16), (4095, 1), (4096, 64)])
def test_tree_of_one_workgroup_with_clusters_and_ties(oracle_mod, n, leaf):
    """One workgroup builds a system of at most 4096 particles: up to 2048 by merging sorted runs of 64, above by
    counting passes; the sums stay on the chip up to 1024 nodes.  A quarter of the particles sits in a cluster 1e-4
    wide and an eighth at one point (runs of equal upper code bits, equal codes, deep cells): order, cells and centres
    must be the oracle's, bit for bit."""
    rng = np.random.default_rng(n)
    w = workloads.uniform_cube(n, 4.0 + 2.0 * n ** (1 / 3), seed=n)
    pos = w.pos.copy()
    pick = rng.permutation(n)
    a, b = pick[:n // 4], pick[n // 4:n // 4 + n // 8]
    pos[:, a] = np.array([[1.0], [2.0], [3.0]]) + 1e-4 * rng.random((3, a.size))
    pos[:, b] = np.array([[3.5], [2.25], [1.75]])
    t = oracle_mod.Tree(pos, w.mom, leaf).export()
    out = run_field(pos, w.mom, leaf=leaf, counters=False)
    g = out["bh"].export_tree()
    assert (g["perm"] == t["perm"]).all()
    assert _compare(pos, w.mom, leaf, oracle_mod, gtree=g) == g["first"].size


def _compare_arrays(pos, mom, leaf, oracle_mod, gtree):
    """_compare for one large system, vectorised: the cells are matched by (first, count) after sorting."""
    t = oracle_mod.Tree(pos, mom, leaf).export()
    assert (gtree["perm"] == t["perm"]).all()
    keep = t["nchild"] != 1
    okey = t["first"][keep].astype(np.int64) * (1 << 32) + t["count"][keep]
    oo = np.argsort(okey)
    gkey = gtree["first"].astype(np.int64) * (1 << 32) + gtree["count"]
    go = np.argsort(gkey)
    assert okey.size == gkey.size
    assert (okey[oo] == gkey[go]).all()
    assert (t["level"][keep][oo] == gtree["level"][go]).all()
    assert ((t["nchild"][keep][oo] == 0) == (gtree["nchild"][go] == 0)).all()
    assert (t["c"][keep][oo] == gtree["centroid"][go]).all()  # bitwise
    return okey.size


@pytest.mark.parametrize("which", ["uniform_2p17", "chains_2p20", "uniform_1310727"])
def test_tree_full_size_bitwise(oracle_mod, which):
    """Radix-sort tiles of several keys per thread: two at 2^17 particles and sixteen at 2^20, both with
    256 tiles per system, the most for which the scatter derives its offsets from the raw tile counts;
    1310727 particles need 321 tiles and take the device-wide scan instead.  The sorted order, the cells
    and their centres must equal the oracle's bit for bit."""
    if which == "uniform_2p17":
        w = workloads.config2()
    elif which == "chains_2p20":
        w = workloads.cached("chains_n1048576_seed1003", lambda: workloads.config3())
    else:
        n = 1310727
        w = workloads.cached("uniform_n1310727_phi0.05",
                             lambda: workloads.uniform_cube(n, workloads.cube_side(n, 0.05), 1007))
    print(f"[tree] {which}: n {w.n}", flush=True)
    out = run_field(w.pos, w.mom, leaf=16, counters=False)
    assert out["flags"] == 0
    g = out["bh"].export_tree()
    ncells = _compare_arrays(w.pos, w.mom, 16, oracle_mod, g)
    assert ncells == g["first"].size


def test_exported_bounding_cubes_of_a_large_batch(oracle_mod):
    """Every system's bounding cube (lo, side, scale) is exported, also beyond the 64th of a batch, and
    equals the oracle's bit for bit (componentwise min and max, one IEEE division)."""
    B, n = 70, 50
    ws = [workloads.uniform_cube(n, 8.0 + 0.05 * b, seed=300 + b) for b in range(B)]
    pos = np.stack([w.pos for w in ws])
    mom = np.stack([w.mom for w in ws])
    out = run_field(pos, mom, counters=False)
    assert out["flags"] == 0
    g = out["bh"].export_tree()
    assert g["bbox"].shape == (B, 5)
    for b, w in enumerate(ws):
        ref = oracle_mod.Tree(w.pos, w.mom, 16).export()["bbox"]
        assert (g["bbox"][b] == ref).all(), (b, g["bbox"][b], ref)


@pytest.mark.parametrize("B", [705, 1000])
def test_export_of_a_batch_of_single_particles_leaves_the_tree_alone(B):
    """Each system is one leaf: its exported record, and the field of the same tree after the export, which is exactly
    zero for a single particle.  From 705 systems on the offsets of an export once ran into the node records."""
    import torch
    from paper_1212_2934_amd.binding import BarnesHut
    rng = np.random.default_rng(B)
    pos = torch.from_numpy(rng.random((B, 3, 1))).cuda()
    mom = torch.from_numpy(rng.standard_normal((B, 3, 1))).cuda()
    bh = BarnesHut(1, B, 16, 0.5, "fp64")
    bh.build(pos)
    for _ in range(2):
        g = bh.export_tree()
        assert g["first"].size == B
        assert (g["first"] == np.arange(B)).all() and (g["perm"] == np.arange(B)).all()
        assert (g["count"] == 1).all() and (g["nchild"] == 0).all() and (g["child"] == -1).all()
        assert (g["centroid"] == pos.cpu().numpy()[:, :, 0]).all()
        H, E = bh.field(mom)
        assert bh.check_status() == 0
        assert (H == 0).all() and (E == 0).all()


@pytest.mark.parametrize("n,batch", [(100, 1), (100, 3), (2, 1000), (5000, 2)])
def test_queries_before_the_first_replay_find_no_nodes(n, batch):
    """A captured step that has not been replayed has built nothing.  On a workspace full of ones (random words in
    earnest) the number of nodes is zero and the export writes no node."""
    import ctypes as C

    import torch
    from paper_1212_2934_amd import binding
    L, P = binding.lib(), C.c_void_p
    p = binding.make_params(n, batch, 16, 0.5, "fp32_mixed")
    nbytes = binding.workspace_bytes(p)
    ws = torch.full((nbytes + 256,), 255, dtype=torch.uint8, device="cuda")
    base = ws.data_ptr() + (-ws.data_ptr()) % 256
    h = P()
    assert L.bh_create(C.byref(p), P(base), nbytes, C.byref(h)) == 0
    d = {k: torch.rand(batch, 3, n, dtype=torch.float64, device="cuda") for k in ("pos", "vel", "mom", "omega")}
    step = torch.zeros(1, dtype=torch.int64, device="cuda")
    C3 = C.c_double * 3
    mdp = binding.md_params(1e-4, 1.0, 0.1, 0.1, 1.0, 0.1, 1.0, 1.0, C3(0.0, 0.0, 0.0), C3(9.0, 9.0, 9.0), None, 7)
    st = binding.md_state(*[d[k].data_ptr() for k in ("pos", "vel", "mom", "omega")], step.data_ptr())
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    g = P()
    assert L.bh_graph_capture_md(h, C.byref(st), C.byref(mdp), P(stream.cuda_stream), C.byref(g)) == 0

    def nodes():
        v = C.c_int64(-1)
        assert L.bh_num_nodes(h, None, C.byref(v)) == 0
        return v.value

    cap = batch * (2 * n + 1)  # the most nodes there can be
    out = [torch.full((cap,), -7, dtype=torch.int32, device="cuda") for _ in range(5)]
    cen = torch.full((3 * cap,), -7.0, dtype=torch.float64, device="cuda")
    assert nodes() == 0
    assert L.bh_export_tree(h, None, *[P(t.data_ptr()) for t in out], P(cen.data_ptr()), None, None) == 0
    torch.cuda.synchronize()
    assert all((t == -7).all() for t in out) and (cen == -7.0).all()
    # after a replay the nodes are there
    assert L.bh_graph_launch(g, P(stream.cuda_stream)) == 0
    torch.cuda.synchronize()
    nn = nodes()
    assert batch <= nn < cap
    assert L.bh_export_tree(h, None, *[P(t.data_ptr()) for t in out], P(cen.data_ptr()), None, None) == 0
    torch.cuda.synchronize()
    count, nchild = out[1].cpu().numpy(), out[3].cpu().numpy()
    assert (count[:batch] == n).all() and (count[:nn] > 0).all() and count[:nn][nchild[:nn] == 0].sum() == batch * n
    assert all((t[nn:] == -7).all() for t in out) and (cen[3 * nn:] == -7.0).all()
    L.bh_graph_destroy(g)
    L.bh_destroy(h)


@pytest.mark.parametrize("n,leaf", [(2, 1), (63, 16), (64, 1), (65, 1), (255, 16), (256, 1), (256, 16), (257, 1), (512, 1), (513, 16)])
def test_tree_at_the_edges_of_the_workgroup_shapes(oracle_mod, n, leaf):
    """64, 256, 512 or 1024 threads build a system, by its size; with leaf size 1 a system has more nodes than the sums on the
    chip hold.  Three systems, in each a quarter of the particles in a cluster 1e-4 wide and an eighth at one point:
    order, cells and centres are the oracle's, bit for bit."""
    rng = np.random.default_rng(7 * n + leaf)
    ws = [workloads.uniform_cube(n, 4.0 + 2.0 * n ** (1 / 3), seed=n + b) for b in range(3)]
    pos, mom = np.stack([w.pos for w in ws]), np.stack([w.mom for w in ws])
    for b in range(3):
        pick = rng.permutation(n)
        a, c = pick[:n // 4], pick[n // 4:n // 4 + n // 8]
        pos[b][:, a] = np.array([[1.0], [2.0], [3.0]]) + 1e-4 * rng.random((3, a.size))
        pos[b][:, c] = np.array([[3.5], [2.25], [1.75]])
    g = run_field(pos, mom, leaf=leaf, counters=False)["bh"].export_tree()
    total = sum(_compare(pos[b], mom[b], leaf, oracle_mod, offset=b * n, gtree=g) for b in range(3))
    assert total == g["first"].size


def test_four_million_pairs():
    """2^22 systems of two particles, more than a launch of 1024 threads a system can hold (2^32 threads): the field of
    each pair is its partner's dipole field."""
    import torch
    from paper_1212_2934_amd import binding
    from paper_1212_2934_amd.binding import BarnesHut
    B = 1 << 22
    need = binding.workspace_bytes(binding.make_params(2, B, 16, 0.5, "fp64")) + (8 << 30)
    if torch.cuda.mem_get_info()[0] < need:
        pytest.skip(f"needs {need >> 30} GiB of free device memory")
    print(f"[pairs] {need >> 30} GiB", flush=True)
    gen = torch.Generator(device="cuda").manual_seed(4)
    pos = torch.rand(B, 3, 2, dtype=torch.float64, device="cuda", generator=gen)
    pos[:, :, 1] += 1.0
    mom = torch.randn(B, 3, 2, dtype=torch.float64, device="cuda", generator=gen)
    bh = BarnesHut(2, B, 16, 0.5, "fp64")
    bh.build(pos)
    H = bh.field(mom, energy=False)
    assert bh.check_status() == 0
    r = pos[:, :, :1] - pos[:, :, 1:]
    m = mom.flip(2)
    r2 = (r * r).sum(1, keepdim=True)
    ref = (3 * r * (m * r).sum(1, keepdim=True) / r2 - m) / r2 ** 1.5
    assert ((H - ref).norm() / ref.norm()).item() <= 1e-14
    del bh
    torch.cuda.empty_cache()


@pytest.mark.parametrize("n,batch", [(4097, 3), (6000, 2), (10000, 3)])
def test_tree_of_a_batch_above_the_one_workgroup_build(oracle_mod, n, batch):
    """Systems of more than 4096 particles are built by launches over the whole batch: tiles, chunks of the upward pass
    (ragged at the end of each system) and the lists of cells across chunks stay inside their system.  Chains, with a
    tenth of the particles in a cluster and some at one point; order, cells and centres are the oracle's, bit for bit."""
    rng = np.random.default_rng(n)
    ws = [workloads.config3(seed=700 + b, n=n) for b in range(batch)]
    pos, mom = np.stack([w.pos for w in ws]), np.stack([w.mom for w in ws])
    for b in range(batch):
        pick = rng.permutation(n)
        a, c = pick[:n // 10], pick[n // 10:n // 10 + 70]
        pos[b][:, a] = np.array([[1.0 + b], [2.0], [3.0]]) + 1e-3 * rng.random((3, a.size))
        pos[b][:, c] = np.array([[3.5], [2.25], [1.75 + b]])
    g = run_field(pos, mom, counters=False)["bh"].export_tree()
    total = sum(_compare(pos[b], mom[b], 16, oracle_mod, offset=b * n, gtree=g) for b in range(batch))
    assert total == g["first"].size
    assert (g["first"][:batch] == n * np.arange(batch)).all()
