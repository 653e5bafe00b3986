"""Calls in flight on a handle.  Every entry point that uses the workspace counts itself in on the device
with its first kernel and out with its last; a call that finds another one in flight sets
BH_FLAG_OVERLAP.  Calls ordered with each other, on one stream or on two streams joined by a wait, never
raise it.  The misuse itself (two calls racing on one workspace) is not run: another call in flight is
simulated from the host by writing the count into the workspace's status words before the call."""
import numpy as np
import pytest
import torch

from paper_1212_2934_amd import binding, workloads
from paper_1212_2934_amd.binding import BarnesHut, md_params

pytestmark = pytest.mark.gpu

IN_FLIGHT = 12  # status word that counts the calls in flight (the workspace starts with the status words)


def _status_words(bh):
    base = bh.workspace.data_ptr()
    off = (-base) % 256
    return bh.workspace[off:off + 64].view(torch.int32)


def _mdp(side):
    C3 = __import__("ctypes").c_double * 3
    return md_params(1e-4, 1.0, 0.1, 0.1, 1.0, 0.1, 1.0, 1.0, C3(0.0, 0.0, 0.0), C3(side, side, side), None, 7)


def _system(n, seed):
    w = workloads.uniform_cube(n, workloads.cube_side(n, 0.05), seed)
    d = {k: torch.from_numpy(np.ascontiguousarray(getattr(w, k)[None])).cuda() for k in ("pos", "mom")}
    d["vel"] = torch.zeros_like(d["pos"])
    d["omega"] = torch.zeros_like(d["pos"])
    d["step"] = torch.zeros(1, dtype=torch.int64, device="cuda")
    return w, d


def _calls(bh, d, mdp):
    """Each entry point once, in stream order."""
    bh.build(d["pos"])
    bh.field(d["mom"])
    bh.field_backward(d["mom"])
    bh.md_step(d, mdp)


@pytest.mark.parametrize("n", [3000, 20000])
def test_ordered_calls_on_two_streams_raise_nothing(n):
    """20000 particles: bh_build and md_step fork onto the handle's own stream as well."""
    torch.cuda.set_device(0)
    w, d = _system(n, 11)
    bh = BarnesHut(n, 1, 16, 0.5, "fp32_mixed")
    mdp = _mdp(workloads.cube_side(n, 0.05))
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    s1.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s1):
        _calls(bh, d, mdp)
    s2.wait_stream(s1)
    with torch.cuda.stream(s2):
        _calls(bh, d, mdp)
    torch.cuda.current_stream().wait_stream(s2)
    torch.cuda.synchronize()
    assert bh.check_status() == 0
    assert int(_status_words(bh)[IN_FLIGHT].item()) == 0


@pytest.mark.parametrize("entry", ["build", "field", "field_backward", "md_step"])
def test_a_call_that_finds_another_in_flight_is_flagged(entry):
    torch.cuda.set_device(0)
    n = 20000
    w, d = _system(n, 12)
    bh = BarnesHut(n, 1, 16, 0.5, "fp32_mixed")
    mdp = _mdp(workloads.cube_side(n, 0.05))
    bh.build(d["pos"])
    torch.cuda.synchronize()
    assert bh.check_status() == 0
    words = _status_words(bh)
    words[IN_FLIGHT] = 1  # as if a call on another stream were running
    if entry == "build":
        bh.build(d["pos"])
    elif entry == "field":
        bh.field(d["mom"])
    elif entry == "field_backward":
        bh.field_backward(d["mom"])
    else:
        bh.md_step(d, mdp)
    torch.cuda.synchronize()
    # the call counted itself in and out again: the simulated call is still in flight
    assert int(words[IN_FLIGHT].item()) == 1
    words[IN_FLIGHT] = 0
    assert bh.check_status() == binding.FLAG_OVERLAP
    bh.field(d["mom"])
    torch.cuda.synchronize()
    assert bh.check_status() == 0


def test_two_handles_step_concurrently_on_unordered_streams():
    """Calls on different handles share nothing (each has its own workspace and stream): two handles
    stepping MD on two streams with no ordering between them give the trajectories each gives alone, and
    neither flags an overlap."""
    torch.cuda.set_device(0)
    n = 20000
    (wa, da), (wb, db) = _system(n, 31), _system(n, 32)
    mdp = _mdp(workloads.cube_side(n, 0.05))
    alone = []
    for d in (da, db):
        bh = BarnesHut(n, 1, 16, 0.5, "fp32_mixed")
        st = {k: v.clone() for k, v in d.items()}
        for _ in range(3):
            bh.md_step(st, mdp)
        torch.cuda.synchronize()
        assert bh.check_status() == 0
        alone.append(st)
    ha, hb = BarnesHut(n, 1, 16, 0.5, "fp32_mixed"), BarnesHut(n, 1, 16, 0.5, "fp32_mixed")
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    sta = {k: v.clone() for k, v in da.items()}
    stb = {k: v.clone() for k, v in db.items()}
    sa.wait_stream(torch.cuda.current_stream())
    sb.wait_stream(torch.cuda.current_stream())
    for _ in range(3):
        with torch.cuda.stream(sa):
            ha.md_step(sta, mdp)
        with torch.cuda.stream(sb):
            hb.md_step(stb, mdp)
    torch.cuda.synchronize()
    assert ha.check_status() == 0 and hb.check_status() == 0
    for st, ref in ((sta, alone[0]), (stb, alone[1])):
        assert torch.equal(st["step"], ref["step"])
        for k in ("pos", "vel", "mom", "omega"):
            err = ((st[k] - ref[k]).abs().max() / ref[k].abs().max()).item()
            assert err <= 1e-12, (k, err)


@pytest.mark.parametrize("n,batch,writes", [(50, 1, False), (50, 3, True), (5000, 2, False)])
@pytest.mark.parametrize("query", ["num_nodes", "export_tree"])
def test_queries_that_write_the_workspace_are_counted(query, n, batch, writes):
    """The tree queries number the nodes of a batch of small systems in the workspace: they count themselves in and
    out and flag another call in flight.  The others only read."""
    torch.cuda.set_device(0)
    pos = torch.rand(batch, 3, n, dtype=torch.float64, device="cuda")
    bh = BarnesHut(n, batch, 16, 0.5, "fp32_mixed")
    bh.build(pos)
    g = bh.export_tree()
    torch.cuda.synchronize()
    words = _status_words(bh)
    assert bh.check_status() == 0 and int(words[IN_FLIGHT].item()) == 0
    words[IN_FLIGHT] = 1  # as if a call on another stream were running
    if query == "num_nodes":
        assert bh.num_nodes() == g["first"].size
    else:
        # num_nodes first, without the simulated call
        words[IN_FLIGHT] = 0
        nn = bh.num_nodes()
        words[IN_FLIGHT] = 1
        out = torch.empty(nn, dtype=torch.int32, device="cuda")
        st = binding.lib().bh_export_tree(bh._h, None, binding._ptr(out), None, None, None, None, None, None,
                                          binding._stream())
        assert st == 0 and (out.cpu().numpy() == g["first"]).all()
    torch.cuda.synchronize()
    assert int(words[IN_FLIGHT].item()) == 1
    words[IN_FLIGHT] = 0
    assert bh.check_status() == (binding.FLAG_OVERLAP if writes else 0)


@pytest.mark.parametrize("n,batch", [(1000, 1), (4096, 1), (300, 7), (64, 2049)])
@pytest.mark.parametrize("entry", ["build", "field", "field_backward", "md_step"])
def test_calls_on_small_systems_are_counted(entry, n, batch):
    """Systems of at most 4096 particles: a build of one workgroup counts itself out, and a step is counted in once for
    each workgroup of its last launch (up to 131072 particles over the batch; 64 x 2049 takes the launches of large
    systems).  A call alone leaves the count at zero, one that finds another in flight is flagged and leaves it."""
    torch.cuda.set_device(0)
    gen = torch.Generator(device="cuda").manual_seed(n)
    side = 2.0 * n ** (1.0 / 3.0) + 1.0
    d = {"pos": side * torch.rand(batch, 3, n, dtype=torch.float64, device="cuda", generator=gen),
         "mom": torch.randn(batch, 3, n, dtype=torch.float64, device="cuda", generator=gen),
         "step": torch.zeros(1, dtype=torch.int64, device="cuda")}
    d["vel"], d["omega"] = torch.zeros_like(d["pos"]), torch.zeros_like(d["pos"])
    mdp = _mdp(side)
    mdp.wca_eps = 0.0  # the random particles overlap
    bh = BarnesHut(n, batch, 16, 0.5, "fp32_mixed")
    bh.build(d["pos"])
    words = _status_words(bh)

    def call():
        if entry == "build":
            bh.build(d["pos"])
        elif entry == "field":
            bh.field(d["mom"])
        elif entry == "field_backward":
            bh.field_backward(d["mom"])
        else:
            bh.md_step(d, mdp)
        torch.cuda.synchronize()

    call()
    assert bh.check_status() == 0 and int(words[IN_FLIGHT].item()) == 0
    words[IN_FLIGHT] = 1  # as if a call on another stream were running
    call()
    assert int(words[IN_FLIGHT].item()) == 1
    words[IN_FLIGHT] = 0
    assert bh.check_status() == binding.FLAG_OVERLAP
    call()
    assert bh.check_status() == 0 and int(words[IN_FLIGHT].item()) == 0
