"""The default launch geometry: what sim_get_tiling reports of a fresh handle is
what its launches use, and setting it back (save and restore) changes no
launch.  Launches are told by their workgroups, from a profiler's trace."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from paper_2109_07719_amd import synth

pytestmark = pytest.mark.gpu

T = 4


def launches(sim, b, K):
    """(kernel, grid, block) of a forward and its backward."""
    from torch.profiler import ProfilerActivity, profile
    f = lambda x: torch.tensor(np.ascontiguousarray(x), dtype=torch.float32, device="cuda")
    q, v, u = f(b.q0), f(b.qd0), f(b.tau)
    gq, gv, ws = torch.ones_like(q), torch.ones_like(v), sim.new_workspace(T, K)
    torch.cuda.synchronize()
    with profile(activities=[ProfilerActivity.CPU, ProfilerActivity.CUDA]) as prof:
        sim.forward(q, v, u, b.dt, K=K, workspace=ws)
        sim.backward(u, b.dt, K, ws, gq, gv)
        torch.cuda.synchronize()
    out = [(e["name"], tuple(e["args"]["grid"]), tuple(e["args"]["block"])) for e in events(prof)
           if "k_forward" in e["name"] or "k_backward" in e["name"]]
    return out


def events(prof):
    import json
    import os
    import tempfile
    with tempfile.TemporaryDirectory() as d:
        path = os.path.join(d, "t.json")
        prof.export_chrome_trace(path)
        return [e for e in json.load(open(path))["traceEvents"] if e.get("cat") == "kernel"]


@pytest.mark.parametrize("name,n", [("chain7", 40), ("trees", 40)])
def test_restoring_the_default_changes_no_launch(name, n):
    from paper_2109_07719_amd.sim import Sim
    draw = (lambda k: synth.chain_system(7, k, T)) if name == "chain7" else (lambda k: synth.tree_system(k, T))
    b = synth.make_batch([draw(k) for k in range(n)], 1e-3)
    sim = Sim(b.systems, b.gravity, dtype=torch.float32)
    t = sim.tiling
    first = launches(sim, b, 1)
    print("case", name, t, first, flush=True)
    assert len(first) == 2 and first[0][2][0] == 64 * t["waves_per_block"]
    sim.set_tiling(4, 1, False)
    other = launches(sim, b, 1)
    assert other[0][2][0] == 256 and other != first
    sim.set_tiling(**t)
    assert launches(sim, b, 1) == first and sim.tiling == t
