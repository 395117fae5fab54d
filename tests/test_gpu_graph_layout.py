"""A graph call after the job lengths of the context have changed: the same arguments plan other
jobs, whose tables lie elsewhere in the workspace, so the call is captured again and gives the
eager call's values bit for bit (the results do not depend on the job lengths)."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2301_03989_amd import workloads as W


@pytest.mark.parametrize("rel", [False, True])
@pytest.mark.parametrize("n,nodes,lengths", [
    (300, 128, (1, 0, 8)),        # small: four-IC jobs, whole blocks, four-IC jobs, lists
    (5000, 64, (8, 1, 0)),        # large: lists of several lengths
])
def test_graph_follows_the_job_lengths(n, nodes, lengths, rel):
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    pc = pcprop.Context(0)
    w = W.nbody_venus(n, seed=7, days=30.0, segments=2, nodes=nodes, tol=1e-13)
    g = w.groups[0]
    groups = [pcprop.Group(0, n, g.t0, g.tf, g.nodes, g.segments, g.tol)]
    model = pcprop.Model(1.0, W.planet_elements(), 0.0, 9.870628680e-9 if rel else 0.0)
    ics = torch.tensor(w.ics, dtype=torch.float64, device="cuda")
    eager = pc.propagate_batched(ics, groups, model)
    assert eager["status"] == 0
    out = torch.empty_like(ics)
    iters = torch.empty((n, g.segments), dtype=torch.int32, device="cuda")
    for length in (0,) + lengths:
        pc.set_job_list(nodes, length)
        before = pc.graph_captures()
        for rep in range(3):   # captured or replayed, with eager work between
            out.fill_(float("nan"))
            r = pc.propagate_batched(ics, groups, model, graph=True, out=out, iters_out=iters)
            assert r["status"] == 0
            assert torch.equal(out, eager["states"]), (length, rep)
            assert torch.equal(iters, eager["iters"]), (length, rep)
        if not rel and n == 300:
            assert pc.graph_captures() == before + 1, length
