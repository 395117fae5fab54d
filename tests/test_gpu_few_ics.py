"""Jobs of at most four ICs evaluate the points of one IC per lane (compiled apart): each IC's
states, node states and sweep counts are those that it has in a job of full columns, bit for bit
(an IC's sweeps round alike in every job body), with starts warm and cold, and a dead IC beside it."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2301_03989_amd import workloads as W


@pytest.mark.parametrize("rel", [False, True])
@pytest.mark.parametrize("nodes", [17, 32, 47, 64, 101, 128, 129, 256])
@pytest.mark.parametrize("n", [1, 3, 4, 5])
def test_few_ics_match_full_columns(nodes, n, rel):
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    pc = pcprop.Context(0)
    w = W.nbody_venus(40, seed=nodes, days=30.0, segments=2, nodes=nodes, tol=1e-13)
    g = w.groups[0]
    model = pcprop.Model(1.0, W.planet_elements(), 0.0, 9.870628680e-9 if rel else 0.0)
    ics = torch.tensor(w.ics, dtype=torch.float64, device="cuda")
    if n == 3:
        ics[1, 2] = float("nan")   # a dead IC in the middle column
    grp = lambda k: [pcprop.Group(0, k, g.t0, g.tf, g.nodes, g.segments, g.tol)]
    for init in ("kepler", "cold"):
        full = pc.propagate_batched(ics, grp(40), model, want_bounds=True, want_nodes=True, init=init, job_list=1)
        few = pc.propagate_batched(ics[:n].contiguous(), grp(n), model, want_bounds=True, want_nodes=True, init=init)
        assert few["status"] == full["status"]
        for key in ("states", "bounds", "nodes", "iters"):
            a, b = few[key].cpu().numpy(), full[key][:n].cpu().numpy()
            assert np.array_equal(a, b, equal_nan=True), key
