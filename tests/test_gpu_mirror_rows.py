"""Products on pairs of mirrored nodes at the sizes where their rows can go wrong: one- and
two-node rows, odd counts (a middle node that is its own mirror), just below and above a strip
of 16 rows and a padded count; calls of fewer ICs than a wave's eight and just past them.

Bars.  A fixed number of sweeps runs the oracle's map in another summation order: each sweep
rounds sums of N terms of size |y| at 1.1e-16, and the map contracts the sweeps before, so 1e-13
covers 256 nodes with room (as the repository's other fixed-sweep tests).  Gradients: the two
sides stop at a relative change of 1e-12 of a contraction; 1e-8 as elsewhere."""
import numpy as np
import pytest

import oracle
from paper_2301_03989_amd import workloads as W
from tests._parity import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

NODES = [15, 16, 17, 18, 31, 32, 33, 34, 47, 63, 65, 95, 97, 127, 129, 130, 191, 225, 255]


@pytest.fixture(scope="module")
def pc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    return pcprop.Context(0)


def _call(pc, w, **kw):
    from paper_2301_03989_amd import pcprop
    ics = torch.tensor(w.ics, dtype=torch.float64, device="cuda")
    groups = [pcprop.Group(g.ic_offset, g.n_ic, g.t0, g.tf, g.nodes, g.segments, g.tol) for g in w.groups]
    r = pc.propagate_batched(ics, groups, pcprop.Model(w.mu_sun, w.pert, w.epoch, w.inv_c2), want_nodes=True, **kw)
    return {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in r.items()}


def _workload(n, nodes, seed=5):
    span = 10.0 if nodes < 20 else 40.0          # days: few nodes carry short segments
    return W.nbody_venus(n, seed=seed, days=span, segments=1, nodes=nodes)


@pytest.mark.parametrize("nodes", NODES)
@pytest.mark.parametrize("kw", [{}, {"order": 2}, {"path": "plain"}], ids=["first", "second", "plain"])
def test_fixed_sweeps_at_every_node(pc, nodes, kw):
    w = _workload(21, nodes)
    g = w.groups[0]
    r = _call(pc, w, fixed_iters=4, **kw)
    ref = oracle.propagate(w.ics, g.t0, g.tf, g.nodes, 1, g.tol, oracle.Model(1.0, w.pert, 0.0), fixed_iters=4,
                           want_nodes=True, **({"order": 2} if "order" in kw else {}))
    assert rel_err(r["nodes"], ref[2]).max() < 1e-13
    assert rel_err(r["states"], ref[0]).max() < 1e-13


@pytest.mark.parametrize("nodes,tile", [(33, 1024), (64, 1024), (128, 1024), (128, 2048), (255, 2048)])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 16, 17])
def test_few_ics_per_job(pc, nodes, tile, n):
    w = _workload(n, nodes, seed=6)
    g = w.groups[0]
    r = _call(pc, w, fixed_iters=3, tile_pairs=tile)
    ref = oracle.propagate(w.ics, g.t0, g.tf, g.nodes, 1, g.tol, oracle.Model(1.0, w.pert, 0.0), fixed_iters=3,
                           want_nodes=True)
    assert rel_err(r["nodes"], ref[2]).max() < 1e-13


@pytest.mark.parametrize("nodes", [15, 17, 33, 34, 65, 129, 255])
@pytest.mark.parametrize("inv_c2", [0.0, 1e-4], ids=["point-mass", "relativistic"])
def test_adjoint_with_node_seeds(pc, nodes, inv_c2):
    from paper_2301_03989_amd import pcprop
    w = _workload(5, nodes, seed=7)
    w.inv_c2 = inv_c2
    g = w.groups[0]
    tf, S = 2 * g.tf, 2
    model = pcprop.Model(1.0, w.pert, 0.0, inv_c2)
    groups = [pcprop.Group(0, 5, 0.0, tf, nodes, S, 1e-13)]
    rng = np.random.default_rng(nodes)
    gf, gn = rng.standard_normal((5, 6)), rng.standard_normal((5, S, nodes, 6)) / nodes
    f = pc.propagate_batched(torch.tensor(w.ics, device="cuda"), groups, model, want_bounds=True)
    grad, _, st = pc.adjoint(f["bounds"], torch.tensor(gf, device="cuda"), groups, model,
                             gbar_nodes=torch.tensor(gn, device="cuda"))
    assert f["status"] == 0 and st == 0
    ref = oracle.adjoint(w.ics, 0.0, tf, nodes, S, 1e-13, oracle.Model(1.0, w.pert, 0.0, inv_c2=inv_c2), gf, gn)
    err = np.linalg.norm(grad.cpu().numpy() - ref, axis=1) / np.linalg.norm(ref, axis=1)
    assert err.max() <= 1e-8, err.max()
