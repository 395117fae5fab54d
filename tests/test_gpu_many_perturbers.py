"""More than 8 perturbers near 128 nodes: the records fit the 512-thread shape's LDS only.  The
FP32 -> FP64 schedule, whose increment sweeps need them there, takes that shape by itself; FP64
calls take the shape that is faster, and their results do not depend on it.

Bar of the schedule against the FP64 oracle: an IC stops on a sweep that changes it by less than
tol = 1e-12 per segment, and a late error grows by less than 2 over the two segments: 4e-12."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle
from paper_2301_03989_amd import workloads as W
from tests._parity import rel_err

INV_C2 = 9.870628680e-9


def _bodies(P):
    rng = np.random.default_rng(5)
    el = [list(e) for e in W.planet_elements()]
    while len(el) < P:   # main-belt bodies
        el.append([1e-9 * rng.uniform(0.5, 2.0), rng.uniform(2.2, 3.3), rng.uniform(0.0, 0.2),
                   rng.uniform(0.0, 0.2), *rng.uniform(0.0, 6.28, 3)])
    return np.array(el)


def _setup(n, nodes, P, rel=False):
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    w = W.nbody_venus(n, seed=P + nodes, days=40.0, segments=2, nodes=nodes, tol=1e-12)
    g = w.groups[0]
    return (pcprop.Context(0), torch.tensor(w.ics, dtype=torch.float64, device="cuda"), w,
            [pcprop.Group(0, n, g.t0, g.tf, g.nodes, g.segments, g.tol)],
            pcprop.Model(1.0, _bodies(P), 0.0, INV_C2 if rel else 0.0))


@pytest.mark.parametrize("rel", [False, True])
@pytest.mark.parametrize("nodes,P", [(116, 9), (128, 9), (68, 16), (128, 16)])
@pytest.mark.parametrize("n", [3, 41])
def test_schedule_keeps_its_increment_sweeps(n, nodes, P, rel):
    assert 3 * nodes * (P + 1) > 3456
    pc, ics, w, groups, model = _setup(n, nodes, P, rel)
    a = pc.propagate_batched(ics, groups, model, precision="fp32-fp64")
    b = pc.propagate_batched(ics, groups, model, precision="fp32-fp64", tile_pairs=2048)
    assert a["status"] == b["status"] == 0
    assert torch.equal(a["states"], b["states"]) and torch.equal(a["iters"], b["iters"])
    g = groups[0]
    ref, _ = oracle.propagate(w.ics, g.t0, g.tf, g.nodes, g.segments, g.tol,
                              oracle.Model(1.0, _bodies(P), 0.0, inv_c2=INV_C2 if rel else 0.0))
    assert rel_err(a["states"].cpu().numpy(), ref).max() < 4e-12


@pytest.mark.parametrize("n", [5, 300, 1500, 2049])
@pytest.mark.parametrize("nodes,P", [(128, 9), (68, 16)])
def test_fp64_results_in_either_shape(n, nodes, P):
    pc, ics, _, groups, model = _setup(n, nodes, P)
    a = pc.propagate_batched(ics, groups, model, want_bounds=True)
    for pairs in (1024, 2048):
        b = pc.propagate_batched(ics, groups, model, want_bounds=True, tile_pairs=pairs)
        for key in ("states", "bounds", "iters"):
            assert torch.equal(a[key], b[key]), (pairs, key)


def test_shape_follows_the_records():
    # job tables of whole blocks: those of the 1024 shape are twice as long
    for n, nodes, P, kw, pairs in ((2049, 128, 8, {}, 1024), (2049, 128, 9, {}, 2048), (2048, 128, 9, {}, 1024),
                                   (2049, 67, 16, {}, 1024), (2049, 68, 16, {}, 2048),
                                   (1500, 128, 9, dict(precision="fp32-fp64"), 2048),
                                   (2049, 64, 16, {}, 1024)):
        pc, _, _, groups, model = _setup(n, nodes, P)
        held = pc.workspace_bytes(groups, model, **kw)
        assert held == pc.workspace_bytes(groups, model, tile_pairs=pairs, **kw), (n, nodes, P, kw)
        assert held != pc.workspace_bytes(groups, model, tile_pairs=3072 - pairs, **kw)
    pc, _, _, groups, model = _setup(2049, 128, 16, rel=True)
    assert pc.workspace_bytes(groups, model) == pc.workspace_bytes(groups, model, tile_pairs=1024)
