"""The ephemeris kernel's lanes per record: 1 to 8 perturbers take 8 lanes, 9 to 16 take 16; the
records of the last, partly filled wave; both dynamics.  Bar: the suite's against the oracle, 1e-11
of the state at tolerance 1e-13 (the oracle's sums run over the same bodies in the same order)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import oracle
from paper_2301_03989_amd import workloads as W

INV_C2 = 9.870628680e-9   # 1/c^2 in AU, solar mass and two-body time units


@pytest.mark.parametrize("rel", [False, True])
@pytest.mark.parametrize("n_pert", [0, 1, 7, 8, 9, 15, 16])
def test_records_of_every_lane_count(n_pert, rel):
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    pc = pcprop.Context(0)
    base = W.planet_elements()
    extra = base.copy()
    extra[:, 0] *= 0.37
    extra[:, 6] += 2.1
    pert = np.concatenate([base, extra])[:n_pert]
    w = W.nbody_venus(5, seed=3, days=30.0, segments=3, nodes=37, tol=1e-13)
    g = w.groups[0]
    c2 = INV_C2 if rel else 0.0
    groups = [pcprop.Group(0, 5, g.t0, g.tf, g.nodes, g.segments, g.tol)]
    out = pc.propagate_batched(torch.tensor(w.ics, dtype=torch.float64, device="cuda"), groups,
                               pcprop.Model(1.0, pert, 0.0, c2))
    assert out["status"] == 0
    ref = oracle.propagate(w.ics, g.t0, g.tf, g.nodes, g.segments, g.tol, oracle.Model(1.0, pert, 0.0, inv_c2=c2))[0]
    got = out["states"].cpu().numpy()
    for a in (slice(0, 3), slice(3, 6)):
        err = np.linalg.norm(got[:, a] - ref[:, a], axis=1) / np.linalg.norm(ref[:, a], axis=1)
        assert err.max() < 1e-11
