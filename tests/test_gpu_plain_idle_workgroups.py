"""Sweeps of the plain path that are queued with more workgroups than jobs left: workgroups past the
job list only arrive, also on the sweep that ends the segment, and the sweeps queued behind it do
nothing.  A few eccentric ICs among many that stop early keep the list short over most of a
segment, and the sweeps queued from the previous segment's count reach past the end of the next.

Bar: both paths run the same sweeps in the same arithmetic, 1e-13 as in the repository's other
comparisons of the two; repeated plain runs are equal bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2301_03989_amd import workloads as W
from tests._parity import rel_err


@pytest.mark.parametrize("streams", [1, 3])
@pytest.mark.parametrize("nodes,n", [(16, 600), (60, 1500), (200, 2100)])
def test_short_job_lists_in_wide_launches(nodes, n, streams):
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    pc = pcprop.Context(0)
    rng = np.random.default_rng(nodes)
    quiet = n - 5
    e = np.concatenate([np.full(quiet, 1e-3), np.full(5, 0.5)])
    el = [np.full(n, 0.9), e, rng.uniform(0.0, 0.1, n)] + [rng.uniform(0.0, 6.28, n) for _ in range(3)]
    ics = torch.tensor(W.elements_to_states(*el), device="cuda")
    span = 0.1 if nodes == 16 else 0.7
    groups = [pcprop.Group(0, n // 2, 0.0, 3 * span, nodes, 3, 1e-12),
              pcprop.Group(n // 2, n - n // 2, 0.0, 4 * span, nodes, 4, 1e-12)]
    model = pcprop.Model(1.0, W.planet_elements(), 0.0)
    fused = pc.propagate_batched(ics, groups, model, want_bounds=True)
    first = None
    for _ in range(4):
        plain = pc.propagate_batched(ics, groups, model, want_bounds=True, path="plain", streams=streams)
        assert plain["status"] == fused["status"] == 0
        assert torch.equal(plain["iters"], fused["iters"])
        assert rel_err(plain["states"].cpu().numpy(), fused["states"].cpu().numpy()).max() < 1e-13
        first = first if first is not None else plain["states"]
        assert torch.equal(plain["states"], first)
