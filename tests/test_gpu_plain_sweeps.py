"""The plain path's sweep kernel: the last workgroup's compaction and decision at the edges of
its job list (one job, a partly filled one, more jobs than its threads), several groups on
fewer streams, and segments that end inside, at and past a queued batch of sweeps.

Bars.  Under the per-IC rule both paths run the same sweeps in the same arithmetic: 1e-13, as
the repository's other comparisons of the two.  Under the group rule an IC runs on past its own
stop: it moves by less than the change that stopped it (1e-12), and the fused result is off by
as little, so 2e-12 for one segment."""
import numpy as np
import pytest

from paper_2301_03989_amd import workloads as W
from tests._parity import rel_err

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def pc():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    return pcprop.Context(0)


def _run(pc, ics, groups, pert, **kw):
    from paper_2301_03989_amd import pcprop
    r = pc.propagate_batched(torch.tensor(ics, device="cuda"), [pcprop.Group(*g) for g in groups],
                             pcprop.Model(1.0, pert, 0.0), want_bounds=True, **kw)
    return {k: (v.cpu().numpy() if hasattr(v, "cpu") else v) for k, v in r.items()}


@pytest.mark.parametrize("n", [1, 8, 9, 4096, 4104, 8200])
def test_job_lists_of_every_length(pc, n):
    w = W.eccentric(256, n_ic=n, seed=31, segments=1)
    g = [(0, n, 0.0, np.pi / 4, 200, 1, 1e-12)]
    a = _run(pc, w.ics, g, w.pert)
    b = _run(pc, w.ics, g, w.pert, path="plain")
    assert b["status"] == a["status"] == 0
    np.testing.assert_array_equal(a["iters"], b["iters"])
    assert rel_err(b["states"], a["states"]).max() < 1e-13
    c = _run(pc, w.ics, g, w.pert, path="plain", conv="group")
    assert c["status"] == 0 and (c["iters"] == c["iters"][0]).all() and c["iters"][0, 0] == a["iters"].max()
    assert rel_err(c["states"], a["states"]).max() < 2e-12


@pytest.mark.parametrize("streams", [1, 2, 5])
@pytest.mark.parametrize("max_iter", [1, 3, 4, 5, 6, 7, 64])
def test_batches_of_sweeps_end_where_the_segment_does(pc, streams, max_iter):
    w = W.eccentric(64, n_ic=60, seed=32, segments=3)
    g = [(0, 20, 0.0, 3 * np.pi / 4, 14, 3, 1e-12), (20, 25, 0.0, 2 * np.pi / 4, 64, 2, 1e-12),
         (45, 15, 0.0, 3 * np.pi / 4, 100, 3, 1e-12)]
    a = _run(pc, w.ics, g, w.pert, max_iter=max_iter)
    b = _run(pc, w.ics, g, w.pert, max_iter=max_iter, path="plain", streams=streams)
    assert a["status"] == b["status"]
    np.testing.assert_array_equal(a["iters"], b["iters"])
    assert rel_err(b["states"], a["states"]).max() < 1e-13
