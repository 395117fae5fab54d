"""The flyby screen runs in the workspace of whole blocks of the 512-thread shape, whatever jobs the
untuned rules of a propagation would choose; a call with flyby isolation whose workspace holds no
table of four-IC jobs, for itself and for its reordered call, runs in whole blocks."""
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2301_03989_amd import workloads as W


def _setup(n, nodes, segments):
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    w = W.eccentric(nodes, n_ic=n, seed=3, segments=segments)
    g = w.groups[0]
    return (pcprop.Context(0), torch.tensor(w.ics, device="cuda"),
            [pcprop.Group(0, n, g.t0, g.tf, g.nodes, g.segments, g.tol)], pcprop.Model(1.0, w.pert, 0.0))


def _hold(monkeypatch, pc, nbytes):
    held = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    monkeypatch.setattr(pc, "workspace", lambda _: held)


@pytest.mark.parametrize("n,nodes,segments", [(65536, 128, 1), (8192, 60, 1), (300, 128, 2)])
def test_screen_needs_no_job_table(monkeypatch, n, nodes, segments):
    pc, ics, groups, model = _setup(n, nodes, segments)
    want = pc.flyby_ratio(ics, groups, model)
    _hold(monkeypatch, pc, pc.workspace_bytes(groups, model, tile_pairs=2048))
    assert torch.equal(pc.flyby_ratio(ics, groups, model), want)


@pytest.mark.parametrize("hill", [0.01, 6.0, 1e6])   # no flybys, some, all
@pytest.mark.parametrize("n,nodes", [(290, 64), (61, 128), (1000, 40)])
def test_isolation_without_four_ic_jobs(monkeypatch, n, nodes, hill):
    pc, ics, groups, model = _setup(n, nodes, 2)
    want = pc.propagate_batched(ics, groups, model, want_bounds=True, flyby_hill=hill)
    _hold(monkeypatch, pc, pc.workspace_bytes(groups, model, flyby_hill=hill,
                                              tile_pairs=1024 if nodes <= 64 else 2048))
    got = pc.propagate_batched(ics, groups, model, want_bounds=True, flyby_hill=hill)
    assert got["status"] == want["status"]
    for key in ("states", "bounds", "iters"):
        assert torch.equal(got[key], want[key]), key
