"""Small calls run jobs of four ICs, one per CU (up to 1024 ICs on 256 CUs): each IC's results are
those of jobs of whole blocks (job_list=1), bit for bit, on ragged counts and several groups, and a
workspace that only holds the whole blocks' job table still runs the call."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from paper_2301_03989_amd import workloads as W


@pytest.mark.parametrize("rel", [False, True])
@pytest.mark.parametrize("counts,nodes", [((5,), (32,)), ((27, 1, 9), (100, 40, 17)), ((301,), (64,)),
                                          ((1024,), (128,)), ((1025,), (128,)), ((250, 33), (200, 33))])
def test_small_calls_match_whole_blocks(monkeypatch, counts, nodes, rel):
    from paper_2301_03989_amd import build, pcprop
    build.ensure_built()
    pc = pcprop.Context(0)
    n = sum(counts)
    w = W.nbody_venus(n, seed=n, days=25.0, segments=2, nodes=max(nodes), tol=1e-13)
    g = w.groups[0]
    off = np.concatenate([[0], np.cumsum(counts)])
    groups = [pcprop.Group(int(o), c, g.t0, g.tf, N, g.segments, g.tol) for o, c, N in zip(off, counts, nodes)]
    model = pcprop.Model(1.0, W.planet_elements(), 0.0, 9.870628680e-9 if rel else 0.0)
    ics = torch.tensor(w.ics, dtype=torch.float64, device="cuda")
    blocks = pc.propagate_batched(ics, groups, model, want_bounds=True, job_list=1)
    small = pc.propagate_batched(ics, groups, model, want_bounds=True)
    for key in ("states", "bounds", "iters"):
        assert torch.equal(small[key], blocks[key]), key
    # the small shape's whole blocks up to 64 nodes (the only untuned choice there), else the large's
    held = pc.workspace_bytes(groups, model, tile_pairs=2048 if max(nodes) > 64 else 1024)
    scratch = torch.empty(held, dtype=torch.uint8, device="cuda")
    monkeypatch.setattr(pc, "workspace", lambda nbytes: scratch)
    again = pc.propagate_batched(ics, groups, model, want_bounds=True)
    assert again["status"] == blocks["status"] == 0
    assert torch.equal(again["states"], blocks["states"])
