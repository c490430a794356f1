"""Replica tables as kernel arguments on another stream and in a recorded graph
(replayed with new positions, eager work in between, and the host tables of
the recorded call overwritten), against eager calls on the default stream."""

import pytest
import torch

import synth
from tests._helpers import gpu_list, small_box

pytestmark = pytest.mark.gpu


class _Setup:
    def __init__(self, nnp, copies):
        self.nnp = nnp
        self.cons = nnp.Model.from_spec(synth.CONS_CFG0, synth.random_weights(synth.CONS_CFG0, 1361))
        self.nc = nnp.Model.from_spec(synth.NC_CFG1, synth.random_weights(synth.NC_CFG1, 1362))
        reps = [small_box(1363 + k, n=n, box=b) for k, (n, b) in enumerate(((5, 11.0), (23, 12.0), (9, 11.5)))] * copies
        self.system = nnp.DeviceSystem([r[0] for r in reps], [r[1] for r in reps], [r[2] for r in reps])
        self.nl = gpu_list(nnp, self.system, 5.4)
        s = self.system
        self.ws = nnp.workspace(self.cons, self.nc, s.n, s.n_rep, self.nl.capacity)
        self.e = torch.empty(s.n_rep, dtype=torch.float64, device="cuda")
        self.f = torch.empty(3, s.n, dtype=torch.float32, device="cuda")
        self.g = torch.empty(3, s.n, dtype=torch.float32, device="cuda")

    def run(self):
        self.nnp.nnp_cons_energy_forces(self.cons, self.system, self.nl, self.ws, self.e, self.f)
        self.nnp.nnp_nc_forces(self.nc, self.system, self.nl, self.ws, self.g)

    def out(self):
        return [t.clone() for t in (self.e, self.f, self.g)]


@pytest.mark.parametrize("copies", [1, 161])
def test_side_stream(gpu_lib, copies):
    """161: tables larger than one launch carries."""
    a = _Setup(gpu_lib, copies)
    a.run()
    want = a.out()
    side = torch.cuda.Stream()
    for t in (a.e, a.f, a.g, a.ws):
        t.fill_(255) if t is a.ws else t.fill_(float("nan"))
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        a.run()
    torch.cuda.current_stream().wait_stream(side)
    assert all(torch.equal(x, y) for x, y in zip(want, a.out()))


def test_graph_replays(gpu_lib):
    a, b = _Setup(gpu_lib, 2), _Setup(gpu_lib, 2)
    a.run()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        a.run()
    a.system.rep_start[:] = -1  # the recorded call's host tables
    a.system.box[:] = -1.0
    shift = torch.tensor([[0.013], [-0.02], [0.017]], dtype=torch.float64, device="cuda")
    for k in range(4):
        for x in (a, b):
            x.system.pos.add_(torch.sin(shift * torch.arange(x.system.n, device="cuda") * (k + 1)) * 0.05)
        b.run()  # eager work between the replays
        a.ws.fill_(255)
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(a.out(), b.out())), f"replay {k}"
