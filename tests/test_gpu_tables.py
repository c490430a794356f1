"""Host tables sent as kernel arguments: replicas on grids of every kind in one
call, more replicas than one launch carries, and a single replica, which needs
no tables, against the same replicas packed."""

import numpy as np
import pytest
import torch

import synth
from tests._helpers import gpu_list, oracle_list, small_box

pytestmark = pytest.mark.gpu


def test_grids_of_many_sizes_in_one_call(gpu_lib):
    """Boxes of 1 (whole replica), 3, 4, 5, 7, 8 and 11 cells per side."""
    boxes = [small_box(960 + m, n=2 * m * m * m + 1, box=3.0 * m + 1.0) for m in (3, 4, 2, 5, 7, 8, 11, 3)]
    system = gpu_lib.DeviceSystem([b[0] for b in boxes], [b[1] for b in boxes], [b[2] for b in boxes])
    nl = gpu_list(gpu_lib, system, 3.0, capacity=400000)
    off, nbr = nl.rows()
    for k, (pos, _, box) in enumerate(boxes):
        a0, a1 = system.rep_start[k], system.rep_start[k + 1]
        o, want = oracle_list(pos, box, 3.0)
        assert np.array_equal(off[a0:a1 + 1] - off[a0], o), f"replica {k}"
        assert np.array_equal(nbr[off[a0]:off[a1]] - a0, want), f"replica {k}"


@pytest.mark.parametrize("copies", [2, 159, 479, 481, 700])
def test_many_small_replicas_equal_alone(gpu_lib, copies):
    """159: three tables just within one launch, 479 and 481: each table within
    one launch and beyond it."""
    print(f"case copies={copies}", flush=True)
    cons = gpu_lib.Model.from_spec(synth.CONS_CFG0, synth.random_weights(synth.CONS_CFG0, 971))
    nc = gpu_lib.Model.from_spec(synth.NC_CFG1, synth.random_weights(synth.NC_CFG1, 972))
    pos, species, box = small_box(973, n=5, box=11.0)
    out = []
    for r in (1, copies):
        system = gpu_lib.DeviceSystem([pos] * r, [species] * r, [box] * r)
        nl = gpu_list(gpu_lib, system, 5.0)
        ws = gpu_lib.workspace(cons, nc, system.n, r, nl.capacity)
        ws.fill_(255)  # NaN: nothing may be read before it is written
        e, f = gpu_lib.nnp_cons_energy_forces(cons, system, nl, ws)
        g = gpu_lib.nnp_nc_forces(nc, system, nl, ws)
        out.append((e.clone(), f.clone(), g.clone()))
    (e1, f1, g1), (e, f, g) = out
    assert torch.equal(e, e1.expand(copies))
    assert torch.equal(f, f1.repeat(1, copies)) and torch.equal(g, g1.repeat(1, copies))
