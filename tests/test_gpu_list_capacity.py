"""A list with a negative capacity is refused by every entry point that takes
one, before any launch (the room for what is kept per entry is reckoned from
the capacity)."""

import numpy as np
import pytest
import torch

import synth
from tests._helpers import gpu_list, small_box

pytestmark = pytest.mark.gpu


def test_negative_capacity_is_refused(gpu_lib):
    from paper_2602_14975_amd import _abi
    cons = gpu_lib.Model.from_spec(synth.CONS_CFG0, synth.random_weights(synth.CONS_CFG0, 1381))
    nc = gpu_lib.Model.from_spec(synth.NC_CFG1, synth.random_weights(synth.NC_CFG1, 1382))
    pos, species, box = small_box(1383, n=20)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.0)
    ws = gpu_lib.workspace(cons, nc, system.n, 1, nl.capacity)
    nl.capacity = -1
    out = torch.full((3, system.n), 7.0, dtype=torch.float32, device="cuda")
    calls = (lambda: gpu_lib.nnp_cons_energy_forces(cons, system, nl, ws, forces=out),
             lambda: gpu_lib.nnp_nc_forces(nc, system, nl, ws, out),
             lambda: gpu_lib.nnp_nc_forces_noalloc(nc, system, nl, out),
             lambda: gpu_lib.nnp_cons_virial(cons, system, nl, ws),
             lambda: gpu_lib.nnp_nc_virial(nc, system, nl, ws),
             lambda: gpu_lib.nnp_nc_weight_grad(nc, system, nl, out, ws))
    for call in calls:
        with pytest.raises(_abi.NnpError, match="capacity"):
            call()
    torch.cuda.synchronize()
    assert bool((out == 7.0).all())
