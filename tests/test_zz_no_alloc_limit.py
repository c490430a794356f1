"""The largest systems that the allocation-free NC force entry point takes (four
species, one replica): taken, with the forces of nnp_nc_forces, and refused
with one atom more."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from tests._helpers import gpu_list, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width,n", [(8, 41117), (16, 25888), (32, 14872), (64, 8034)])
def test_largest_system_of_the_static_scratch(gpu_lib, width, n):
    from paper_2602_14975_amd import _abi
    print(f"case width={width} n={n}", flush=True)
    spec = ModelSpec("nc", width, 1, 8, 3.5)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 3110 + width))
    for k in (n, n + 1):
        pos, species, box = small_box(3120 + width, n=k, box=(k / 0.08) ** (1.0 / 3.0))
        system = gpu_lib.DeviceSystem(pos, species, box)
        nl = gpu_list(gpu_lib, system, 3.5)
        out = torch.full((3, k), 7.0, dtype=torch.float32, device="cuda")
        if k == n:
            gpu_lib.nnp_nc_forces_noalloc(m, system, nl, out)
            ws = gpu_lib.workspace(None, m, k, 1, nl.capacity)
            assert torch.equal(out, gpu_lib.nnp_nc_forces(m, system, nl, ws))
        else:
            with pytest.raises(_abi.NnpError, match="static maximum"):
                gpu_lib.nnp_nc_forces_noalloc(m, system, nl, out)
            torch.cuda.synchronize()
            assert bool((out == 7.0).all())
