"""NC embedding with two atoms to a wavefront (width 32): last blocks of every
fill, rows longer than a chunk of 64 list entries, both precisions, packed
replicas against each alone."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from oracle import models as om
from tests._helpers import FP32_TOL, gpu_list, oracle_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,bf16", [(2, 0), (3, 0), (15, 0), (17, 1), (18, 0), (31, 0), (250, 1), (251, 0)])
def test_last_blocks(gpu_lib, n, bf16):
    spec = ModelSpec("nc", 32, 1, 8, 3.5)
    print(f"case n={n} bf16={bf16}", flush=True)
    box = 6.0 if n < 20 else 11.0
    pos, species, _ = small_box(1300 + n, n=n, box=box)
    box = max(box, 9.5)
    w = random_weights(spec, 1310 + n)
    m = gpu_lib.Model.from_spec(spec, w, precision=bf16)
    out = []
    for r in (1, 3):
        system = gpu_lib.DeviceSystem([pos] * r, [species] * r, [box] * r)
        nl = gpu_list(gpu_lib, system, 4.5)
        ws = gpu_lib.workspace(None, m, system.n, r, nl.capacity)
        ws.fill_(255)  # NaN: nothing may be read before it is written
        out.append(gpu_lib.nnp_nc_forces(m, system, nl, ws).clone())
    assert torch.equal(out[1], out[0].repeat(1, 3))
    F = om.nc_forces(spec, w, pos, species, box, *oracle_list(pos, box, 3.5))
    # BF16: the bound of the other BF16 parity tests
    assert rel_rmse(out[0].cpu().numpy().T.astype(np.float64), F) <= (1e-2 if bf16 else FP32_TOL)
