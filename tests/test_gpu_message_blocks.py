"""Matrix-core message kernels with one and with two atoms to a block: the
forces of a replica are the same bits alone (one atom to a block) and packed
to totals where a block holds two atoms (an odd last atom among them) or one
again, and agree with the FP64 oracle."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from oracle import models as om
from tests._helpers import FP32_TOL, gpu_list, oracle_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,copies,bf16", [(301, 3, 0), (301, 5, 0), (301, 6, 1), (256, 3, 0), (769, 2, 1),
                                           (7, 110, 0)])
def test_block_size_does_not_change_the_bits(gpu_lib, n, copies, bf16):
    print(f"case n={n} copies={copies} bf16={bf16}", flush=True)
    spec = ModelSpec("cons", 128, 2, 16, 5.0)
    pos, species, box = small_box(820 + n, n=n, box=max(11.0, (n / 0.06) ** (1.0 / 3.0)))
    w = random_weights(spec, 830 + n)
    m = gpu_lib.Model.from_spec(spec, w, precision=bf16)
    out = []
    for r in (1, copies):
        system = gpu_lib.DeviceSystem([pos] * r, [species] * r, [box] * r)
        nl = gpu_list(gpu_lib, system, 5.0)
        ws = gpu_lib.workspace(m, None, system.n, r, nl.capacity)
        ws.fill_(255)  # NaN: nothing may be read before it is written
        f = gpu_lib.nnp_cons_energy_forces(m, system, nl, ws)[1].clone()
        fv = gpu_lib.nnp_cons_virial(m, system, nl, ws)[1]
        assert torch.equal(f, fv)
        out.append(f)
    alone, packed = out
    for r in range(copies):
        assert torch.equal(packed[:, r * n:(r + 1) * n], alone), f"replica {r}"
    _, F = om.cons_energy_forces(spec, w, pos, species, box, *oracle_list(pos, box, 5.0))
    # BF16: the bound of the other BF16 parity tests
    assert rel_rmse(alone.cpu().numpy().T.astype(np.float64), F) <= (1e-2 if bf16 else FP32_TOL)
