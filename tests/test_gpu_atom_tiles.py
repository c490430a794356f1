"""Per-atom blocks with tiles of 16 and of 32 atoms: edges of the small tiles
and both sides of the sizes where the tile changes (5,418 atoms FP32, 12,288
BF16), against the older dense kernels and, at small sizes, the FP64 oracle."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from oracle import models as om
from tests._helpers import FP32_TOL, gpu_list, oracle_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


def _eval(nnp, model, system, nl, ws, mode):
    from paper_2602_14975_amd import _abi
    _abi.check(nnp.lib().nnp_set_dense_kernels(mode))
    try:
        e, f = nnp.nnp_cons_energy_forces(model, system, nl, ws)
        return e.cpu().numpy(), f.cpu().numpy().T.astype(np.float64)
    finally:
        nnp.lib().nnp_set_dense_kernels(0)


@pytest.mark.parametrize("n,layers,bf16", [(15, 2, 0), (16, 3, 0), (17, 2, 0), (47, 1, 0), (16, 2, 1), (49, 3, 1),
                                           (5418, 2, 0), (5419, 2, 0), (5441, 3, 0), (8192, 2, 1), (8193, 3, 1),
                                           (12288, 2, 1), (12289, 2, 1), (1, 2, 0), (1, 1, 1)])
def test_tiles_at_their_edges(gpu_lib, n, layers, bf16):
    print(f"case n={n} layers={layers} bf16={bf16}", flush=True)
    spec = ModelSpec("cons", 128, layers, 16, 5.0)
    pos, species, box = small_box(900 + n, n=n, box=max(11.0, (n / 0.06) ** (1.0 / 3.0)))
    w = random_weights(spec, 910 + n)
    m = gpu_lib.Model.from_spec(spec, w, precision=bf16)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.0)
    ws = gpu_lib.workspace(m, None, n, 1, nl.capacity)
    ws.fill_(255)  # NaN: nothing may be read before it is written
    e, f = _eval(gpu_lib, m, system, nl, ws, 0)
    e1, f1 = _eval(gpu_lib, m, system, nl, ws, 1)
    # the bounds of the blocks' other parity tests; one atom alone: no force
    assert rel_rmse(f, f1) <= (5e-3 if bf16 else 2e-6) if n > 1 else not f.any() and not f1.any()
    assert abs(e[0] - e1[0]) <= (2e-2 if bf16 else 1e-6) * abs(e1[0]) + (2e-2 * n if bf16 else 1e-4)
    if n < 100:
        E, F = om.cons_energy_forces(spec, w, pos, species, box, *oracle_list(pos, box, 5.0))
        assert n == 1 or rel_rmse(f, F) <= (1e-2 if bf16 else FP32_TOL)
        assert abs(e[0] - E) <= (2e-2 if bf16 else 1e-6) * abs(E) + (2e-2 * n if bf16 else 1e-4)


@pytest.mark.parametrize("n,third,box", [(3997, 300, 41.0), (5997, 400, 46.5)])
def test_bf16_tiles_give_the_same_bits(gpu_lib, n, third, box):
    """Two replicas alone, then with a third one: of 3,997 atoms in tiles of
    16 both times, of 5,997 in tiles of 16 and of 32 (every other choice by
    size is the same for both)."""
    spec = ModelSpec("cons", 128, 3, 16, 5.0)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 941), precision=1)
    a = small_box(942, n=n, box=box)
    b = small_box(943, n=third, box=17.5)
    out = []
    for reps in ([a, a], [a, a, b]):
        system = gpu_lib.DeviceSystem([r[0] for r in reps], [r[1] for r in reps], [r[2] for r in reps])
        nl = gpu_list(gpu_lib, system, 5.0)
        ws = gpu_lib.workspace(m, None, system.n, system.n_rep, nl.capacity)
        e, f = gpu_lib.nnp_cons_energy_forces(m, system, nl, ws)
        out.append((e[:2].clone(), f[:, :2 * n].clone()))
    assert torch.equal(out[0][1], out[1][1]) and torch.equal(out[0][0], out[1][0])
