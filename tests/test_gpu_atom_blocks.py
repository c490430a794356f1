"""Per-atom blocks of width-128 conservative models at sizes in tiles of 16
atoms, around multiples of 32: parity with the FP64 oracle and with the older
dense kernels, one to four layers, packed replicas, and the same bits every
time.  (Tiles of 32 atoms: test_gpu_atom_tiles.py, test_gpu_atom_last_tiles.py.)"""

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


@pytest.mark.parametrize("n,layers,bf16", [(1, 2, 0), (31, 1, 0), (32, 2, 0), (33, 3, 0), (64, 4, 0), (161, 2, 0),
                                           (31, 2, 1), (97, 3, 1)])
def test_blocks_at_tile_edges(gpu_lib, n, layers, bf16):
    spec = ModelSpec("cons", 128, layers, 16, 5.0)
    print(f"case n={n} layers={layers} bf16={bf16}", flush=True)
    pos, species, box = small_box(700 + n, n=n, box=max(11.0, (n / 0.06) ** (1.0 / 3.0)))
    w = random_weights(spec, 710 + n)
    m = gpu_lib.Model.from_spec(spec, w, precision=bf16)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.0)
    ws = gpu_lib.workspace(m, None, n, 1, nl.capacity)
    ws.fill_(255)  # NaN: nothing may be read before it is written
    e, f = _eval(gpu_lib, m, system, nl, ws, 0)
    e1, f1 = _eval(gpu_lib, m, system, nl, ws, 1)
    E, F = om.cons_energy_forces(spec, w, pos, species, box, *oracle_list(pos, box, 5.0))
    if n == 1:
        assert np.all(f == 0.0)
    else:
        # BF16: the bound of the other BF16 parity tests
        assert rel_rmse(f, F) <= (1e-2 if bf16 else FP32_TOL)
        assert rel_rmse(f, f1) <= (5e-3 if bf16 else 2e-6)
    assert abs(e[0] - E) <= (2e-2 if bf16 else 1e-6) * abs(E) + (2e-2 * n if bf16 else 1e-4)


def test_blocks_give_the_same_bits_and_replicas_do_not_mix(gpu_lib):
    spec = ModelSpec("cons", 128, 3, 16, 5.0)
    w = random_weights(spec, 731)
    m = gpu_lib.Model.from_spec(spec, w)
    boxes = [small_box(740 + r, n=k, box=14.0) for r, k in enumerate((33, 70, 128))]
    big = gpu_lib.DeviceSystem([b[0] for b in boxes] * 20, [b[1] for b in boxes] * 20, [b[2] for b in boxes] * 20)
    nl = gpu_list(gpu_lib, big, 5.0)
    ws = gpu_lib.workspace(m, None, big.n, big.n_rep, nl.capacity)
    runs = [gpu_lib.nnp_cons_energy_forces(m, big, nl, ws)[1].clone() for _ in range(6)]
    assert all(torch.equal(runs[0], r) for r in runs[1:])
    per = sum(b[0].shape[0] for b in boxes)
    first = runs[0][:, :per]
    assert all(torch.equal(first, runs[0][:, k * per:(k + 1) * per]) for k in range(20))
