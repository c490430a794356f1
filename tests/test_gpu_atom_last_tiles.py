"""Per-atom blocks in tiles of 32 atoms: last tiles whose second group of 16
atoms is absent, present in part and all but whole, and the same bits every
time, at sizes past the tiles of 16 (5,418 atoms FP32, 12,288 BF16), against
the older dense kernels.  (Last tiles of 1 to 12 atoms: test_gpu_atom_tiles.py,
test_gpu_species_blocks.py.)"""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from tests._helpers import gpu_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


def _eval(nnp, model, system, nl, ws, mode):
    from paper_2602_14975_amd import _abi
    _abi.check(nnp.lib().nnp_set_dense_kernels(mode))
    try:
        ws.fill_(255)  # NaN: nothing may be read before it is written
        e, f = nnp.nnp_cons_energy_forces(model, system, nl, ws)
        return float(e.cpu()[0]), f.cpu().numpy().astype(np.float64)
    finally:
        nnp.lib().nnp_set_dense_kernels(0)


@pytest.mark.parametrize("n,layers,n_species,bf16", [
    (5424, 1, 4, 0), (5424, 3, 4, 0), (5425, 2, 1, 0), (5425, 2, 8, 0), (5439, 2, 6, 0), (5439, 1, 4, 0),
    (12304, 2, 4, 1), (12305, 3, 4, 1), (12305, 1, 4, 1), (12319, 2, 4, 1)])
def test_last_tile(gpu_lib, n, layers, n_species, bf16):
    print(f"case n={n} layers={layers} species={n_species} bf16={bf16}", flush=True)
    spec = ModelSpec("cons", 128, layers, 16, 5.0, n_species=n_species)
    pos, _, box = small_box(1300 + n, n=n, box=(n / 0.06) ** (1.0 / 3.0))
    species = np.random.default_rng(n).integers(0, n_species, size=n).astype(np.int32)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 1310 + n), precision=bf16)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.0)
    ws = gpu_lib.workspace(m, None, n, 1, nl.capacity)
    e, f = _eval(gpu_lib, m, system, nl, ws, 0)
    e1, f1 = _eval(gpu_lib, m, system, nl, ws, 1)
    # the bounds of the blocks' other parity tests, over all atoms and over
    # those of the last tile
    tail = slice(n // 32 * 32, n)
    for a, b in ((f, f1), (f[:, tail], f1[:, tail])):
        assert rel_rmse(a, b) <= (5e-3 if bf16 else 2e-6)
    assert abs(e - e1) <= (2e-2 if bf16 else 1e-6) * abs(e1) + (2e-2 * n if bf16 else 1e-4)


@pytest.mark.parametrize("copies,bf16", [(30, 0), (60, 1)])
def test_the_same_bits_and_replicas_do_not_mix(gpu_lib, copies, bf16):
    """231 atoms in three replicas, 6,930 and 13,860 atoms packed: copies lie at
    every place of a tile."""
    spec = ModelSpec("cons", 128, 3, 16, 5.0)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 1331), precision=bf16)
    boxes = [small_box(1340 + r, n=k, box=14.0) for r, k in enumerate((33, 70, 128))]
    big = gpu_lib.DeviceSystem([b[0] for b in boxes] * copies, [b[1] for b in boxes] * copies,
                               [b[2] for b in boxes] * copies)
    nl = gpu_list(gpu_lib, big, 5.0)
    ws = gpu_lib.workspace(m, None, big.n, big.n_rep, nl.capacity)
    runs = []
    for _ in range(6):
        ws.fill_(255)
        runs.append([t.clone() for t in gpu_lib.nnp_cons_energy_forces(m, big, nl, ws)])
    assert all(torch.equal(runs[0][0], r[0]) and torch.equal(runs[0][1], r[1]) for r in runs[1:])
    e, f = runs[0]
    assert torch.equal(f, f[:, :231].repeat(1, copies)) and torch.equal(e, e[:3].repeat(copies))
