"""Reverse by one message of each edge (FP32 models past the first layer, and
the first by species): atoms with more edges than a wavefront has lanes, with
one and with none, one to four layers, with and without the first layer by
species, packed replicas; forces and virials against the FP64 oracle and the
older kernels."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from oracle import models as om
from tests._helpers import FP32_TOL, gpu_list, oracle_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu

VIR_TOL = 2e-5  # relative, float32 path, as in the other virial tests


def _eval(nnp, m, system, nl, ws, dense, messages):
    from paper_2602_14975_amd import _abi
    _abi.check(nnp.lib().nnp_set_dense_kernels(dense))
    _abi.check(nnp.lib().nnp_set_message_kernels(messages))
    try:
        ws.fill_(255)  # NaN: nothing may be read before it is written
        e, f, W = nnp.nnp_cons_virial(m, system, nl, ws)
        return float(e.cpu()[0]), f.cpu().numpy().T.astype(np.float64), W.cpu().numpy()
    finally:
        nnp.lib().nnp_set_dense_kernels(0)
        nnp.lib().nnp_set_message_kernels(0)


# (n, box): 118 edges an atom; 16; about one; none for most
@pytest.mark.parametrize("n,box,layers", [(300, 11.0, 3), (300, 11.0, 1), (81, 14.0, 4), (81, 14.0, 2), (40, 26.0, 3),
                                          (24, 60.0, 2), (2, 60.0, 3)])
@pytest.mark.parametrize("messages", [0, 2])
def test_forces_and_virial(gpu_lib, n, box, layers, messages):
    print(f"case n={n} box={box} layers={layers} messages={messages}", flush=True)
    spec = ModelSpec("cons", 128, layers, 16, 5.0)
    pos, species, _ = small_box(980 + n, n=n, box=box)
    if n == 2:
        pos[1] = pos[0] + [0.9, -1.1, 0.7]
    w = random_weights(spec, 990 + n)
    m = gpu_lib.Model.from_spec(spec, w)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.2)
    ws = gpu_lib.workspace(m, None, n, 1, nl.capacity)
    e, f, W = _eval(gpu_lib, m, system, nl, ws, 0, messages)
    e1, f1, W1 = _eval(gpu_lib, m, system, nl, ws, 1, messages)  # no per-atom blocks: both messages of each edge
    off, nbr = oracle_list(pos, box, 5.0)
    E, F = om.cons_energy_forces(spec, w, pos, species, box, off, nbr)
    scale = VIR_TOL * (abs(om.cons_virial(spec, w, pos, species, box, off, nbr)) + 5.0 * np.abs(F).sum())
    assert rel_rmse(f, F) <= FP32_TOL and rel_rmse(f, f1) <= 2e-6
    assert abs(W[0] - om.cons_virial(spec, w, pos, species, box, off, nbr)) <= scale and abs(W[0] - W1[0]) <= scale
    assert abs(e - E) <= 1e-6 * abs(E) + 1e-4
    alone = np.bincount(np.repeat(np.arange(n), np.diff(off)), minlength=n) == 0
    assert np.all(f[alone] == 0.0)


def test_replicas_equal_alone(gpu_lib):
    spec = ModelSpec("cons", 128, 3, 16, 5.0)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 996))
    reps = [small_box(997 + k, n=n, box=b) for k, (n, b) in enumerate(((300, 11.0), (31, 20.0), (120, 13.0)))]
    pack = gpu_lib.DeviceSystem([r[0] for r in reps], [r[1] for r in reps], [r[2] for r in reps])
    nl = gpu_list(gpu_lib, pack, 5.4)
    ws = gpu_lib.workspace(m, None, pack.n, 3, nl.capacity)
    _, f, W = gpu_lib.nnp_cons_virial(m, pack, nl, ws)
    for k, (pos, species, box) in enumerate(reps):
        one = gpu_lib.DeviceSystem(pos, species, box)
        nl1 = gpu_list(gpu_lib, one, 5.0)
        ws1 = gpu_lib.workspace(m, None, one.n, 1, nl1.capacity)
        _, f1, W1 = gpu_lib.nnp_cons_virial(m, one, nl1, ws1)
        assert torch.equal(f[:, pack.rep_start[k]:pack.rep_start[k + 1]], f1) and W[k] == W1[0]
