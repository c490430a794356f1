"""Reverse by one message of each edge with its rows in cell order (an
integration call's): the bisection over the neighbours' caller indices and the
stores through the permutation, rows of more than 64 edges and of few, packed
replicas, against the same positions in the caller's order, bit for bit."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from tests._helpers import gpu_list, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers", [1, 2, 3])
@pytest.mark.parametrize("messages", [0, 2])
def test_cell_order_rows(gpu_lib, layers, messages):
    from paper_2602_14975_amd import _abi
    print(f"case layers={layers} messages={messages}", flush=True)
    spec = ModelSpec("cons", 128, layers, 16, 5.0)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 1351))
    # 118 edges an atom on 3 x 3 x 3 cells, about three on 4 x 4 x 4
    reps = [small_box(1352, n=1000, box=16.5), small_box(1353, n=77, box=24.0)]
    _abi.check(gpu_lib.lib().nnp_set_message_kernels(messages))
    try:
        system = gpu_lib.DeviceSystem([r[0] for r in reps], [r[1] for r in reps], [r[2] for r in reps])
        n = system.n
        prm = gpu_lib.respa_params(0.05, 1, 0.0, seed=4000, mode="sts", skin=0.4)
        t = gpu_lib.Trajectory(m, None, system, np.zeros((n, 3)), np.full(n, 12.0), np.ones(n), prm, virial=True)
        t.respa_step(1)
        order = t.order[:n].cpu().numpy()
        assert not np.array_equal(order, np.arange(n)) and np.array_equal(np.sort(order), np.arange(n))
        nl = gpu_list(gpu_lib, system, 5.0)
        ws = gpu_lib.workspace(m, None, n, 2, nl.capacity)
        ws.fill_(255)  # NaN: nothing may be read before it is written
        e, f, W = gpu_lib.nnp_cons_virial(m, system, nl, ws)
        assert torch.equal(t.f_cons, f) and torch.equal(t.energy, e) and torch.equal(t.virial, W)
        off, _ = nl.rows()
        assert np.diff(off).max() > 64 and f.any()
    finally:
        gpu_lib.lib().nnp_set_message_kernels(0)
