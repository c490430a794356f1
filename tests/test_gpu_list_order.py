"""Lists of a caller whose rows do not ascend: energies, forces and virials are
those of the same entries in ascending order but for the order of the sums."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from tests._helpers import FP32_TOL, gpu_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers", [1, 3])
@pytest.mark.parametrize("messages", [0, 1, 2])
def test_rows_in_any_order(gpu_lib, layers, messages):
    from paper_2602_14975_amd import _abi
    print(f"case layers={layers} messages={messages}", flush=True)
    spec = ModelSpec("cons", 128, layers, 16, 5.0)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 1371))
    pos, species, box = small_box(1372, n=300, box=11.5)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.3, with_rev=False)
    ws = gpu_lib.workspace(m, None, system.n, 1, nl.capacity)
    off, nbr = nl.rows()
    rng = np.random.default_rng(1373)
    orders = (nbr, np.concatenate([nbr[a:b][::-1] for a, b in zip(off, off[1:])]),
              np.concatenate([rng.permutation(nbr[a:b]) for a, b in zip(off, off[1:])]))
    out = []
    _abi.check(gpu_lib.lib().nnp_set_message_kernels(messages))
    try:
        for rows in orders:
            nl.nbr[:len(rows)] = torch.as_tensor(np.ascontiguousarray(rows), device="cuda")
            ws.fill_(255)  # NaN: nothing may be read before it is written
            e, f, W = gpu_lib.nnp_cons_virial(m, system, nl, ws)
            out.append((float(e.cpu()[0]), f.cpu().numpy().astype(np.float64), float(W.cpu()[0])))
    finally:
        gpu_lib.lib().nnp_set_message_kernels(0)
    (e0, f0, w0), rest = out[0], out[1:]
    # the bounds against the oracle, which each of them keeps
    scale = 2e-5 * (abs(w0) + 5.0 * np.abs(f0).sum())
    for e, f, w in rest:
        assert rel_rmse(f, f0) <= 2 * FP32_TOL and abs(w - w0) <= 2 * scale
        assert abs(e - e0) <= 2e-6 * abs(e0) + 2e-4
