"""NC evaluation kernels at the sizes where their chunks and tiles end: rows
of a few to more than 64 edges (the pair head takes 32 at a time), atom
counts around a wavefront's four owners, with the head over the message
step's records and the one that walks the list bit for bit the same."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, random_weights
from oracle import models as om
from tests._helpers import FP32_TOL, gpu_list, oracle_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,box,rc_list,width", [(1, 12.0, 3.5, 32), (5, 12.0, 4.5, 16), (67, 11.0, 3.5, 32),
                                                 (300, 11.0, 4.5, 16), (700, 11.0, 3.5, 32), (257, 12.0, 5.0, 8)])
def test_rows_of_all_lengths(gpu_lib, n, box, rc_list, width):
    spec = ModelSpec("nc", width, 1, 8, 3.5)
    print(f"case n={n} box={box} list={rc_list} width={width}", flush=True)
    pos, species, _ = small_box(860 + n, n=n, box=box)
    w = random_weights(spec, 870 + n)
    m = gpu_lib.Model.from_spec(spec, w)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, rc_list)
    ws = gpu_lib.workspace(None, m, n, 1, nl.capacity)
    ws.fill_(255)  # NaN: nothing may be read before it is written
    f = gpu_lib.nnp_nc_forces(m, system, nl, ws)
    fl = gpu_lib.nnp_nc_forces_noalloc(m, system, nl)
    assert torch.equal(f, fl)
    fv, vir = gpu_lib.nnp_nc_virial(m, system, nl, ws)
    assert torch.equal(f, fv)
    F = om.nc_forces(spec, w, pos, species, box, *oracle_list(pos, box, 3.5))
    got = f.cpu().numpy().T.astype(np.float64)
    if n == 1:
        assert np.all(got == 0.0) and float(vir[0]) == 0.0
        return
    assert rel_rmse(got, F) <= FP32_TOL
    W = om.nc_virial_proxy(spec, w, pos, species, box, *oracle_list(pos, box, 3.5))
    # float32 shares whose signs differ: the sum of their sizes is at most sum |F| r
    assert abs(float(vir[0]) - W) <= 1e-5 * (abs(W) + 3.5 * np.abs(F).sum())
