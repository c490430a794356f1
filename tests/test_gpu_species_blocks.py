"""The first layer's products by species inside the per-atom blocks (up to six
species; more take launches of their own): species counts at both sides of
that, tile edges, one and two layers, against the separate products."""

import numpy as np
import pytest

from synth.weights import ModelSpec, random_weights
from tests._helpers import gpu_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_species,n,layers", [(1, 15, 2), (2, 33, 1), (3, 5419, 2), (4, 5450, 1), (6, 17, 2),
                                                (6, 5418, 1), (7, 100, 2), (8, 5420, 2)])
def test_species_counts(gpu_lib, n_species, n, layers):
    from paper_2602_14975_amd import _abi
    print(f"case species={n_species} n={n} layers={layers}", flush=True)
    spec = ModelSpec("cons", 128, layers, 16, 5.0, n_species=n_species)
    pos, _, box = small_box(1200 + n, n=n, box=max(11.0, (n / 0.06) ** (1.0 / 3.0)))
    species = np.random.default_rng(n_species).integers(0, n_species, size=n).astype(np.int32)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 1210 + n_species))
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.0)
    ws = gpu_lib.workspace(m, None, n, 1, nl.capacity)
    out = []
    for mode in (0, 1):
        _abi.check(gpu_lib.lib().nnp_set_dense_kernels(mode))
        try:
            ws.fill_(255)  # NaN: nothing may be read before it is written
            e, f = gpu_lib.nnp_cons_energy_forces(m, system, nl, ws)
        finally:
            gpu_lib.lib().nnp_set_dense_kernels(0)
        out.append((float(e.cpu()[0]), f.cpu().numpy().astype(np.float64)))
    (e0, f0), (e1, f1) = out
    # the bounds of the blocks' other parity tests
    assert rel_rmse(f0, f1) <= 2e-6
    assert abs(e0 - e1) <= 1e-6 * abs(e1) + 1e-4
