"""Reductions of the NC weight gradient over rows: chunks of 256 rows and row
groups within them, per-species column sums, at the row counts where a chunk
or a group ends, against the FP64 oracle."""

import numpy as np
import pytest
import torch

from synth.weights import ModelSpec, manifest, random_weights
from oracle import models as om
from tests._helpers import gpu_list, oracle_list, rel_rmse, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,n_species,width", [(7, 1, 16), (85, 4, 32), (255, 8, 16), (256, 2, 32), (257, 5, 64),
                                              (1030, 8, 32)])
def test_weight_gradient_at_chunk_edges(gpu_lib, n, n_species, width):
    spec = ModelSpec("nc", width, 1, 8, 3.5, n_species=n_species)
    print(f"case n={n} S={n_species} width={width}", flush=True)
    pos, _, box = small_box(910 + n, n=n, box=max(8.0, (n / 0.08) ** (1.0 / 3.0)))
    rng = np.random.default_rng(n)
    species = rng.integers(0, n_species, size=n).astype(np.int32)
    w = random_weights(spec, 920 + n)
    g = rng.normal(size=(n, 3)).astype(np.float32)
    m = gpu_lib.Model.from_spec(spec, w)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 3.5)
    ws = gpu_lib.workspace(None, m, n, 1, nl.capacity)
    got = gpu_lib.nnp_nc_weight_grad(m, system, nl, torch.as_tensor(g.T.copy(), device="cuda"), ws).cpu().numpy()
    want = om.nc_weight_grad(spec, w, pos, species, box, *oracle_list(pos, box, 3.5), g)
    k = 0
    for name, shape, _ in manifest(spec):
        size = int(np.prod(shape))
        a, b = got[k:k + size], want[k:k + size]
        k += size
        # float32 adjoints of a few hundred terms each (1e-4 a tensor, as for the water boxes)
        assert np.linalg.norm(b) == 0 or rel_rmse(a, b) <= 1e-4, name
