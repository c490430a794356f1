"""Neighbour rows around the lengths where the fill changes its way (128
entries kept by the count; pairs of 64 lanes; four keys per read) and at the
longest row, against the oracle, and in the working order of the integrator."""

import numpy as np
import pytest

from tests._helpers import gpu_list, oracle_list

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k", [2, 64, 65, 66, 68, 128, 129, 130, 131, 193, 1000, 1025])
def test_rows_of_every_kind(gpu_lib, k):
    """A cluster of k atoms (rows of k - 1 entries) beside a sparse gas, in a
    shuffled order."""
    print(f"case k={k}", flush=True)
    rng = np.random.default_rng(1000 + k)
    d = rng.normal(size=(k, 3))
    cluster = np.array([25.0, 4.0, 13.0]) + 1.2 * d / np.linalg.norm(d, axis=1, keepdims=True)
    gas = rng.uniform(0.0, 31.0, size=(150, 3))
    pos = np.concatenate([cluster, gas])[rng.permutation(k + 150)]
    system = gpu_lib.DeviceSystem(pos, np.zeros(len(pos), np.int32), 31.0)
    want_off, want = oracle_list(pos, 31.0, 3.0)
    assert np.diff(want_off).max() >= k - 1
    if np.diff(want_off).max() > 1024:  # past the longest row: refused
        with pytest.raises(Exception, match="1024"):
            gpu_list(gpu_lib, system, 3.0, capacity=k * k + 8192)
        return
    nl = gpu_list(gpu_lib, system, 3.0, capacity=k * k + 8192)
    off, nbr = nl.rows()
    assert np.array_equal(off, want_off) and np.array_equal(nbr, want)


def test_two_builds_in_one_workspace(gpu_lib):
    """The second build starts from the counters that the first one left."""
    from paper_2602_14975_amd.nnp import NeighborList, workspace
    rng = np.random.default_rng(1100)
    ws = workspace(None, None, 900, 1, 1)
    ws.fill_(255)
    for n, box in ((900, 31.0), (500, 16.0), (900, 40.0)):
        pos = rng.uniform(0.0, box, size=(n, 3))
        system = gpu_lib.DeviceSystem(pos, np.zeros(n, np.int32), box)
        nl = NeighborList(n, 5.0, 200000, with_rev=True)
        gpu_lib.nnp_neighbors(system, nl, ws)
        off, nbr = nl.rows()
        want_off, want = oracle_list(pos, box, 5.0)
        assert np.array_equal(off, want_off) and np.array_equal(nbr, want)
