"""Device bytes that a server reckons for a replica: no more than when the list
build kept nothing between its passes and the dense kernels had buffers of
their own, so that a budget holds the replicas it held then."""

import pytest

from synth.weights import ModelSpec, random_weights

pytestmark = pytest.mark.gpu

REPLICAS = ((192, 12.4), (1000, 21.5), (1536, 24.8))


# (conservative width, layers, precision, NC width): bytes of each replica then,
# of a server of 256 MiB with eight slots
@pytest.mark.parametrize("shape,then", [
    ((8, 1, 0, 8), (2750410, 14196566, 21801235)),
    ((16, 2, 1, 16), (3598803, 18613126, 28584798)),
    ((32, 1, 0, 32), (4338150, 22455272, 34485236)),
    ((64, 2, 0, 32), (6994477, 36281687, 55721512)),
    ((128, 1, 0, 32), (13106997, 67908484, 104302956)),
    ((128, 3, 0, 32), (18808708, 97604894, 149916642)),
    ((128, 3, 1, 16), (18439095, 95684136, 146966907)),
])
def test_replica_bytes_have_not_grown(gpu_lib, shape, then):
    from paper_2602_14975_amd import serve
    width, layers, precision, nc_width = shape
    cs, ns = ModelSpec("cons", width, layers, 16, 5.0), ModelSpec("nc", nc_width, 1, 8, 3.5)
    cons = gpu_lib.Model.from_spec(cs, random_weights(cs, 1), precision=precision)
    nc = gpu_lib.Model.from_spec(ns, random_weights(ns, 2), precision=precision)
    server = serve.Server(cons, nc, gpu_lib.respa_params(2.0, 4, 300.0, seed=1), 256 << 20, 8)
    try:
        now = [server.replica_bytes(n, box) for n, box in REPLICAS]
    finally:
        server.close()
    assert all(a <= b for a, b in zip(now, then)), (now, then)
