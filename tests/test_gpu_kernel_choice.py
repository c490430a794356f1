"""The choice of message kernels while another thread changes it: every
evaluation runs on one choice from its first launch to its last, so that it
gives the bits of one of the three."""

import threading

import pytest
import torch

from synth.weights import ModelSpec, random_weights
from tests._helpers import gpu_list, small_box

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,bf16", [(1, 0), (2, 0), (3, 0), (2, 1)])
def test_an_evaluation_keeps_its_choice(gpu_lib, layers, bf16):
    print(f"case layers={layers} bf16={bf16}", flush=True)
    spec = ModelSpec("cons", 128, layers, 16, 5.0)
    pos, species, box = small_box(1210, n=60, box=11.0)
    m = gpu_lib.Model.from_spec(spec, random_weights(spec, 1211), precision=bf16)
    system = gpu_lib.DeviceSystem(pos, species, box)
    nl = gpu_list(gpu_lib, system, 5.0)
    ws = gpu_lib.workspace(m, None, system.n, 1, nl.capacity)
    choose = gpu_lib.lib().nnp_set_message_kernels
    stop = threading.Event()

    def toggle():
        k = 0
        while not stop.is_set():
            choose(k % 3)
            k += 1

    other = threading.Thread(target=toggle)
    try:
        want = []
        for mode in (0, 1, 2):
            assert choose(mode) == 0
            want.append([t.clone() for t in gpu_lib.nnp_cons_virial(m, system, nl, ws)])
        ws.fill_(255)  # NaN: nothing may be read that this evaluation did not write
        other.start()
        got = [[t.clone() for t in gpu_lib.nnp_cons_virial(m, system, nl, ws)] for _ in range(300)]
    finally:
        stop.set()
        if other.is_alive():
            other.join()
        choose(0)
    for k, g in enumerate(got):
        assert any(all(torch.equal(a, b) for a, b in zip(g, w)) for w in want), f"evaluation {k}"
